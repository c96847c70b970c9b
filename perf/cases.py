"""Timed cases of the framework's public entry points.

Each case is one call (or, for a denoising step, the two calls) that a serving
program makes on the GPU: a whole denoising step (``dit_step`` or
``dit_step_noalloc``, then ``euler_update``), one transformer block of a
sequence-parallel group's step (``dit_block_forward``), or the joint attention
of a rank's heads (``dit_attention``).  Sizes are those of the served models
(``paper_2510_01565_amd/workloads.py``): the 3072-wide 57-block model and the
1536-wide 24-block model in bf16, and the small fp32 model, at 256 to 2048 px,
square and not, alone and packed.

A case is a dict of plain values:
  call   "step", "double", "single" or "attention"
  model  "flux", "sd3" or "small" (the small one is fp32); for "attention"
         only its head dimension and element type matter
  grids  token grids of the packed requests, "HxW,HxW,..."
  texts  their text token counts, "N,N,..."
  heads  (attention) heads this rank owns
  invariant  (bf16 steps and blocks) DIT_FLAG_BATCH_INVARIANT
  noalloc    (steps) the entry point without a workspace argument
"""
import dataclasses
import math

import torch

from paper_2510_01565_amd import dit, workloads

MODELS = {"flux": workloads.FLUX_FULL, "sd3": workloads.SD3_MEDIUM, "small": workloads.SMALL_BLOCK}
WEIGHT_STD = 0.02
DT = 1.0 / 28.0
MAX_TOKENS = 23808  # of a drawn block or attention call: the packed 256 + 512 + 1024 + 2048 px batch


def listed():
    return [
        # the smallest call: the fp32 model's whole step on one 256 px request; launches and latency count
        {"name": "step_small_f32_256px", "call": "step", "model": "small", "grids": "16x16", "texts": "32"},
        # one single-stream block at the smallest resolution served: weights read for few rows
        {"name": "single_256px", "call": "single", "model": "flux", "grids": "16x16", "texts": "512"},
        # one double-stream block at 512 px, the size of the block benchmark
        {"name": "double_512px", "call": "double", "model": "flux", "grids": "32x32", "texts": "512"},
        # the two block kinds at 1024 px, the resolution most requests have
        {"name": "double_1024px", "call": "double", "model": "flux", "grids": "64x64", "texts": "512"},
        {"name": "single_1024px", "call": "single", "model": "flux", "grids": "64x64", "texts": "512"},
        # the largest block: the 256 / 512 / 1024 / 2048 px requests packed into one batch
        {"name": "single_packed_mixed", "call": "single", "model": "flux", "grids": "16x16,32x32,64x64,128x128",
         "texts": "512,512,512,512"},
        # two requests of other aspect ratios (1216 x 832 px, and an odd grid with a short prompt), packed in the
        # mode in which a request's bits do not depend on its batch
        {"name": "double_ragged_invariant", "call": "double", "model": "flux", "grids": "52x76,47x63",
         "texts": "512,197", "invariant": True},
        # the second served model's joint block at 1024 px: narrower, 64-wide heads, 333 text tokens
        {"name": "sd3_double_1024px", "call": "double", "model": "sd3", "grids": "64x64", "texts": "333"},
        # attention of one rank of a 4-way sequence-parallel group at 2048 px: 6 of 24 heads over all tokens
        {"name": "attention_2048px_sp4", "call": "attention", "model": "flux", "grids": "128x128", "texts": "512",
         "heads": 6},
        # attention of one rank of a 2-way group of the second model over a packed batch
        {"name": "attention_sd3_packed_sp2", "call": "attention", "model": "sd3", "grids": "16x16,32x32,64x64",
         "texts": "333,333,333", "heads": 12},
        # the second model's whole step at 512 px, by the entry point for loops that may not allocate
        {"name": "step_sd3_512px_noalloc", "call": "step", "model": "sd3", "grids": "32x32", "texts": "333",
         "noalloc": True},
        # the headline workload: the whole 57-block step on one 1024 px request
        {"name": "step_flux_1024px", "call": "step", "model": "flux", "grids": "64x64", "texts": "512"},
    ]


def _draw_requests(rng, n, most, text):
    """n token grids of 16 to 128 a side (log-uniform, aspect ratios up to 2) with their text counts, `most` tokens in all."""
    grids, texts, left = [], [], most
    for k in range(n):
        room = left // (n - k)
        nt = text if rng.random() < 0.6 else rng.randint(1, text)
        h = math.exp(rng.uniform(math.log(16), math.log(128)))
        r = math.exp(rng.uniform(-0.35, 0.35))
        a, b = (min(128, max(12, round(x))) for x in (h * r, h / r))
        while a * b + nt > room:
            a, b = max(1, a * 7 // 8), max(1, b * 7 // 8)
        grids.append("%dx%d" % (a, b))
        texts.append("%d" % nt)
        left -= a * b + nt
    return ",".join(grids), ",".join(texts)


def draw(rng):
    call = rng.choices(["double", "single", "attention", "step", "small"], [4, 4, 4, 2, 1])[0]
    n = rng.choice([1, 1, 1, 2, 3, 4])
    if call == "small":
        g, t = [], []
        for _ in range(min(n, 3)):
            g.append("%dx%d" % (rng.randint(8, 32), rng.randint(8, 32)))
            t.append("%d" % rng.randint(1, 64))
        return {"call": "step", "model": "small", "grids": ",".join(g), "texts": ",".join(t)}
    model = "flux" if call == "single" else rng.choice(["flux", "flux", "sd3"])
    if call == "step":
        model = rng.choice(["flux", "sd3", "sd3"])
    text = 512 if model == "flux" else 333
    grids, texts = _draw_requests(rng, n, 4608 if call == "step" else MAX_TOKENS, text)
    case = {"call": call, "model": model, "grids": grids, "texts": texts}
    if call == "attention":
        case["heads"] = rng.choice([24, 12, 6, 3])
    elif rng.random() < 0.2:
        case["invariant"] = True
    return case


# ---------------------------------------------------------------------------- the calls
def _sizes(case):
    grids = [tuple(int(x) for x in g.split("x")) for g in case["grids"].split(",")]
    return grids, [int(x) for x in case["texts"].split(",")]


def _model(case):
    m = MODELS[case["model"]]
    if case["call"] == "double":
        return dataclasses.replace(m, n_double=1, n_single=0)
    if case["call"] == "single":
        return dataclasses.replace(m, n_double=0, n_single=1)
    return m


def _dtype(m):
    return torch.bfloat16 if m.dtype == "bf16" else torch.float32


class _Draws:
    """Seeded normal tensors on the GPU, in the order they are asked for."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, dtype, std=1.0):
        x = torch.randn(shape, generator=self.gen, device="cuda", dtype=dtype)
        return x if std == 1.0 else x.mul_(std)

    def uniform(self, n):
        return torch.rand(n, generator=self.gen, device="cuda").tolist()


def _inputs(case, seed):
    """Everything random of a case: weights and biases N(0, 0.02^2), activations N(0, 1)."""
    m, dr = _model(case), _Draws(seed)
    grids, texts = _sizes(case)
    ti, tt, dt = sum(h * w for h, w in grids), sum(texts), _dtype(m)
    x = {"t": dr.uniform(len(grids))}
    if case["call"] == "attention":
        for name in ("q", "k", "v"):
            x[name] = dr.normal((ti + tt, case["heads"], m.head_dim), dt)
        return x
    shapes = dit.weight_manifest(dit.make_config(m))
    x["w"] = {name: dr.normal(shape, dt, WEIGHT_STD) for name, shape in shapes}
    if case["call"] == "step":
        x["latents"] = dr.normal((ti, m.in_channels), dt)
        x["text"] = dr.normal((tt, m.text_dim), dt)
    else:
        x["hidden"] = dr.normal((tt + ti, m.hidden), torch.float32)
        x["cond"] = dr.normal((len(grids), m.hidden), torch.float32)
    return x


def prepare(case, seed):
    m = _model(case)
    grids, texts = _sizes(case)
    s = _inputs(case, seed)
    s["call"] = case["call"]
    s["batch"] = dit.Batch([g[0] for g in grids], [g[1] for g in grids], texts, s["t"])
    if case["call"] == "attention":
        s["dims"] = (case["heads"], m.head_dim, dit.DIT_BF16 if m.dtype == "bf16" else dit.DIT_F32)
        s["o"] = torch.empty_like(s["q"])
        s["ws_bytes"] = dit.attention_workspace_size(s["batch"], *s["dims"])
        s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device="cuda")
        return s
    s["cfg"] = dit.make_config(m, dit.DIT_FLAG_BATCH_INVARIANT if case.get("invariant") else 0)
    s["weights"] = dit.Weights(list(s["w"].values()))
    s["noalloc"] = bool(case.get("noalloc"))
    if not s["noalloc"]:
        s["ws_bytes"] = dit.workspace_size(s["cfg"], s["batch"])
        s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device="cuda")
    if case["call"] == "step":
        s["velocity"] = torch.empty_like(s["latents"])
        s["channels"], s["dtype"] = m.in_channels, dit.DIT_BF16 if m.dtype == "bf16" else dit.DIT_F32
        s["dt"] = [DT] * len(grids)
    return s


def run(s):
    if s["call"] == "attention":
        dit.dit_attention(s["batch"], *s["dims"], s["q"], s["k"], s["v"], s["o"], s["ws"], s["ws_bytes"])
        return s["o"]
    if s["call"] == "step":
        if s["noalloc"]:
            dit.dit_step_noalloc(s["cfg"], s["weights"], s["batch"], s["latents"], s["text"], s["velocity"])
        else:
            dit.dit_step(s["cfg"], s["weights"], s["batch"], s["latents"], s["text"], s["velocity"], s["ws"],
                         s["ws_bytes"])
        dit.euler_update(s["batch"], s["channels"], s["dtype"], s["latents"], s["velocity"], s["dt"])
        return {"velocity": s["velocity"], "latents": s["latents"]}
    # the residual stream is updated in place, as between the blocks of a step
    dit.dit_block_forward(s["cfg"], s["weights"], 0 if s["call"] == "double" else 1, 0, s["batch"], s["hidden"],
                          s["cond"], s["ws"], s["ws_bytes"])
    return s["hidden"]


def work(case):
    m = _model(case)
    grids, texts = _sizes(case)
    n_img = [h * w for h, w in grids]
    n, total, es = len(grids), sum(n_img) + sum(texts), 2 if m.dtype == "bf16" else 4
    if case["call"] == "attention":
        width = case["heads"] * m.head_dim
        return {"bytes": 4.0 * total * width * es,
                "flops": sum(4.0 * (a + b) ** 2 * width for a, b in zip(n_img, texts))}
    params = {name: math.prod(shape) for name, shape in dit.weight_manifest(dit.make_config(m))}
    if case["call"] == "step":
        return {"bytes": float(es * (sum(params.values()) + 4 * sum(n_img) * m.in_channels + sum(texts) * m.text_dim)),
                "flops": workloads.flops_per_step(m, texts, n_img)["total"]}
    h, f = m.hidden, m.mlp_ratio * m.hidden
    block = sum(v for k, v in params.items() if k.startswith(("double.", "single.")))
    rows = (12 if case["call"] == "double" else 3) * h  # modulation rows of one block
    linears = 3 * h + h + 2 * f  # output columns x input rows per token, over h
    attn = sum(4.0 * (a + b) ** 2 * h for a, b in zip(n_img, texts))
    return {"bytes": float(es * (block + rows * (h + 1)) + 8 * total * h),
            "flops": 2.0 * total * h * linears + attn + 2.0 * n * rows * h}


def tolerance(case):
    if case["model"] == "small":
        return {"rel": 1e-5, "max": 1e-4}
    if case["call"] == "attention":
        return {"rel": 1e-2, "max": 1e-1}
    if case["call"] == "step":
        return {"rel": 2e-2, "max": 2e-1}
    return {"rel": 1e-2, "max": 1e-1}


# ---------------------------------------------------------------------------- the same in 64 bits
def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _norm(x, shift, scale, eps):
    x = x - x.mean(-1, keepdim=True)
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * (1.0 + scale) + shift


def _rope(x, grid, theta):
    """Pairs of the first half of the head dimension rotate by the grid row, of the second by the column."""
    gh, gw = grid
    half = x.shape[-1] // 2
    p = torch.arange(gh * gw, device=x.device)
    w = theta ** (-2.0 * torch.arange(half // 2, device=x.device, dtype=torch.float64) / half)
    ang = torch.cat([(p // gw)[:, None] * w, (p % gw)[:, None] * w], 1)[:, None, :]
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()], -1).flatten(-2)


def _attend(q, k, v):
    out = torch.empty_like(q)
    for h in range(q.shape[1]):
        p = torch.softmax(q[:, h] @ k[:, h].T / math.sqrt(q.shape[-1]), -1)
        out[:, h] = p @ v[:, h]
    return out


class _Exact:
    def __init__(self, case, x):
        self.m, self.w = _model(case), x["w"]
        self.grids, self.texts = _sizes(case)
        self.off, self.tied = {}, self.m.tie_streams
        row = 0
        for i in range(self.m.n_double):
            for st in ("img",) if self.tied else ("img", "txt"):
                self.off["double.%d.%s" % (i, st)] = (row, 6)
                row += 6 * self.m.hidden
        for i in range(self.m.n_single):
            self.off["single.%d" % i] = (row, 3)
            row += 3 * self.m.hidden
        self.off["final"] = (row, 2)

    def linear(self, x, name):
        return x @ self.w[name + ".w"].double().T + self.w[name + ".b"].double()

    def mod(self, key, c):
        row, n = self.off[key]
        end = row + n * self.m.hidden
        y = torch.nn.functional.silu(c) @ self.w["mod.w"][row:end].double().T + self.w["mod.b"][row:end].double()
        return y.chunk(n, -1)

    def qkv(self, y):
        return [z.reshape(y.shape[0], self.m.heads, self.m.head_dim) for z in y.chunk(3, -1)]

    def rows(self):
        """Row ranges of each request: (text range, image range) of the stream-major order."""
        t, i = 0, sum(self.texts)
        for (h, w), nt in zip(self.grids, self.texts):
            yield slice(t, t + nt), slice(i, i + h * w)
            t, i = t + nt, i + h * w

    def double(self, i, x, c):
        m = self.m
        for r, (ts, im) in enumerate(self.rows()):
            st = {}
            for name, sl in (("txt", ts), ("img", im)):
                own = "img" if self.tied else name
                st[name] = (sl, "double.%d.%s." % (i, own), self.mod("double.%d.%s" % (i, own), c[r]))
            qkv = {}
            for name, (sl, pre, md) in st.items():
                qkv[name] = self.qkv(self.linear(_norm(x[sl], md[0], md[1], m.ln_eps), pre + "qkv"))
            for j in (0, 1):
                qkv["img"][j] = _rope(qkv["img"][j], self.grids[r], m.rope_theta)
            o = _attend(*(torch.cat([qkv["txt"][j], qkv["img"][j]]) for j in range(3))).flatten(1)
            nt = self.texts[r]
            for name, (sl, pre, md) in st.items():
                y = x[sl] + md[2] * self.linear(o[:nt] if name == "txt" else o[nt:], pre + "proj")
                z = _gelu(self.linear(_norm(y, md[3], md[4], m.ln_eps), pre + "mlp1"))
                x[sl] = y + md[5] * self.linear(z, pre + "mlp2")
        return x

    def single(self, i, x, c):
        m, pre = self.m, "single.%d." % i
        for r, (ts, im) in enumerate(self.rows()):
            sh, sc, g = self.mod("single.%d" % i, c[r])
            y = torch.cat([x[ts], x[im]])
            nt = self.texts[r]
            z = self.linear(_norm(y, sh, sc, m.ln_eps), pre + "lin1")
            q, k, v = self.qkv(z[:, :3 * m.hidden])
            q, k = (torch.cat([u[:nt], _rope(u[nt:], self.grids[r], m.rope_theta)]) for u in (q, k))
            o = torch.cat([_attend(q, k, v).flatten(1), _gelu(z[:, 3 * m.hidden:])], 1)
            y = y + g * self.linear(o, pre + "lin2")
            x[ts], x[im] = y[:nt], y[nt:]
        return x

    def step(self, x):
        m = self.m
        t = torch.tensor(x["t"], dtype=torch.float64, device="cuda")
        half = m.time_freq_dim // 2
        f = torch.exp(-math.log(10000.0) * torch.arange(half, dtype=torch.float64, device="cuda") / half)
        a = 1000.0 * t[:, None] * f
        c = self.linear(torch.cat([a.cos(), a.sin()], 1), "time_in1")
        c = self.linear(torch.nn.functional.silu(c), "time_in2")
        h = torch.cat([self.linear(x["text"].double(), "txt_in"), self.linear(x["latents"].double(), "img_in")])
        for i in range(m.n_double):
            h = self.double(i, h, c)
        for i in range(m.n_single):
            h = self.single(i, h, c)
        v = torch.empty_like(x["latents"], dtype=torch.float64)
        for r, (_, im) in enumerate(self.rows()):
            sh, sc = self.mod("final", c[r])
            lo = sum(self.texts)
            v[im.start - lo:im.stop - lo] = self.linear(_norm(h[im], sh, sc, m.ln_eps), "final")
        return {"velocity": v, "latents": x["latents"].double() - DT * v}


def exact(case, seed):
    x = _inputs(case, seed)
    grids, texts = _sizes(case)
    if case["call"] == "attention":
        out, at = torch.empty_like(x["q"], dtype=torch.float64), 0
        for (h, w), nt in zip(grids, texts):
            sl = slice(at, at + h * w + nt)
            out[sl] = _attend(x["q"][sl].double(), x["k"][sl].double(), x["v"][sl].double())
            at = sl.stop
        return out
    if case["call"] == "step":
        for k in ("1", "2"):  # the timestep MLP's two layers under one name each
            x["w"]["time_in%s.w" % k], x["w"]["time_in%s.b" % k] = x["w"]["time_in.w" + k], x["w"]["time_in.b" + k]
    e = _Exact(case, x)
    if case["call"] == "step":
        return e.step(x)
    return (e.double if case["call"] == "double" else e.single)(0, x["hidden"].double(), x["cond"].double())
