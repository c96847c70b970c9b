// Joint text+image attention, O = softmax(Q K^T / sqrt(d)) V per head and per
// request, never materialising the L x L score matrix (online softmax over
// 64-key tiles).
//
// bf16 kernel (head_dim 128 or 64) on the gfx950 matrix cores.  Each wavefront owns
// 32 queries.  It computes the transposed score tile S^T = K Q^T with
// v_mfma_f32_32x32x16_bf16, so every lane holds the scores of ONE query
// (column lane % 32) for half of the keys: the row max and row sum are
// register reductions plus one exchange with lane ^ 32, no LDS.  The
// probabilities are rounded to bf16 and fed straight from registers as the B
// operand of O^T = V^T P^T; for that V is kept transposed (V^T [d][keys]) and
// its 16-key groups are stored in LDS in the order the score registers hold
// them.  K and V^T tiles are double-buffered in LDS (XOR-swizzled 16-byte
// chunks); the softmax runs in the log2 domain (exp2 with log2(e)/sqrt(d)
// folded into the scale).  Blocks of one head are mapped onto one XCD so its
// K/V tiles are shared through that XCD's L2.
#include <float.h>
#include <math.h>

#include <algorithm>

#include "device_common.h"

namespace dit {

namespace {

// q-tiles of every request of the batch, longest requests first
struct AttnSched {
  int n;                     // number of requests with tokens
  int req[kMaxReq];
  int tile_off[kMaxReq + 1]; // prefix sum of q-tiles per head
};

// Lazy rescaling: the running max used for exp2 is only raised when a new
// score exceeds it by more than 2^RESCALE_SLACK; until then probabilities may
// reach 2^8, which fp32 and bf16 hold exactly as well as any other value.
// O and l always share the max they were computed with, so O / l is exact.
constexpr float RESCALE_SLACK = 8.0f;

// Scheduling pattern for a run of N (LDS read, MFMA) pairs where MFMA i uses
// read i: the first A reads, then one MFMA and one read alternately, then the
// last A MFMAs -- A fragment reads stay in flight ahead of the matrix cores.
template <int N, int A>
__device__ __forceinline__ void sched_read_ahead() {
  __builtin_amdgcn_sched_group_barrier(0x100, A, 0);
  static_for<N - A>([&](auto) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  });
  __builtin_amdgcn_sched_group_barrier(0x008, A, 0);
}

// s_waitcnt with vmcnt = 0 and the other counters left alone (gfx9 encoding).
__device__ __forceinline__ void wait_vmcnt0() { __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8)); }
// s_waitcnt with vmcnt = 0 and lgkmcnt = 0: this wave's tile loads have
// landed and its LDS fragment reads have returned
__device__ __forceinline__ void wait_vmcnt0_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(7 << 4); }

// NW waves x 32 queries per block, head dimension HD (64 or 128), BKV keys
// (64 or 128) per tile.
//
// Pipeline over key tiles j: K and V^T tiles arrive by direct-to-LDS buffer
// loads in two stages, tile j + 1 loading while tile j runs scores, softmax
// and P V in turn.
//
// KG = 2: two groups of NW waves share the block's queries and split its key
// tiles into a first and a second half, each group with LDS stages of its
// own; the second group hands its O, max and sum to the first through LDS at
// the end.  For launches that leave CUs with one block or none: a lone block
// of 4 waves runs its tiles one after the other at one wave per SIMD.
//
// attn_unit: the block's work on query tile q0 of head h of request r against
// key tiles [jb0, je0).  part < 0: all keys, O is written; otherwise its
// unnormalised O, maxima and sums go to slot `part` of the `parts` in
// a.split_buf.  smem: KG * STAGES tile pairs, free again when it returns.
template <int NW, int HD, int STAGES, int BKV, int KG>
__device__ __forceinline__ void attn_unit(const AttnArgs& a, char* smem, int r, int h, int q0, int jb0, int je0,
                                          int part, int parts) {
  static_assert(STAGES == 2, "two LDS stages, the loop is unrolled over them");
  constexpr int BQ = NW * 32;
  static_assert(HD == 64 || HD == 128, "head dim");
  static_assert(BKV == 64 || BKV == 128, "key tile");
  constexpr int CH = HD / 8;       // 16-byte chunks per key row of the K tile
  constexpr int KPI = 64 / CH;     // keys per load instruction (64 lanes x 16 bytes)
  constexpr int VCH = BKV / 8;     // 16-byte chunks per d row of the V^T tile
  constexpr int VRPI = 64 / VCH;   // V^T rows per load instruction
  constexpr int KT_U4 = BKV * CH;  // K tile: [BKV keys][CH chunks of 8 d], chunk slot swizzled by kswz
  constexpr int VT_U4 = HD * VCH;  // V^T tile: [HD d][VCH chunks of 8 key slots], chunk slot swizzled by vswz
  constexpr int KI = BKV / KPI / NW;  // K-tile load instructions per wave
  constexpr int VI = HD / VRPI / NW;  // V^T-tile load instructions per wave
  static_assert(KI * KPI * NW == BKV && VI * VRPI * NW == HD, "tile config");
  // slot of chunk c in key row `key` / V^T row `dr`: the 16 rows one
  // ds_read_b128 serves per cycle land on 16 different 16-byte bank groups
  // (an involution in c)
  auto kswz = [](int key, int c) { return HD == 128 ? c ^ (key & 15) : c ^ ((key >> 1) & 7); };
  auto vswz = [](int dr, int c) { return BKV == 128 ? c ^ (dr & 15) : c ^ ((dr >> 1) & 7); };
  const int L = a.meta.joint_off[r + 1] - a.meta.joint_off[r];

  const int tid = threadIdx.x, lane = tid & 63;
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / NW;  // key group
  const int wave = (tid >> 6) - kg * NW;                                      // query wave
  const int hl = lane >> 5;  // lane half

  const bf16_t* __restrict__ Qg = (const bf16_t*)a.q + (long)a.qk_off[r] * a.q_tok + (long)h * a.q_head;
  const bf16_t* __restrict__ Kg = (const bf16_t*)a.k + (long)a.qk_off[r] * a.k_tok + (long)h * a.k_head;
  const bf16_t* __restrict__ Vg = (const bf16_t*)a.vt + (long)a.vt_off[r] + (long)h * a.vt_head;
  const int Lpad = a.vt_off[r + 1] - a.vt_off[r];

  // K and V^T tiles move by range-checked buffer loads straight into LDS
  // (64 lanes x 16 bytes per wave instruction, no registers).  Each lane's
  // byte offset inside a tile is fixed here; a tile only moves the buffer's
  // base.  Keys past L fall outside the K buffer of the tile and read as
  // zeros (their scores are masked); V^T columns past L lie in the request's
  // zeroed padding.
  int kvo[KI], vvo[VI];
#pragma unroll
  for (int q = 0; q < KI; ++q) {
    const int key = (wave * KI + q) * KPI + lane / CH;
    kvo[q] = (key * (int)a.k_tok + kswz(key, lane % CH) * 8) * 2;
  }
#pragma unroll
  for (int q = 0; q < VI; ++q) {
    const int dr = (wave * VI + q) * VRPI + lane / VCH;
    vvo[q] = (dr * (int)a.vt_d + vswz(dr, lane % VCH) * 8) * 2;
  }
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  constexpr int STAGE_B = (KT_U4 + VT_U4) * 16;
  char* const lbase = smem + kg * STAGES * STAGE_B;
  auto tile_load = [&](int j, auto stc) __attribute__((always_inline)) {
    constexpr int st = decltype(stc)::value;
    const int kv0 = j * BKV;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Kg + (long)kv0 * a.k_tok), (short)0, ((L - 1 - kv0) * (int)a.k_tok + HD) * 2, kBufferWord3);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Vg + kv0), (short)0, ((HD - 1) * (int)a.vt_d + Lpad - kv0) * 2, kBufferWord3);
#pragma unroll
    for (int q = 0; q < KI; ++q) {
      const int vo = kvo[q];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rk, (__attribute__((address_space(3))) void*)(lbase + st * STAGE_B + (wv * KI + q) * KPI * CH * 16), 16,
          vo, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < VI; ++q) {
      const int vo = vvo[q];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rv, (__attribute__((address_space(3))) void*)(lbase + st * STAGE_B + KT_U4 * 16 + (wv * VI + q) * VRPI * VCH * 16),
          16, vo, 0, 0, 0);
    }
  };

  const int nt_all = (L + BKV - 1) / BKV;
  // this group's share: the first half, rounded up, or the rest
  const int half = (je0 - jb0 + KG - 1) / KG;
  const int jb = jb0 + kg * half, je = KG == 1 ? je0 : min(jb + half, je0);
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  if (KG == 1 || jb < je) tile_load(jb, S0{});

  // Q fragments (B operand of S^T = K Q^T): query q0 + wave*32 + lane%32, d chunk 2*ks + lane/32
  const int qrow = q0 + wave * 32 + (lane & 31);
  bf16x8_t qf[HD / 16];
#pragma unroll
  for (int ks = 0; ks < HD / 16; ++ks) {
    uint4 u = make_uint4(0, 0, 0, 0);
    if (qrow < L) u = *(const uint4*)(Qg + (long)qrow * a.q_tok + (ks * 2 + hl) * 8);
    qf[ks] = __builtin_bit_cast(bf16x8_t, u);
  }

  f32x16_t o[HD / 32];
#pragma unroll
  for (int db = 0; db < HD / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  // The running max starts at the lowest finite value: a range of keys whose
  // scores are all -inf then adds nothing (from -inf it would give -inf - -inf),
  // wherever the query's keys are cut into ranges.
  float m_i = -FLT_MAX, l_i = 0.f;
  const float sl2 = a.scale * 1.4426950408889634f;

  // S^T of one 64-key tile: two 32x32 blocks (keys kb*32 + (i/4)*8 + hl*4 + i%4 of
  // register i, query lane % 32)
  // Per-lane LDS byte offsets of the fragment reads, fixed before the loop:
  // K fragment of k-step ks (key lane % 32 of key block 0; key block 1 is
  // 32 rows further) and V^T fragment of key step ks2 (d row lane % 32 of d
  // block 0; d block db is 32 rows further).  Stage and block offsets are
  // immediates of the reads.
  int kfo[HD / 16], vfo[BKV / 16];
#pragma unroll
  for (int ks = 0; ks < HD / 16; ++ks) kfo[ks] = ((lane & 31) * CH + kswz(lane & 31, ks * 2 + hl)) * 16;
#pragma unroll
  for (int ks2 = 0; ks2 < BKV / 16; ++ks2) {
    const int dr = lane & 31;
    vfo[ks2] = KT_U4 * 16 + (dr * VCH + vswz(dr, ks2 * 2 + hl)) * 16;
  }
  auto lds_frag = [&](int byte_off) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8_t, *(const uint4*)(lbase + byte_off));
  };

  // S^T of one key tile: BKV / 32 blocks of 32x32 (keys kb*32 + (i/4)*8 + hl*4 + i%4 of
  // register i, query lane % 32)
  auto scores = [&](auto stc, f32x16_t* s) __attribute__((always_inline)) {
    constexpr int st = decltype(stc)::value;
#pragma unroll
    for (int kb = 0; kb < BKV / 32; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < HD / 16; ++ks) {
#pragma unroll
      for (int kb = 0; kb < BKV / 32; ++kb) {
        // key kb*32 + lane%32 keeps the swizzle term of key lane%32 (kb*32 is a multiple of 16)
        const bf16x8_t u = lds_frag(kfo[ks] + st * STAGE_B + kb * 32 * CH * 16);
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u, qf[ks], s[kb], 0, 0, 0);
      }
    }
    // keep four fragment reads ahead of the MFMAs that consume them
    sched_read_ahead<BKV / 32 * HD / 16, 4>();
  };
  // Probabilities of one tile against the running max m_i, rounded to bf16 in
  // the order the P V operand wants them (key pairs packed by one convert);
  // returns this lane's sum of the rounded values (two bf16 products per
  // v_dot2 with (1, 1)), which is also what O accumulates.
  auto exps_pack = [&](const f32x16_t* s, bf16x8_t* pf) __attribute__((always_inline)) {
    float t0 = 0.f, t1 = 0.f;
    const bf16x2_t one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int x = 0; x < BKV / 16; ++x) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = (x & 1) * 8 + 2 * e;
        // v_exp_f32 directly: results below 2^-126 flush to zero, which the
        // softmax sum and the bf16 probabilities cannot tell from their true value
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[x >> 1][i], sl2, -m_i));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[x >> 1][i + 1], sl2, -m_i));
        const bf16x2_t pk = {(__bf16)p0, (__bf16)p1};
        if (e & 1) t1 = __builtin_amdgcn_fdot2_f32_bf16(pk, one, t1, false);
        else t0 = __builtin_amdgcn_fdot2_f32_bf16(pk, one, t0, false);
        w[e] = __builtin_bit_cast(uint32_t, pk);
      }
      pf[x] = __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
    }
    return t0 + t1;
  };
  // Online softmax of tile j's scores, then O += P V.  The probabilities are
  // first taken against the current running max; only if some lane's sum
  // exceeds 2^RESCALE_SLACK (or overflows, as on the first tile) is the true
  // row max formed, the max raised, O and l rescaled, and the tile redone.
  // O and l always share the max they were computed with, so O / l is exact.
  // Only a request's last key tile can hold keys past L, and only that tile
  // is run with masking (a run-time test inside every tile is turned by the
  // compiler into a compare and select per score on every tile).
  auto softmax_pv = [&](int j, auto stc, auto maskc, f32x16_t* s) __attribute__((always_inline)) {
    constexpr int st = decltype(stc)::value;
    if constexpr (decltype(maskc)::value) {
      const int kv0 = j * BKV;
#pragma unroll
      for (int kb = 0; kb < BKV / 32; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = kv0 + kb * 32 + (i >> 2) * 8 + hl * 4 + (i & 3);
          if (key >= L) s[kb][i] = -INFINITY;
        }
    }
    bf16x8_t pf[BKV / 16];
    float t = exps_pack(s, pf);
    if (__any(!(t <= (float)(1 << (int)RESCALE_SLACK)))) {
      float mx = s[0][0];
#pragma unroll
      for (int kb = 0; kb < BKV / 32; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kb][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * sl2;
      const float m_new = fmaxf(m_i, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_i - m_new);
      m_i = m_new;
      l_i *= alpha;
#pragma unroll
      for (int db = 0; db < HD / 32; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
      t = exps_pack(s, pf);
    }
    l_i += t;
#pragma unroll
    for (int ks2 = 0; ks2 < BKV / 16; ++ks2) {
#pragma unroll
      for (int db = 0; db < HD / 32; ++db) {
        // d row db*32 + lane%32 keeps the swizzle term of row lane%32
        const bf16x8_t u = lds_frag(vfo[ks2] + st * STAGE_B + db * 32 * VCH * 16);
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u, pf[ks2], o[db], 0, 0, 0);
      }
    }
    sched_read_ahead<BKV / 16 * HD / 32, 4>();
  };
  // Tile j sits in stage j % 2.  Each tile starts with the loads of tile
  // j + 1 into the other stage (freed by the barrier that ended tile j - 1)
  // and ends with this wave's loads landed and a bare barrier: after it every
  // wave's part of tile j + 1 is in LDS and no wave reads tile j any more.
  // (A __syncthreads() fence would drain nothing more but costs a wait on
  // every outstanding memory operation.)
  f32x16_t sc_t[BKV / 32];
  wait_vmcnt0();
  asm volatile("s_barrier" ::: "memory");
  // The wait before the barrier also covers the LDS reads: the compiler may
  // place the last P V MFMAs (and the waits for their V^T fragments) after the
  // barrier, and the stage those fragments come from is reloaded right after
  // it by the other waves.
  auto step = [&](int j, auto stc, auto maskc) __attribute__((always_inline)) {
    constexpr int st = decltype(stc)::value;
    if (j + 1 < je) tile_load(j + 1, std::integral_constant<int, st ^ 1>{});
    scores(stc, sc_t);
    softmax_pv(j, stc, maskc, sc_t);
    wait_vmcnt0_lgkmcnt0();
    asm volatile("s_barrier" ::: "memory");
  };
  using NoMask = std::false_type;
  using Mask = std::true_type;
  // tiles [jb, jm) hold no key past L; tile jm (if any) is the request's last
  const int jm = (je == nt_all && L % BKV != 0) ? je - 1 : je;
  int j = jb;
  for (; j + 1 < jm; j += 2) {
    step(j, S0{}, NoMask{});
    step(j + 1, S1{}, NoMask{});
  }
  if (j < jm) step(j++, S0{}, NoMask{});
  if (j < je) {
    if (((j - jb) & 1) == 0) step(j, S0{}, Mask{});
    else step(j, S1{}, Mask{});
  }
  if constexpr (KG > 1) {
    // at most one tile fewer in the second group, which still meets the barrier
    if (je - jb < half) asm volatile("s_barrier" ::: "memory");
    // the groups' results meet as [wave][register][lane] in LDS, whose tiles
    // nobody reads any more
    constexpr int NR = HD / 2;  // O registers of a lane
    float* const sh = (float*)smem + (wave * (NR + 2)) * 64 + lane;
    static_assert(NW * (NR + 2) * 64 * 4 <= KG * STAGES * STAGE_B, "merge LDS");
    if (kg == 1) {
#pragma unroll
      for (int db = 0; db < HD / 32; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) sh[(db * 16 + i) * 64] = o[db][i];
      sh[NR * 64] = m_i;
      sh[(NR + 1) * 64] = l_i;
    }
    __syncthreads();
    if (kg == 1) return;
    // a group without a tile has the lowest max, sum 0 and O 0
    const float m1 = sh[NR * 64], mm = fmaxf(m_i, m1);
    const float a0 = __builtin_amdgcn_exp2f(m_i - mm), a1 = __builtin_amdgcn_exp2f(m1 - mm);
    m_i = mm;
    l_i = l_i * a0 + sh[(NR + 1) * 64] * a1;
#pragma unroll
    for (int db = 0; db < HD / 32; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] = o[db][i] * a0 + sh[(db * 16 + i) * 64] * a1;
  }

  const float l = l_i + __shfl_xor(l_i, 32, 64);
  if (part >= 0) {
    // a key range: O unnormalised, with its max m_i and sum l (every range
    // holds at least one key, so both are finite), for the merge
    const long qs = (long)part * BQ + wave * 32 + (lane & 31);  // query slot
    float* po = a.split_buf + qs * HD;
#pragma unroll
    for (int db = 0; db < HD / 32; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(float4*)(po + db * 32 + g * 8 + hl * 4) =
            make_float4(o[db][g * 4 + 0], o[db][g * 4 + 1], o[db][g * 4 + 2], o[db][g * 4 + 3]);
    if (hl == 0) {
      float2* pml = (float2*)(a.split_buf + (long)parts * BQ * HD);
      pml[qs] = make_float2(m_i, l);
    }
    return;
  }
  if (qrow < L) {
    const float inv = 1.0f / l;
    const int row = a.o_stream_major ? padded_to_row(a.meta, r, qrow) : a.meta.joint_off[r] + qrow;
    bf16_t* og = (bf16_t*)a.o + (long)row * a.o_tok + (long)h * a.o_head;
#pragma unroll
    for (int db = 0; db < HD / 32; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dd = db * 32 + g * 8 + hl * 4;
        uint2 w;
        w.x = pack_bf16x2(o[db][g * 4 + 0] * inv, o[db][g * 4 + 1] * inv);
        w.y = pack_bf16x2(o[db][g * 4 + 2] * inv, o[db][g * 4 + 3] * inv);
        *(uint2*)(og + dd) = w;
      }
  }
}

template <int NW, int HD, int STAGES, int BKV, int KG>
__global__ __launch_bounds__(NW * KG * 64)
    __attribute__((amdgpu_waves_per_eu(HD == 64 ? (NW * KG == 8 ? 4 : 3) : 2)))
void attn_bf16_kernel(const AttnArgs a, const AttnSched sc) {
  __shared__ uint4 smem[KG * STAGES * BKV * HD / 4];  // [stage][K tile | V^T tile]
  const int per_head = sc.tile_off[sc.n];
  // unit (query tile x head) of this block and, on a key-split launch, its
  // key range: blocks of one XCD take consecutive indices, and a split
  // launch numbers the pieces key range first, so the blocks of one XCD
  // share K/V ranges
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  int piece = 0, id = bid;
  if (a.kv_pieces > 1) {
    piece = bid / a.units;
    id = bid - piece * a.units;
  }
  id += a.unit0;
  const int h = id / per_head;
  const int t = id - h * per_head;
  int slot = 0;
  while (slot + 1 < sc.n && t >= sc.tile_off[slot + 1]) ++slot;
  const int r = sc.req[slot];
  const int nt = (a.meta.joint_off[r + 1] - a.meta.joint_off[r] + BKV - 1) / BKV;
  attn_unit<NW, HD, STAGES, BKV, KG>(a, (char*)smem, r, h, (t - sc.tile_off[slot]) * NW * 32,
                                     piece * nt / a.kv_pieces, (piece + 1) * nt / a.kv_pieces,
                                     a.kv_pieces > 1 ? bid : -1, a.units * a.kv_pieces);
}

// ---- Evenly shared key tiles.  Query tiles of 256 come in whole rounds of one
// per CU only for few shapes, and a last round that is not full costs a whole
// tile's time (16 896 tokens, 6 heads: 396 tiles in 2 rounds, 77% of them
// filled).  Here the first rounds run as whole tiles, and every key tile of the
// others is one step of a line (groups of equally long requests, longest
// first; in a group head by head, tile by tile) that kStreamBlocks blocks cut
// into equal runs.  A run holds the end of one query tile, whole tiles, and the
// beginning of another: the whole ones are written, the two ends go to slots
// 2 b and 2 b + 1, and a second kernel adds each cut tile's parts in key order.
constexpr int kStreamBlocks = 256;
struct AttnStream {
  int n_groups;
  int slot0[kMaxReq + 1];  // requests (AttnSched slots) of each group
  int skip;                // whole tiles of group 0 that ran before
  int steps, run;          // key tiles in all, and per block
};

// where step s of the line falls: query tile (group, unit) and the line's steps [begin, end) of that tile
struct StreamAt {
  int group, unit, begin, end;
};
__device__ __forceinline__ StreamAt stream_at(const AttnArgs& a, const AttnSched& sc, const AttnStream& st, int bkv,
                                              int s) {
  StreamAt at;
  int base = 0;
  for (int g = 0;; ++g) {
    const int r = sc.req[st.slot0[g]];
    const int nt = (a.meta.joint_off[r + 1] - a.meta.joint_off[r] + bkv - 1) / bkv;
    const int skip = g == 0 ? st.skip : 0;
    const int units = a.heads * (sc.tile_off[st.slot0[g + 1]] - sc.tile_off[st.slot0[g]]) - skip;
    if (g + 1 == st.n_groups || s < base + units * nt) {
      const int u = (s - base) / nt;
      at.group = g;
      at.unit = u + skip;
      at.begin = base + u * nt;
      at.end = at.begin + nt;
      return at;
    }
    base += units * nt;
  }
}
// request, head and first query of a unit
__device__ __forceinline__ void stream_unit(const AttnSched& sc, const AttnStream& st, const StreamAt& at, int bq,
                                            int& r, int& h, int& q0) {
  const int t0 = sc.tile_off[st.slot0[at.group]], per_head = sc.tile_off[st.slot0[at.group + 1]] - t0;
  h = at.unit / per_head;
  const int t = t0 + at.unit - h * per_head;
  int slot = st.slot0[at.group];
  while (slot + 1 < st.slot0[at.group + 1] && t >= sc.tile_off[slot + 1]) ++slot;
  r = sc.req[slot];
  q0 = (t - sc.tile_off[slot]) * bq;
}

template <int HD, int BKV>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void attn_stream_kernel(const AttnArgs a, const AttnSched sc, const AttnStream st) {
  constexpr int NW = 8;
  __shared__ uint4 smem[2 * BKV * HD / 4];
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int s0 = b * st.run, s1 = min(s0 + st.run, st.steps);
#pragma unroll 1
  for (int s = s0; s < s1;) {
    const StreamAt at = stream_at(a, sc, st, BKV, s);
    const int e = min(at.end, s1);
    int r, h, q0;
    stream_unit(sc, st, at, NW * 32, r, h, q0);
    const bool whole = s == at.begin && e == at.end;
    attn_unit<NW, HD, 2, BKV, 1>(a, (char*)smem, r, h, q0, s - at.begin, e - at.begin,
                                 whole ? -1 : s == s0 ? 2 * b : 2 * b + 1, 2 * kStreamBlocks);
    s = e;
  }
}

// Adds the parts of the query tile that the start of run blockIdx.x + 1 cuts
// (nothing to do if it cuts none, or if an earlier run's start cuts the same
// tile): O = sum_p 2^(m_p - M) O_p / sum_p 2^(m_p - M) l_p in key order.  64
// queries per block, four threads per query.
template <int HD, int BKV>
__global__ __launch_bounds__(256) void attn_stream_merge_kernel(const AttnArgs a, const AttnSched sc,
                                                                const AttnStream st) {
  constexpr int BQ = 256, DH = HD / 4;
  const int b1 = blockIdx.x + 1, cut = b1 * st.run;
  if (cut >= st.steps) return;
  const StreamAt at = stream_at(a, sc, st, BKV, cut);
  if (at.begin == cut || at.begin < cut - st.run) return;
  // a start at the tile's own first step does not cut it: the run before b1 is
  // the first with a part (its last segment, or its only one)
  int r, h, q0;
  stream_unit(sc, st, at, BQ, r, h, q0);
  const int ql = blockIdx.y * 64 + (threadIdx.x >> 2), dd = (threadIdx.x & 3) * DH;
  const int qrow = q0 + ql, L = a.meta.joint_off[r + 1] - a.meta.joint_off[r];
  if (qrow >= L) return;
  const int bb = b1 - 1, be = (at.end - 1) / st.run;
  // run p's part: its first segment (slot 2 p) if the tile began at or before the run did
  auto slot = [&](int p) { return (long)(2 * p + (at.begin <= p * st.run ? 0 : 1)) * BQ + ql; };
  const float2* pml = (const float2*)(a.split_buf + 2L * kStreamBlocks * BQ * HD);
  float M = -INFINITY;
  for (int p = bb; p <= be; ++p) M = fmaxf(M, pml[slot(p)].x);
  float acc[DH] = {}, lsum = 0.f;
  for (int p = bb; p <= be; ++p) {
    const long qs = slot(p);
    const float2 ml = pml[qs];
    const float w = exp2f(ml.x - M);
    lsum = fmaf(w, ml.y, lsum);
    const float4* src = (const float4*)(a.split_buf + qs * HD + dd);
#pragma unroll
    for (int c = 0; c < DH / 4; ++c) {
      const float4 v = src[c];
      acc[4 * c + 0] = fmaf(w, v.x, acc[4 * c + 0]);
      acc[4 * c + 1] = fmaf(w, v.y, acc[4 * c + 1]);
      acc[4 * c + 2] = fmaf(w, v.z, acc[4 * c + 2]);
      acc[4 * c + 3] = fmaf(w, v.w, acc[4 * c + 3]);
    }
  }
  const float inv = 1.0f / lsum;
  const int row = a.o_stream_major ? padded_to_row(a.meta, r, qrow) : a.meta.joint_off[r] + qrow;
  bf16_t* og = (bf16_t*)a.o + (long)row * a.o_tok + (long)h * a.o_head + dd;
#pragma unroll
  for (int c = 0; c < DH / 8; ++c) {
    uint4 w;
    w.x = pack_bf16x2(acc[8 * c + 0] * inv, acc[8 * c + 1] * inv);
    w.y = pack_bf16x2(acc[8 * c + 2] * inv, acc[8 * c + 3] * inv);
    w.z = pack_bf16x2(acc[8 * c + 4] * inv, acc[8 * c + 5] * inv);
    w.w = pack_bf16x2(acc[8 * c + 6] * inv, acc[8 * c + 7] * inv);
    *(uint4*)(og + 8 * c) = w;
  }
}

// Merge of a key-split launch: for each query of unit unit0 + blockIdx.x, the
// KP key ranges' unnormalised outputs O_p with maxima m_p (log2 domain) and
// sums l_p combine as O = sum_p 2^(m_p - M) O_p / sum_p 2^(m_p - M) l_p with
// M = max_p m_p, added in piece order.  Two threads per query, HD / 2
// dimensions each.
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(const AttnArgs a, const AttnSched sc) {
  constexpr int BQ = 128;
  constexpr int DH = HD / 2;
  const int u = blockIdx.x;
  const int id = a.unit0 + u;
  const int per_head = sc.tile_off[sc.n];
  const int h = id / per_head;
  const int t = id - h * per_head;
  int slot = 0;
  while (slot + 1 < sc.n && t >= sc.tile_off[slot + 1]) ++slot;
  const int r = sc.req[slot];
  const int ql = threadIdx.x >> 1, part = threadIdx.x & 1;
  const int qrow = (t - sc.tile_off[slot]) * BQ + ql;
  const int L = a.meta.joint_off[r + 1] - a.meta.joint_off[r];
  if (qrow >= L) return;
  const int KP = a.kv_pieces, U = a.units;
  const float2* pml = (const float2*)(a.split_buf + (long)U * KP * BQ * HD);
  float M = -INFINITY;
  for (int p = 0; p < KP; ++p) M = fmaxf(M, pml[(long)(p * U + u) * BQ + ql].x);
  float acc[DH];
#pragma unroll
  for (int i = 0; i < DH; ++i) acc[i] = 0.f;
  float lsum = 0.f;
  for (int p = 0; p < KP; ++p) {
    const long qs = (long)(p * U + u) * BQ + ql;
    const float2 ml = pml[qs];
    const float w = exp2f(ml.x - M);
    lsum = fmaf(w, ml.y, lsum);
    const float4* src = (const float4*)(a.split_buf + qs * HD + part * DH);
#pragma unroll
    for (int c = 0; c < DH / 4; ++c) {
      const float4 v = src[c];
      acc[4 * c + 0] = fmaf(w, v.x, acc[4 * c + 0]);
      acc[4 * c + 1] = fmaf(w, v.y, acc[4 * c + 1]);
      acc[4 * c + 2] = fmaf(w, v.z, acc[4 * c + 2]);
      acc[4 * c + 3] = fmaf(w, v.w, acc[4 * c + 3]);
    }
  }
  const float inv = 1.0f / lsum;
  const int row = a.o_stream_major ? padded_to_row(a.meta, r, qrow) : a.meta.joint_off[r] + qrow;
  bf16_t* og = (bf16_t*)a.o + (long)row * a.o_tok + (long)h * a.o_head + part * DH;
#pragma unroll
  for (int c = 0; c < DH / 8; ++c) {
    uint4 w;
    w.x = pack_bf16x2(acc[8 * c + 0] * inv, acc[8 * c + 1] * inv);
    w.y = pack_bf16x2(acc[8 * c + 2] * inv, acc[8 * c + 3] * inv);
    w.z = pack_bf16x2(acc[8 * c + 4] * inv, acc[8 * c + 5] * inv);
    w.w = pack_bf16x2(acc[8 * c + 6] * inv, acc[8 * c + 7] * inv);
    *(uint4*)(og + 8 * c) = w;
  }
}

// ----------------------------------------------------------------------------
// fp32 attention (head_dim 64) for fp32 models, on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 products and sums).  A block owns 16 queries of
// a head; its four waves share out the 16-key tiles, each with its own running
// max, sum and O, and the four results are merged at the end in wave order.
// A tile's scores are S^T = K Q^T, so a lane holds four keys of one query; as in
// the bf16 kernel the probabilities feed O^T = V^T P^T from registers: MFMA
// step r of a tile takes key 4 (lane / 16) + r from every lane quarter, and
// V^T's 16-byte pieces hold the same keys (its middle quads are swapped in
// memory).  K and V^T go straight from memory to registers; the next tile's K
// replaces this one's once the scores are done, its V^T once O is.  The small
// model's launches (288 keys, 6 heads) are bound by latency: 108 blocks with 5
// tiles per wave; 13 us between events, launch included, against 98 us for four
// lanes per query on the vector ALUs.  Two or three tiles per step, or whole
// tiles loaded one step ahead into a second set of registers, are 0-4% slower
// over the small model's whole step (288 keys: 92.4, 93.0, 93.5 against 91.7 us;
// 2336 keys: 333, 348, 341 against 328 us).  exp2 of a log2(e)-scaled argument
// adds one rounding of the argument (about 2e-6 relative at the scores met).
constexpr int FD = 64;
constexpr int FQ = 16;

__global__ __launch_bounds__(256) void attn_f32_kernel(const AttnArgs a, const AttnSched sc) {
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ float osh[4][FQ][FD + 4];
  __shared__ float2 ml[4][FQ];  // running max (log2 domain) and sum
  const int per_head = sc.tile_off[sc.n], id = block_id();
  const int h = id / per_head;
  const int t = id - h * per_head;
  if (blockIdx.y > 0 && h >= a.heads) return;
  int slot = 0;
  while (slot + 1 < sc.n && t >= sc.tile_off[slot + 1]) ++slot;
  const int r = sc.req[slot];
  const int q0 = (t - sc.tile_off[slot]) * FQ;
  const int L = a.meta.joint_off[r + 1] - a.meta.joint_off[r];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, kq = lane >> 4;

  const float* Qg = (const float*)a.q + (long)a.qk_off[r] * a.q_tok + (long)h * a.q_head;
  const float* Kg = (const float*)a.k + (long)a.qk_off[r] * a.k_tok + (long)h * a.k_head;
  const float* Vg = (const float*)a.vt + (long)a.vt_off[r] + (long)h * a.vt_head;

  // dims 16 c + 4 kq .. + 3 of query lr (rows past L repeat the last query)
  float4 q[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) q[c] = *(const float4*)(Qg + (long)min(q0 + lr, L - 1) * a.q_tok + c * 16 + kq * 4);
  // V^T row 16 c + lr, the four slots that hold keys 4 kq .. + 3 of a tile
  const int vq = vt_slot(kq * 4);
  const int nt = (L + 15) / 16;
  const int t0 = wave * nt / 4, t1 = (wave + 1) * nt / 4;  // the wave's tiles
  float4 kf[4], vf[4];
  auto load_k = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      kf[c] = *(const float4*)(Kg + (long)min(j * 16 + lr, L - 1) * a.k_tok + c * 16 + kq * 4);
  };
  auto load_v = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) vf[c] = *(const float4*)(Vg + (long)(c * 16 + lr) * a.vt_d + j * 16 + vq);
  };
  auto at = [](const float4& v, auto ec) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value;
    return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
  };
  const float sl2 = a.scale * kLog2e;
  float m = -FLT_MAX, l = 0.f;   // m: of the query, in the log2 domain, finite (see attn_unit); l: of this lane's keys
  f32x4_t o[4] = {};             // O^T rows 16 c + 4 kq .. + 3 of query lr
  if (t0 < t1) {
    load_k(t0);
    load_v(t0);
  }
  for (int j = t0; j < t1; ++j) {
    // two chains of MFMAs: each result waits for the one before it
    f32x4_t s0 = {}, s1 = {};
#pragma unroll
    for (int c = 0; c < 4; c += 2)
      static_for<4>([&](auto ec) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(at(kf[c], ec), at(q[c], ec), s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(at(kf[c + 1], ec), at(q[c + 1], ec), s1, 0, 0, 0);
      });
    if (j + 1 < t1) load_k(j + 1);
    float s[4], mx = m;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = j * 16 + kq * 4 + i < L ? (s0[i] + s1[i]) * sl2 : -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float al = exp2f(m - mx);
    m = mx;
    l *= al;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = exp2f(s[i] - mx);
      l += s[i];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[c][i] *= al;
    static_for<4>([&](auto ec) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(at(vf[c], ec), s[decltype(ec)::value], o[c], 0, 0, 0);
    });
    if (j + 1 < t1) load_v(j + 1);
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (kq == 0) ml[wave][lr] = make_float2(m, l);
#pragma unroll
  for (int c = 0; c < 4; ++c) *(float4*)&osh[wave][lr][c * 16 + kq * 4] = make_float4(o[c][0], o[c][1], o[c][2], o[c][3]);
  __syncthreads();
  // 16 lanes per query, 4 dims each.  A wave without a tile has the lowest max and
  // weighs nothing; wave 3 always has one.
  const int ql = tid >> 4, dd = (tid & 15) * 4, qrow = q0 + ql;
  if (qrow >= L) return;
  float mm = ml[0][ql].x;
#pragma unroll
  for (int w = 1; w < 4; ++w) mm = fmaxf(mm, ml[w][ql].x);
  float ls = 0.f;
  float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float wt = exp2f(ml[w][ql].x - mm);
    const float4 v = *(const float4*)&osh[w][ql][dd];
    ls = fmaf(wt, ml[w][ql].y, ls);
    y = make_float4(fmaf(wt, v.x, y.x), fmaf(wt, v.y, y.y), fmaf(wt, v.z, y.z), fmaf(wt, v.w, y.w));
  }
  const float inv = 1.0f / ls;
  const int row = a.o_stream_major ? padded_to_row(a.meta, r, qrow) : a.meta.joint_off[r] + qrow;
  *(float4*)((float*)a.o + (long)row * a.o_tok + (long)h * a.o_head + dd) =
      make_float4(y.x * inv, y.y * inv, y.z * inv, y.w * inv);
}

AttnSched make_sched(const BatchMeta& m, int bq) {
  AttnSched sc{};
  int order[kMaxReq];
  int n = 0;
  for (int r = 0; r < m.n_req; ++r)
    if (m.joint_off[r + 1] > m.joint_off[r]) order[n++] = r;
  // longest requests first: their tiles take longest, start them early
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0; --j) {
      const int a = order[j - 1], b = order[j];
      if (m.joint_off[b + 1] - m.joint_off[b] > m.joint_off[a + 1] - m.joint_off[a]) {
        order[j - 1] = b;
        order[j] = a;
      }
    }
  sc.n = n;
  sc.tile_off[0] = 0;
  for (int i = 0; i < n; ++i) {
    const int r = order[i];
    sc.req[i] = r;
    const int L = m.joint_off[r + 1] - m.joint_off[r];
    sc.tile_off[i + 1] = sc.tile_off[i] + (L + bq - 1) / bq;
  }
  return sc;
}

}  // namespace

// keys per tile of the bf16 kernel; a request's V^T columns are padded to a
// multiple of kSeqPad, so a tile never reads past them
constexpr int kKeyTile = 64;
static_assert(kSeqPad % kKeyTile == 0, "V^T padding");

template <int NW, int HD, int KG = 1>
hipError_t launch_attn_cfg(const AttnArgs& a, hipStream_t s) {
  const AttnSched sc = make_sched(a.meta, NW * 32);
  const long blocks = (long)sc.tile_off[sc.n] * a.heads;
  if (blocks == 0) return hipSuccess;
  AttnArgs b = a;
  b.unit0 = 0;
  b.units = (int)blocks;
  b.kv_pieces = 1;
  hipLaunchKernelGGL((attn_bf16_kernel<NW, HD, 2, kKeyTile, KG>), dim3((unsigned)blocks), dim3(NW * KG * 64), 0, s, b,
                     sc);
  return hipGetLastError();
}

// Key split of the last round.  A launch of U 128-query units on the 512
// block slots of the GPU (two per CU) runs floor(U / 512) full rounds and a
// last one of T = U mod 512 units.  A unit alone on its CU runs about twice
// as fast as one of a pair, so a last round of up to 256 units costs about
// what its share of work would; below a quarter round, though, it still
// costs more (measured on MI355X at 16 384 tokens and head dim 128: 0.25 of
// a round of units took 0.37 of a round's time, 0.5 took 0.5).  When
// T <= 128 after R >= 2 full rounds, those T units instead run as T x P
// blocks of one key range each (P = floor(512 / T) >= 4 pieces, 1/P as long),
// and a merge kernel combines the pieces.  Measured against the unsplit
// launch at 16 384-17 152 tokens and 24-25 heads: 1.1-1.7% faster for
// T = 24-128 (P = 21-4), equal at P = 3 and 1% slower at P = 2, hence the
// bound.  Requests of one length only (the units of a mixed batch differ in
// cost), head dim 128.
struct SplitPlan {
  int main_units, tail_units, pieces;  // pieces 0: no split
};

constexpr int kAttnSlots = 2 * 256;  // 128-query blocks resident per GPU (two per CU, 256 CUs)

SplitPlan split_plan(const BatchMeta& m, int heads, int head_dim) {
  SplitPlan p{0, 0, 0};
  if (head_dim != 128) return p;
  const AttnSched sc = make_sched(m, 128);
  if (sc.n == 0) return p;
  const int L0 = m.joint_off[sc.req[0] + 1] - m.joint_off[sc.req[0]];
  for (int i = 1; i < sc.n; ++i)
    if (m.joint_off[sc.req[i] + 1] - m.joint_off[sc.req[i]] != L0) return p;
  const long units = (long)sc.tile_off[sc.n] * heads;
  const long full = units / kAttnSlots, tail = units % kAttnSlots;
  if (full < 2 || tail == 0 || 4 * tail > kAttnSlots) return p;
  const int key_tiles = (L0 + kKeyTile - 1) / kKeyTile;
  const int pieces = (int)std::min<long>(kAttnSlots / tail, key_tiles);
  if (pieces < 2) return p;
  p.main_units = (int)(full * kAttnSlots);
  p.tail_units = (int)tail;
  p.pieces = pieces;
  return p;
}

// The plan of evenly shared key tiles: R whole rounds, then equal runs.  It is
// taken where it is modelled 2% below what the launch would otherwise be, in
// steps (one key tile of a 256-query block on a full GPU, 1.67 us), from
// timings at 1 357 - 16 896 tokens and 3 - 24 heads:
//  shared out: a tile of n keys costs n + 4, and a run 28 more than its length
//  (its two ends written and merged);
//  256-query tiles in rounds: the last round, at most as long as a full one,
//  costs 0.35 + 0.75 of its fill (power lets fewer busy CUs run faster), 0.9
//  of that if it is the only one;
//  128-query blocks: they share out by themselves, but their K / V^T tiles serve
//  half the queries, 1.07 + 8 / n of the even share.
// Against the launch used otherwise (us, 24 heads unless said): 16 896 tokens
// 3017 -> 2810, 12 heads 1550 -> 1436, 6 heads 769 -> 749; 8 612 tokens 851 ->
// 797; 768 + 1 536 + 4 608 + 16 896 tokens 3313 -> 3186.  Not taken: 4 608 tokens
// (equal), 8 612 with 12 heads (2% slower), 16 896 with 3 heads (4% slower).
struct StreamPlan {
  AttnSched sc;
  AttnStream st;
  int main_units;
};

static_assert(kAttnShareBytes >= (size_t)2 * kStreamBlocks * 256 * (128 + 2) * sizeof(float), "slots of the runs' ends");

bool stream_plan(const BatchMeta& m, int heads, int head_dim, StreamPlan* out) {
  if (head_dim != 128) return false;
  StreamPlan p{};
  p.sc = make_sched(m, 256);
  if (p.sc.n == 0) return false;
  auto len = [&](int slot) { return m.joint_off[p.sc.req[slot] + 1] - m.joint_off[p.sc.req[slot]]; };
  long steps = 0, units0 = 0;
  int n0 = 0;
  for (int i = 0; i < p.sc.n;) {
    int j = i;
    while (j < p.sc.n && len(j) == len(i)) ++j;
    const long units = (long)heads * (p.sc.tile_off[j] - p.sc.tile_off[i]);
    const int nt = (len(i) + kKeyTile - 1) / kKeyTile;
    if (i == 0) {
      units0 = units;
      n0 = nt;
    }
    steps += units * nt;
    p.st.slot0[p.st.n_groups++] = i;
    p.st.slot0[p.st.n_groups] = j;
    i = j;
  }
  if (steps >= (1L << 30)) return false;
  const long rounds = units0 / kStreamBlocks;
  p.main_units = (int)(rounds * kStreamBlocks);
  p.st.skip = p.main_units;
  p.st.steps = (int)(steps - (long)p.main_units * n0);
  p.st.run = (p.st.steps + kStreamBlocks - 1) / kStreamBlocks;
  const double shared = (double)rounds * (n0 + 4) + p.st.run + 28;
  const long last = units0 % kStreamBlocks;  // 256-query tiles of the last round
  double other = (1.07 + 8.0 / n0) * (double)steps / kStreamBlocks;
  if (p.st.n_groups == 1 && 2 * last > kStreamBlocks) {  // where 256-query tiles would run
    const double part = std::min(1.0, 0.35 + 0.75 * (double)last / kStreamBlocks);
    other = (n0 + 4) * (rounds > 0 ? (double)rounds + part : 0.9 * part);
  }
  if (p.st.steps == 0 || shared > 0.98 * other) return false;
  *out = p;
  return true;
}

size_t split_bytes(const SplitPlan& p, int head_dim) {
  return p.pieces ? (size_t)p.tail_units * p.pieces * 128 * (head_dim + 2) * sizeof(float) : 0;
}

// Measured on MI355X: software pipelines that overlap a tile's softmax with
// the next tile's score MFMAs (255 VGPRs, spills) or with the previous tile's
// P V MFMAs (separate K and V^T rings of 2 or 4 stages, ~205 VGPRs) gave the
// same bits and were no faster where attention matters most (16 896 tokens),
// so the plain order with 2 buffers is used.
// Block shape at head dim 128.  Blocks of 128 queries (4 waves) run two per
// CU; their last round of a launch holds the leftover blocks, and when these
// are at most one per CU each runs alone on its CU, much faster than as one
// of two.  Blocks of 256 queries (8 waves, one per CU) read each K/V tile once
// for twice the queries but get no such lone tail.  So with U units (128
// queries x heads) on 2 x 256 block slots, the 128-query blocks win when the
// 256-query launch's last round (of 256 slots) is at most half full and the
// 256-query blocks otherwise: with an even number of 128-query tiles per
// request that is frac(U / 512) <= 1/2; with an odd number each request
// adds a half-empty 256-query block (at 19 072 tokens, 24 heads: 1800
// blocks, a last round of 8; the 128-query blocks are 6% faster there).
// Measured on MI355X (in-process A/B) at
// 16 896 tokens: 6 heads (U = 792) 256-query blocks -11%, 12 heads (1584)
// +4%, 18 heads
// (2376) -7%, 24 heads (3168) +2%; at 4608 tokens: 24 heads (864) -4%,
// 48 heads (1728) +3%; whole steps at 256 px (144) +1.8% and 512 px (288)
// -0.9%.  The rule assumes equal units, i.e. requests of one length; for a
// batch of mixed lengths (longest first, so the last round holds the short
// units) the 128-query blocks are kept (the packed 256-2048 px step: +0.6%
// with 256-query blocks).
//
// At head dim 64 the softmax's vector work is the longer half of a tile, and
// more waves per SIMD fill it: 128-query blocks run three per CU (155 VGPRs, 768
// slots), 256-query blocks two (held to 128 VGPRs, 512 slots; one per CU at 153;
// 13 VGPRs are spilled, 21 in the kernel of two key groups, all of them in the
// masked last tile, none in the loop over the tiles).  wide_64() compares the two by their rounds, in units of the time a
// lone 128-query block takes for 1.3 times its keys, as measured at 1 792 -
// 16 717 tokens and 3 - 24 heads: a full round costs 1.6 (768 units) and 1.95
// (512 blocks), and the last round 0.4 / 0.87 / 1.36 for up to 1 / 2 / 3
// 128-query blocks per CU and 0.9 / 1.76 for up to 1 / 2 256-query blocks.  Up
// to 768 units the 128-query blocks are never slower.  In a batch of mixed
// lengths the last round holds the shortest tiles and costs less than this, so
// 256-query blocks are taken there only if they all fit at once (2097 + 1970
// tokens, 24 heads: 792 units in two rounds or 408 blocks in one).  Against one 256-query
// block per CU at every size: 210 units 75 -> 53 us, 528 101 -> 76, 840
// 154 -> 143, 1584 566 -> 481, 3144 1737 -> 1735; a packed batch of 589, 1357 and
// 4429 tokens (12 heads) 148 -> 110.
bool wide_64(long units, long units8) {
  if (units <= 768) return false;
  static const double narrow_last[] = {0.0, 0.4, 0.87, 1.36}, wide_last[] = {0.0, 0.9, 1.76};
  const double narrow = 0.2 + 1.6 * (double)(units / 768) + narrow_last[(units % 768 + 255) / 256];
  const double wide = 0.25 + 1.95 * (double)(units8 / 512) + wide_last[(units8 % 512 + 255) / 256];
  return wide < narrow;
}

// What a launch runs: its last query tiles' keys shared out evenly (stream
// plan), the keys of a short last round split (split plan), two key groups per
// block, or plain blocks of 256 or 128 queries.
enum AttnCfg { ATTN_SHARED = 0, ATTN_KEY_SPLIT, ATTN_KEY_GROUPS, ATTN_256, ATTN_128 };

AttnCfg pick_attn(const AttnArgs& a, StreamPlan* stream, SplitPlan* split) {
  if (a.split_buf && a.split_bytes >= kAttnShareBytes && stream_plan(a.meta, a.heads, a.head_dim, stream))
    return ATTN_SHARED;
  *split = split_plan(a.meta, a.heads, a.head_dim);
  if (split->pieces && a.split_buf && a.split_bytes >= split_bytes(*split, a.head_dim)) return ATTN_KEY_SPLIT;
  const AttnSched sc4 = make_sched(a.meta, 4 * 32);
  const long units = (long)sc4.tile_off[sc4.n] * a.heads;
  bool equal = true;
  const int L0 = a.meta.joint_off[sc4.req[0] + 1] - a.meta.joint_off[sc4.req[0]];
  for (int i = 1; i < sc4.n; ++i)
    equal = equal && a.meta.joint_off[sc4.req[i] + 1] - a.meta.joint_off[sc4.req[i]] == L0;
  // the 256-query launch's own block count (not units / 2 when a request has
  // an odd number of 128-query tiles) and the fill of its last round
  const AttnSched sc8 = make_sched(a.meta, 8 * 32);
  const long units8 = (long)sc8.tile_off[sc8.n] * a.heads;
  constexpr long kSlots8 = 256;  // 256-query blocks resident per GPU at head dim 128 (one per CU)
  const long last8 = units8 % kSlots8;
  const bool wide = a.head_dim == 128 ? equal && (last8 == 0 || 2 * last8 > kSlots8)
                                      : wide_64(units, units8) && (equal || units8 <= 512);
  // Two key groups per block where every block has a CU to itself and at least
  // 20 key tiles: 168 units x 28 tiles 62.6 -> 52.2 us at head dim 128 and 42.6
  // -> 36.9 at 64, 240 x 40 88.7 -> 81.4 and 57.5 -> 51.6, 240 x 20 32.2 -> 31.1
  // and 21.9 -> 21.3; equal at 12 tiles and up to 12% slower below (the second
  // group's tiles and the merge), equal or slower with more than 256 units.
  if (a.allow_split && units <= 256 && L0 >= 20 * kKeyTile) return ATTN_KEY_GROUPS;
  return wide ? ATTN_256 : ATTN_128;
}

template <int HD>
hipError_t launch_attn_hd(const AttnArgs& a, hipStream_t s) {
  StreamPlan p;
  SplitPlan sp;
  const AttnCfg cfg = pick_attn(a, &p, &sp);
  if constexpr (HD == 128) {
    if (cfg == ATTN_SHARED) {
      if (p.main_units) {
        AttnSched main = p.sc;
        main.n = p.st.slot0[1];
        AttnArgs b = a;
        b.unit0 = 0;
        b.units = p.main_units;
        b.kv_pieces = 1;
        hipLaunchKernelGGL((attn_bf16_kernel<8, HD, 2, kKeyTile, 1>), dim3((unsigned)p.main_units), dim3(512), 0, s, b,
                           main);
      }
      hipLaunchKernelGGL((attn_stream_kernel<HD, kKeyTile>), dim3(kStreamBlocks), dim3(512), 0, s, a, p.sc, p.st);
      hipLaunchKernelGGL((attn_stream_merge_kernel<HD, kKeyTile>), dim3(kStreamBlocks - 1, 4), dim3(256), 0, s, a, p.sc,
                         p.st);
      return hipGetLastError();
    }
    if (cfg == ATTN_KEY_SPLIT) {
      const AttnSched sc = make_sched(a.meta, 128);
      AttnArgs b = a;
      b.unit0 = 0;
      b.units = sp.main_units;
      b.kv_pieces = 1;
      hipLaunchKernelGGL((attn_bf16_kernel<4, HD, 2, kKeyTile, 1>), dim3((unsigned)sp.main_units), dim3(256), 0, s, b, sc);
      b.unit0 = sp.main_units;
      b.units = sp.tail_units;
      b.kv_pieces = sp.pieces;
      hipLaunchKernelGGL((attn_bf16_kernel<4, HD, 2, kKeyTile, 1>), dim3((unsigned)(sp.tail_units * sp.pieces)), dim3(256),
                         0, s, b, sc);
      hipLaunchKernelGGL((attn_merge_kernel<HD>), dim3((unsigned)sp.tail_units), dim3(256), 0, s, b, sc);
      return hipGetLastError();
    }
  }
  if (cfg == ATTN_KEY_GROUPS) return launch_attn_cfg<4, HD, 2>(a, s);
  if (cfg == ATTN_256) return launch_attn_cfg<8, HD>(a, s);
  return launch_attn_cfg<4, HD>(a, s);
}

hipError_t launch_attention_bf16(const AttnArgs& a, hipStream_t s) {
  if (a.head_dim == 128) return launch_attn_hd<128>(a, s);
  if (a.head_dim == 64) return launch_attn_hd<64>(a, s);
  return hipErrorInvalidValue;
}

const char* attention_bf16_config_name(const AttnArgs& a) {
  static const char* names[] = {"attention_bf16_shared", "attention_bf16_key_split", "attention_bf16_key_groups",
                                "attention_bf16_256", "attention_bf16_128"};
  StreamPlan p;
  SplitPlan sp;
  return names[pick_attn(a, &p, &sp)];
}

size_t attn_split_bytes(const BatchMeta& m, int heads, int head_dim) {
  return split_bytes(split_plan(m, heads, head_dim), head_dim);
}

hipError_t launch_attention_f32(const AttnArgs& a, hipStream_t s) {
  if (a.head_dim != FD) return hipErrorInvalidValue;
  const AttnSched sc = make_sched(a.meta, FQ);
  const long blocks = (long)sc.tile_off[sc.n] * a.heads;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(attn_f32_kernel, grid_of(blocks), dim3(256), 0, s, a, sc);
  return hipGetLastError();
}

}  // namespace dit
