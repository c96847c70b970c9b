// bf16 GEMM on the gfx950 matrix cores: Y = A W^T + b, fp32 accumulation,
// with the step's fused epilogues (QKV scatter + 2-D RoPE, GELU, gated
// residual, plain stores).
//
// Both operands are K-contiguous ([M, K] and [N, K]), which is the layout
// v_mfma_f32_32x32x16_bf16 wants for its A and B lanes (8 consecutive K values
// per lane).  Tiles move global -> LDS -> registers -> MFMA:
//  * when K is a multiple of the K tile, with direct-to-LDS loads
//    (global_load_lds_dwordx4: each wave instruction writes 64 x 16 bytes of
//    LDS without passing through registers) into a ring of STAGES buffers, so
//    the loads of tile k + STAGES - 1 are in flight while tile k is multiplied;
//  * otherwise through registers into two buffers, zero-filling the K tail.
// LDS rows are XOR-swizzled per 16-byte chunk so that the 16 rows one
// ds_read_b128 serves per cycle hit all 64 banks.  Blocks are remapped so
// every XCD owns one contiguous range of output tiles (its L2 keeps the
// operand panels those tiles share), in a grouped-M order.  One launch may
// hold two problems ("groups") sharing N -- the text and image streams of a
// double-stream block -- so the small text GEMM fills otherwise idle CUs.
#include <string>

#include "device_common.h"

namespace dit {

namespace {


struct TileCoord {
  int group, m0, n0;
};

template <int BM, int BN>
__device__ __forceinline__ TileCoord tile_coord(const GemmProblem& P, int id) {
  const int tiles_n = (P.N + BN - 1) / BN;
  const int tm0 = (P.g[0].M + BM - 1) / BM;
  const int tiles0 = tm0 * tiles_n;
  int g = 0, tm = tm0;
  if (id >= tiles0) {
    g = 1;
    id -= tiles0;
    tm = (P.g[1].M + BM - 1) / BM;
  }
  // grouped order: 8 M-tiles share each run of N-tiles, for L2 reuse of both operands
  constexpr int GM = 8;
  const int per_group = GM * tiles_n;
  const int grp = id / per_group;
  const int first_m = grp * GM;
  const int gsize = min(tm - first_m, GM);
  const int in_grp = id - grp * per_group;
  TileCoord c;
  c.group = g;
  c.m0 = (first_m + in_grp % gsize) * BM;
  c.n0 = (in_grp / gsize) * BN;
  return c;
}

// LDS slot (in 16-byte chunks) of chunk `kc` of tile row `row` for rows of
// CPR chunks.  64 banks of 4 bytes serve 16 lanes of a ds_read_b128 per cycle:
// the 16 consecutive rows read at one chunk index must cover all banks.
template <int CPR>
__device__ __forceinline__ int lds_slot(int row, int kc) {
  if constexpr (CPR == 8) return row * 8 + (kc ^ ((row >> 1) & 7));  // 128-byte rows: pairs of rows share 64 banks
  else return row * 4 + (kc ^ ((row >> 2) & 3));                      // 64-byte rows: quads of rows share 64 banks
}

// s_waitcnt with vmcnt = n and the other counters left alone (gfx9 encoding:
// vmcnt[3:0] and [15:14], expcnt[6:4], lgkmcnt[11:8]).

template <int n>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(n >= 0 && n < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));
}

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// cache policy of a buffer access at agent scope (sc1)
constexpr int kAgentScope = 16;

// Single instructions as volatile asm statements, which the compiler keeps in
// the order written: a main loop built from them runs exactly its schedule.
// The compiler does not see what they do, so the loop that uses them issues
// its own LDS waits, and wait states separate its last MFMAs from any other
// reader of the accumulators.
template <int OFF>
__device__ __forceinline__ void asm_lds_read16(i32x4_t& d, int addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "i"(OFF));
}
__device__ __forceinline__ void asm_mfma16(f32x4_t& c, const i32x4_t& a, const i32x4_t& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// wait until at most N LDS operations of this wave are outstanding; none is
// emitted for N >= 15, since the counter never holds more than 15
template <int N>
__device__ __forceinline__ void asm_lgkm_wait() {
  if constexpr (N < 15) asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(N));
}

// ON: v, of an origin unknown to the compiler, so that what is computed from it
// stays in the branch that asks for it instead of moving ahead of that branch.
template <bool ON>
__device__ __forceinline__ int opaque(int v) {
  if constexpr (ON) asm volatile("" : "+v"(v));
  return v;
}

// One staged group of 32 rows x W columns of a tile, corner (m, n), bias added
// (staging pitch W + 4 floats).  Consecutive lanes take consecutive 16-byte
// pieces of an output row, so a wave's access covers whole runs of W columns;
// a lane's loads all leave before its first store (one in-order counter holds
// both).  H is a multiple of 64, the head dimension 64 or 128, and n and W are
// multiples of 16, so an 8-column piece lies in one head of one of Q, K, V or the
// MLP input, but a group of 48 columns need not.
// FAST: for group loops that are unrolled (see the kernel's epilogue).  m and n
// are scalars and with them the branches, no mode's address arithmetic runs for
// another mode, and whole groups of plain columns leave LDS entirely before they
// are stored, without a branch between their pieces.
template <int W, bool FAST>
__device__ __forceinline__ void epilogue_group(const EpiArgs& E, const RowEntry* rows, const float* stg, int m, int n,
                                               int M, int N, int lane) {
  constexpr int SP = W + 4;
  if (n >= N || m >= M) return;
  const int v0 = E.mode == EPI_QKV ? 2 * E.hidden : N, v1 = E.mode == EPI_QKV ? 3 * E.hidden : N;  // V columns
  const int hs = E.head_dim == 128 ? 7 : 6;  // its logarithm: 128 or 64 in bf16
  if (n < v1 && n + W > v0) {
    // A lane takes one column of the group.  Rows at consecutive positions of
    // one request are consecutive keys of V^T: two 16-key groups (four 16-byte
    // stores) when they start on one, else quads of keys (8-byte stores) between
    // up to three single keys at either end.  Image counts that are not a
    // multiple of 16 leave every later row unaligned; with a 2-byte store per
    // key a QKV launch of 8056 x 21504 x 3072 (67 x 116 image) took 896 us between
    // events, now 826, and 24 of 3414 x 4608 x 1536 93 -> 68 us each.
    const int ln = opaque<FAST>(lane), hn = n + ln - v0, h = hn >> hs, dd = hn - h * E.head_dim;
    if (ln < W && n + ln >= v0 && n + ln < v1 && n + ln < N) {
      bf16_t* vt = (bf16_t*)E.vt + ((long)h * E.head_dim + dd) * E.vt_ld;
      const int p0 = rows[0].pos;
      if (m + 31 < M && rows_consecutive(rows[0], rows[31], 32)) {
        if ((p0 & 15) == 0) {
#pragma unroll
          for (int r16 = 0; r16 < 32; r16 += 16) {
            // slot s of a group holds key vt_slot(s): swap the middle quads
            float w[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) w[q] = stg[(r16 + vt_slot(q)) * SP + ln];
            store16(vt + p0 + r16, w);
          }
        } else {
          const int a = -p0 & 3;  // rows ahead of the first whole quad
          const float* col = stg + a * SP + ln;
          for (int q = 0; q < a; ++q) vt[vt_slot(p0 + q)] = f2bf(stg[q * SP + ln]);
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            if (t == 7 && a > 0) break;
            uint2 w;
            w.x = pack_bf16x2(col[(4 * t) * SP], col[(4 * t + 1) * SP]);
            w.y = pack_bf16x2(col[(4 * t + 2) * SP], col[(4 * t + 3) * SP]);
            *(uint2*)(vt + vt_slot(p0 + a + 4 * t)) = w;
          }
          for (int q = 28 + a; a > 0 && q < 32; ++q) vt[vt_slot(p0 + q)] = f2bf(stg[q * SP + ln]);
        }
      } else {
        for (int q = 0; q < 32 && m + q < M; ++q) vt[vt_slot(rows[q].pos)] = f2bf(stg[q * SP + ln]);
      }
    }
    if (n >= v0 && n + W <= v1) return;
  }
  if (E.mode == EPI_RESID || E.mode == EPI_STORE_F32) {
    constexpr int PPR = W / 4, NP = 16 * PPR / 64;  // 16-byte pieces of a row, pieces of a lane in half the rows
    const int ln = opaque<FAST>(lane);
    float* const o = (float*)E.out + (long)m * E.ldo + n;
    const int last = M - 1 - m, cols = N - n;
    if constexpr (FAST) {
      if (E.mode == EPI_STORE_F32) {
        if (cols >= W) {
          float4 v[2 * NP];
#pragma unroll
          for (int t = 0; t < 2 * NP; ++t) {
            const int id = ln + 64 * t;
            v[t] = *(const float4*)&stg[id / PPR * SP + id % PPR * 4];
          }
#pragma unroll
          for (int t = 0; t < 2 * NP; ++t) {
            const int id = ln + 64 * t, r = id / PPR;
            if (r <= last) *(float4*)(o + (long)r * E.ldo + id % PPR * 4) = v[t];
          }
        } else if (ln < cols) {
          // a last group cut by N: one column per lane, row by row
#pragma unroll 1
          for (int r0 = 0; r0 < 32; r0 += 8) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = stg[(r0 + q) * SP + ln];
#pragma unroll
            for (int q = 0; q < 8; ++q)
              if (r0 + q <= last) o[(long)(r0 + q) * E.ldo + ln] = v[q];
          }
        }
        return;
      }
    }
#pragma unroll 1
    for (int l0 = ln; l0 < 128 * NP; l0 += 64 * NP) {
      float4 v[NP];
      if (FAST || E.mode == EPI_RESID) {  // N is a multiple of 4; pieces past the edges load the last row or piece
        const float* const gate = E.mods + E.gate_off + n;
#pragma unroll
        for (int t = 0; t < NP; ++t) {
          const int id = l0 + 64 * t, r = min(id / PPR, last), c = min(id % PPR * 4, cols - 4);
          v[t] = *(const float4*)(o + (long)r * E.ldo + c);
        }
#pragma unroll
        for (int t = 0; t < NP; ++t) {
          const int id = l0 + 64 * t, r = min(id / PPR, last), c = min(id % PPR * 4, cols - 4);
          const float4 g = *(const float4*)(gate + (long)rows[r].req * E.mods_ld + c);
          const float4 y = *(const float4*)&stg[r * SP + c];
          v[t].x += g.x * y.x;
          v[t].y += g.y * y.y;
          v[t].z += g.z * y.z;
          v[t].w += g.w * y.w;
        }
      } else {
#pragma unroll
        for (int t = 0; t < NP; ++t) {
          const int id = l0 + 64 * t;
          v[t] = *(const float4*)&stg[id / PPR * SP + id % PPR * 4];
        }
      }
#pragma unroll
      for (int t = 0; t < NP; ++t) {
        const int id = l0 + 64 * t, r = id / PPR, c = id % PPR * 4;
        float* const dst = o + (long)r * E.ldo + c;
        if (r > last) continue;
        if (FAST) {
          if (c < cols) *(float4*)dst = v[t];
        } else if (c + 4 <= cols) {
          *(float4*)dst = v[t];
        } else {
          if (c < cols) dst[0] = v[t].x;
          if (c + 1 < cols) dst[1] = v[t].y;
          if (c + 2 < cols) dst[2] = v[t].z;
        }
      }
    }
    return;
  }
  constexpr int PPR = W / 8, NP = 32 * PPR / 64;
  const int ln = opaque<FAST>(lane);
  if (FAST && (E.mode != EPI_QKV || n >= v1) && n + W <= N) {
    // whole pieces of columns that are stored side by side
    const bool mlp = E.mode == EPI_QKV;
    const long ld = mlp ? E.gelu_ld : E.ldo;
    bf16_t* const o = (bf16_t*)(mlp ? E.gelu_out : E.out) + (long)m * ld +
                      (mlp ? E.gelu_col0 + n - E.n_qkv : E.mode == EPI_GELU ? E.col0 + n : n);
    float v[NP][8];
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const float* const src = &stg[(ln + 64 * t) / PPR * SP + (ln + 64 * t) % PPR * 8];
      *(float4*)&v[t][0] = *(const float4*)src;
      *(float4*)&v[t][4] = *(const float4*)(src + 4);
    }
    if (E.mode != EPI_STORE_T)
#pragma unroll
      for (int t = 0; t < NP; ++t)
#pragma unroll
        for (int q = 0; q < 8; ++q) v[t][q] = gelu_tanh(v[t][q]);
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const int r = (ln + 64 * t) / PPR;
      uint4 w;
      w.x = pack_bf16x2(v[t][0], v[t][1]);
      w.y = pack_bf16x2(v[t][2], v[t][3]);
      w.z = pack_bf16x2(v[t][4], v[t][5]);
      w.w = pack_bf16x2(v[t][6], v[t][7]);
      if (m + r < M) *(uint4*)(o + (long)r * ld + (ln + 64 * t) % PPR * 8) = w;
    }
    return;
  }
#pragma unroll 1
  for (int t = 0; t < NP; ++t) {
    const int id = ln + 64 * t, r = id / PPR, c = id % PPR * 8, nc = n + c;
    float v[8];
    *(float4*)&v[0] = *(const float4*)&stg[r * SP + c];
    *(float4*)&v[4] = *(const float4*)&stg[r * SP + c + 4];
    bf16_t* dst;
    if (E.mode == EPI_QKV && nc < v0) {
      const int d = E.head_dim, k = nc >= E.hidden, hn = nc - k * E.hidden, h = hn >> hs, dd = hn - h * d;
      const RowEntry re = rows[r];  // garbage past row M, not used then
      if (m + r < M && re.gi >= 0) {
        const int half = d >> 1;
        const int pos = dd < half ? re.gi : re.gj;
        const float4* cs = (const float4*)(E.rope + pos * (d >> 2) + ((dd < half ? dd : dd - half) >> 1));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 t4 = cs[q];
          const float u0 = v[4 * q], w0 = v[4 * q + 1], u1 = v[4 * q + 2], w1 = v[4 * q + 3];
          v[4 * q] = u0 * t4.x - w0 * t4.y;
          v[4 * q + 1] = u0 * t4.y + w0 * t4.x;
          v[4 * q + 2] = u1 * t4.z - w1 * t4.w;
          v[4 * q + 3] = u1 * t4.w + w1 * t4.z;
        }
      }
      dst = (bf16_t*)(k ? E.k : E.q) + ((long)h * E.T + re.pos) * d + dd;
    } else {
      if (E.mode != EPI_STORE_T)
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = gelu_tanh(v[q]);
      if (E.mode == EPI_QKV) dst = (bf16_t*)E.gelu_out + (long)(m + r) * E.gelu_ld + E.gelu_col0 + (nc - E.n_qkv);
      else dst = (bf16_t*)E.out + (long)(m + r) * E.ldo + (E.mode == EPI_GELU ? E.col0 : 0) + nc;
    }
    if (m + r >= M || nc >= N || (nc >= v0 && nc < v1)) continue;
    if (nc + 8 <= N) {
      uint4 w;
      w.x = pack_bf16x2(v[0], v[1]);
      w.y = pack_bf16x2(v[2], v[3]);
      w.z = pack_bf16x2(v[4], v[5]);
      w.w = pack_bf16x2(v[6], v[7]);
      *(uint4*)dst = w;
    } else {
#pragma unroll
      for (int q = 0; q < 7; ++q)
        if (nc + q < N) dst[q] = f2bf(v[q]);
    }
  }
}

// 4-wave blocks run two per CU: at most 256 registers
template <int BM, int BN, int NWM, int NWN, int BK, int STAGES, bool DTL>
__global__ __launch_bounds__(NWM* NWN * 64, NWM * NWN == 4 ? 2 : 1) void gemm_bf16_kernel(const GemmProblem P) {
  constexpr int NT = NWM * NWN * 64;
  constexpr int NWAVES = NWM * NWN;
  constexpr int WTM = BM / NWM, WTN = BN / NWN;
  // wave tiles: rows in 32-row fragments; columns in 32-column fragments on
  // the register path, in 16-column fragments on the direct-to-LDS path
  constexpr int FM = WTM / 32, FN = WTN / 32, FN16 = WTN / 16;
  constexpr int CPR = BK / 8;                     // 16-byte chunks per tile row
  constexpr int STAGE = (BM + BN) * CPR;          // uint4 per stage
  static_assert(FM * 32 == WTM && FN16 * 16 == WTN && (DTL || FN * 32 == WTN), "wave tile");
  static_assert(FM >= 1 && FN16 >= 1 && (BK == 32 || BK == 64) && STAGES >= 2 && BK % 32 == 0, "tile config");
  static_assert(STAGES * STAGE * 16 <= 160 * 1024, "LDS");

  __shared__ uint4 lds[STAGES * STAGE];

  // tile of this block and, when K is split, its piece; the pieces of a tile
  // have consecutive indices and so run on one XCD
  int tile_id = xcd_remap(blockIdx.x, gridDim.x), piece = 0;
  const int np = DTL ? P.sk_p : 1;
  if (np > 1) {
    piece = tile_id % np;
    tile_id /= np;
  }
  const TileCoord tc = tile_coord<BM, BN>(P, tile_id);
  const int gi = tc.group;
  const bf16_t* __restrict__ A = (const bf16_t*)(gi ? P.g[1].A : P.g[0].A);
  const bf16_t* __restrict__ W = (const bf16_t*)(gi ? P.g[1].W : P.g[0].W);
  const long lda = gi ? P.g[1].lda : P.g[0].lda;
  const long ldw = gi ? P.g[1].ldw : P.g[0].ldw;
  const int M = gi ? P.g[1].M : P.g[0].M;
  const int K = gi ? P.g[1].K : P.g[0].K;
  const int N = P.N;
  const int m0 = tc.m0, n0 = tc.n0;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / NWN, wn = wave % NWN;

  // Accumulators.  Direct-to-LDS path: 16x16 blocks, the 32x32 fragment
  // (i, j) being the 2 x 2 blocks 2i.., 2j..; register path: 32x32 blocks.
  constexpr int AM = DTL ? 2 * FM : 1, AN = DTL ? FN16 : 1;
  constexpr int CM = DTL ? 1 : FM, CN = DTL ? 1 : FN;
  f32x4_t acc16[AM][AN];
  f32x16_t acc[CM][CN];
#pragma unroll
  for (int i = 0; i < AM; ++i)
#pragma unroll
    for (int j = 0; j < AN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc16[i][j][r] = 0.f;
#pragma unroll
  for (int i = 0; i < CM; ++i)
#pragma unroll
    for (int j = 0; j < CN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // K tiles [kb, kb + KT) of this block
  const int KT_all = (K + BK - 1) / BK;
  const int kb = piece * KT_all / np;
  const int KT = (piece + 1) * KT_all / np - kb;

  // register path: fragments of k-step ks (16 wide) of stage st: lane row
  // (lane & 31), chunk 2 ks + lane / 32
  bf16x8_t fa[2][FM], fb[2][FN];
  auto fload = [&](int st, int ks, int buf) {
    const int ch = ks * 2 + (lane >> 5);
    const uint4* S = lds + st * STAGE;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row = wm * WTM + i * 32 + (lane & 31);
      fa[buf][i] = __builtin_bit_cast(bf16x8_t, S[lds_slot<CPR>(row, ch)]);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int row = wn * WTN + j * 32 + (lane & 31);
      fb[buf][j] = __builtin_bit_cast(bf16x8_t, S[lds_slot<CPR>(BM + row, ch)]);
    }
  };
  auto compute = [&](int st) {
    fload(st, 0, 0);
    static_for<BK / 16>([&](auto kk) {
      constexpr int ks = decltype(kk)::value;
      constexpr int cur = ks & 1;
      if constexpr (ks + 1 < BK / 16) fload(st, ks + 1, cur ^ 1);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
    });
    // Instruction order for the scheduler: the first k-step's fragment reads,
    // then each k-step's MFMAs alternating with the next k-step's reads, so
    // LDS latency hides under the matrix cores inside every wave.
    constexpr int NR = FM + FN, NM = FM * FN, NP = NR < NM ? NR : NM;
    __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);  // DS read
    static_for<BK / 16 - 1>([&](auto) {
      static_for<NP>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      });
      if constexpr (NM > NP) __builtin_amdgcn_sched_group_barrier(0x008, NM - NP, 0);
      if constexpr (NR > NP) __builtin_amdgcn_sched_group_barrier(0x100, NR - NP, 0);
    });
    __builtin_amdgcn_sched_group_barrier(0x008, NM, 0);
  };

  if (DTL) {  // a compile-time constant: the other path is dropped
    // ---- direct-to-LDS ring.  LDS holds [A stage 0 | A stage 1 | B stage 0 |
    // B stage 1], rows of BK bf16 (CPR 16-byte chunks, XOR-swizzled).  Wave
    // instruction q of a tile moves 64 lanes x 16 bytes = RPI tile rows; lane l
    // fills slot l % CPR of row l / CPR and so fetches the logical chunk that
    // the swizzle puts in that slot.  Loads are range-checked buffer loads
    // over the whole operand: rows past M / N read as zeros (their products
    // only reach discarded outputs).
    //
    // Every address is fixed before the loop: a lane's global offset of each
    // load instruction (the k offset of a tile travels in the scalar offset),
    // the LDS destination of each instruction (scalar, wave-uniform) and the
    // lane's LDS fragment address for each k-step (the stage and fragment
    // index are immediate offsets), so the loop issues MFMAs, LDS reads and
    // buffer loads and no vector ALU work.
    //
    // MFMAs are v_mfma_f32_16x16x32_bf16: a 64-wide K tile is two 32-wide
    // k-steps, each split into two phases by fragment row, four phases of
    // FM x 2FN MFMAs.  Fragment registers hold one whole K tile.  Tile X is
    // read in the last phase of X-1 (k-step 0) and the first phase of X
    // (k-step 1); a barrier after X's first phase frees X's stage and the
    // loads of tile X+2 into it are spread over phases 1 and 2; a second
    // barrier, in the last phase ahead of its fragment reads, makes tile X+1
    // visible.  A load thus has about one K tile between its issue and the
    // barrier that needs it.
    static_assert(BK == 64 && STAGES == 2, "schedule for 64-wide K tiles, two stages");
    constexpr int RPI = 64 / CPR;                       // tile rows per instruction
    constexpr int AI = BM / RPI / NWAVES, BI = BN / RPI / NWAVES;
    static_assert(AI * RPI * NWAVES == BM && BI * RPI * NWAVES == BN, "tile config");
    constexpr int IPT = AI + BI;                        // load instructions per tile per wave
    constexpr int ROWB = CPR * 16;                      // bytes per LDS row
    constexpr int A_STAGE = BM * ROWB, B_STAGE = BN * ROWB;
    constexpr int B_REGION = STAGES * A_STAGE;
    constexpr int FM2 = 2 * FM, FN2 = FN16;             // 16-row / 16-column fragments per wave tile
    constexpr int NR2 = FM2 + FN2;                      // fragment reads per k-step
    constexpr int NMP = FM * FN2;                       // MFMAs per phase
    constexpr bool PINGPONG = BM == 256 && BN == 256;
    static_assert(B_REGION + STAGES * B_STAGE <= (int)sizeof(lds), "LDS");
    static_assert((STAGES - 1) * A_STAGE + (FM2 - 1) * 16 * ROWB < 65536 &&
                  (STAGES - 1) * B_STAGE + (FN2 - 1) * 16 * ROWB < 65536, "ds_read immediate offsets");
    const int wv = __builtin_amdgcn_readfirstlane(wave);  // wave index in a scalar register
    const __amdgpu_buffer_rsrc_t rsa = __builtin_amdgcn_make_buffer_rsrc((void*)A, (short)0, (int)((long)M * lda * 2),
                                                                         kBufferWord3);
    const __amdgpu_buffer_rsrc_t rsw = __builtin_amdgcn_make_buffer_rsrc((void*)W, (short)0, (int)((long)N * ldw * 2),
                                                                         kBufferWord3);
    // per-lane global byte offsets of the load instructions (k offset excluded)
    int goa[AI], gob[BI];
    {
      const int lr = lane / CPR, sl = lane % CPR;
#pragma unroll
      for (int q = 0; q < AI; ++q) {
        const int row = (wv * AI + q) * RPI + lr;
        const int kc = lds_slot<CPR>(row, sl) - row * CPR;  // the XOR is an involution
        goa[q] = ((m0 + row) * (int)lda + kc * 8) * 2;
      }
#pragma unroll
      for (int q = 0; q < BI; ++q) {
        const int row = (wv * BI + q) * RPI + lr;
        const int kc = lds_slot<CPR>(row, sl) - row * CPR;
        gob[q] = ((n0 + row) * (int)ldw + kc * 8) * 2;
      }
    }
    // per-lane LDS byte address of fragment 0 at k-step ks, stage 0: row
    // lane % 16, chunk 4 ks + lane / 16.  Rows of fragment i differ by 16 i,
    // which leaves the swizzle term unchanged.
    int fra[2], frb[2];
    {
      const int ra = wm * WTM + (lane & 15), rb = wn * WTN + (lane & 15);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        fra[ks] = lds_slot<CPR>(ra, 4 * ks + (lane >> 4)) * 16;
        frb[ks] = B_REGION + lds_slot<CPR>(rb, 4 * ks + (lane >> 4)) * 16;
      }
    }
    char* const lbase = (char*)lds;
    // load instructions [q0, q1) of tile kt (A's first, then B's) into stage st
    auto load_part = [&](int st, int kt, int q0, int q1) __attribute__((always_inline)) {
      const int koff = (kb + kt) * BK * 2;
#pragma unroll
      for (int q = 0; q < AI; ++q) {
        if (q < q0 || q >= q1) continue;
        // copied to a local first: the array element passed straight to the
        // builtin makes the host pass drop the kernel launch stub
        const int vo = goa[q];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsa, (__attribute__((address_space(3))) void*)(lbase + st * A_STAGE + (wv * AI + q) * RPI * ROWB), 16,
            vo, koff, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < BI; ++q) {
        if (AI + q < q0 || AI + q >= q1) continue;
        const int vo = gob[q];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsw,
            (__attribute__((address_space(3))) void*)(lbase + B_REGION + st * B_STAGE + (wv * BI + q) * RPI * ROWB),
            16, vo, koff, 0, 0);
      }
    };
    if constexpr (PINGPONG) {
      // The 256x256 tile.  Two wave groups (waves 0-3 and 4-7, one wave of each
      // per SIMD) take turns: while one issues a cluster of 16 MFMAs, the other
      // reads the fragments of its next cluster and issues its share of the
      // loads, so LDS reads, loads and MFMAs run beside each other all the time
      // instead of every wave reading at once; block barriers hold the groups
      // one turn apart.  A K tile is Q clusters.  Cluster c multiplies the
      // wave's c-th quarter of A rows (2 fragments) with all its B columns;
      // A and B tiles lie in LDS as Q parts, part c holding every wave's c-th
      // quarter side by side.  Read phase k = Q kt + c takes part c of A of
      // tile kt and part c of B of tile kt + 1 (B fragments are held for a
      // whole tile, two tiles in turn), 6 reads in every phase.  A part is
      // read in one phase, and the loads of the part two tiles on leave into
      // its place in the next phase: the other group read it one turn earlier,
      // ahead of the barrier in between.  A load has 2Q - 2 read phases (1.5 K
      // tiles) until the wait before the barrier that makes it visible.
      // Every output is summed in the same order as in the other schedules.
      // Rate at 16384 x 3072 x 15360 (plain store): 1.44 - 1.50 PFLOP/s against
      // 1.35 - 1.42 with the schedule below, matrix cores busy 0.89 of the
      // cycles against 0.77 at a clock that power holds at 1.63 against 1.77
      // GHz; 4608 x 9216 x 3072: 1.29 against 1.23.  Tiles of fewer MFMAs per
      // phase (256x128, 128x256) gain 4 - 10% on repeated launches but lose
      // 0.3 - 1.5% inside a step, where operands and code arrive cold, and keep
      // the schedule below; raised priority for the MFMA turn and a barrier two
      // or four MFMAs ahead of its end measured 1% and 13 - 15% slower.
      constexpr int Q = 4;
      constexpr int AF = FM2 / Q, BF = FN2, BQ = FN2 / Q;  // A fragments of a cluster; B fragments in all, and per phase
      constexpr int ASUB = A_STAGE / Q, BSUB = B_STAGE / Q;  // bytes of a part
      constexpr int LA = AI / Q, LB = BI / Q;                // load instructions of a part per wave
      static_assert(NWAVES == 8 && AF * Q == FM2 && BQ * Q == FN2 && LA * Q == AI && LB * Q == BI, "ping-pong tile");
      const int lds0 = (int)(unsigned)(size_t)(__attribute__((address_space(3))) char*)lbase;
      // per-lane LDS addresses of fragment 0 of part 0, stage 0, for the two k-steps
      int ar[2], br[2];
      {
        const int ra = wm * (WTM / Q) + (lane & 15), rb = wn * (WTN / Q) + (lane & 15);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          ar[ks] = lds0 + lds_slot<CPR>(ra, 4 * ks + (lane >> 4)) * 16;
          br[ks] = lds0 + B_REGION + lds_slot<CPR>(rb, 4 * ks + (lane >> 4)) * 16;
        }
      }
      // per-lane global byte offsets of this wave's load instructions of each part
      int pa[Q][LA], pb[Q][LB];
#pragma unroll
      for (int c = 0; c < Q; ++c) {
        const int sl = lane % CPR;
#pragma unroll
        for (int q = 0; q < LA; ++q) {
          const int row = (wv * LA + q) * RPI + lane / CPR;
          const int kc = lds_slot<CPR>(row, sl) - row * CPR;
          pa[c][q] = ((m0 + row / (WTM / Q) * WTM + c * (WTM / Q) + row % (WTM / Q)) * (int)lda + kc * 8) * 2;
        }
#pragma unroll
        for (int q = 0; q < LB; ++q) {
          const int row = (wv * LB + q) * RPI + lane / CPR;
          const int kc = lds_slot<CPR>(row, sl) - row * CPR;
          pb[c][q] = ((n0 + row / (WTN / Q) * WTN + c * (WTN / Q) + row % (WTN / Q)) * (int)ldw + kc * 8) * 2;
        }
      }
      // part c of K tile kt into stage st
      auto load_a = [&](auto stc, auto cc, int kt) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, c = decltype(cc)::value;
        const int koff = (kb + min(kt, KT - 1)) * BK * 2;
#pragma unroll
        for (int q = 0; q < LA; ++q) {
          const int vo = pa[c][q];
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rsa,
              (__attribute__((address_space(3))) void*)(lbase + st * A_STAGE + c * ASUB + (wv * LA + q) * RPI * ROWB),
              16, vo, koff, 0, 0);
        }
      };
      auto load_b = [&](auto stc, auto cc, int kt) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, c = decltype(cc)::value;
        const int koff = (kb + min(kt, KT - 1)) * BK * 2;
#pragma unroll
        for (int q = 0; q < LB; ++q) {
          const int vo = pb[c][q];
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rsw,
              (__attribute__((address_space(3))) void*)(lbase + B_REGION + st * B_STAGE + c * BSUB +
                                                        (wv * LB + q) * RPI * ROWB),
              16, vo, koff, 0, 0);
        }
      };
      i32x4_t fa[2][AF], fb[2][2][BF];  // A fragments [k-step][row], B fragments [tile parity][k-step][column]
      auto read_a = [&](auto stc, auto cc) __attribute__((always_inline)) {
        constexpr int off = decltype(stc)::value * A_STAGE + decltype(cc)::value * ASUB;
        static_for<2 * AF>([&](auto ic) {
          constexpr int ks = decltype(ic)::value / AF, i = decltype(ic)::value % AF;
          asm_lds_read16<off + i * 16 * ROWB>(fa[ks][i], ar[ks]);
        });
      };
      auto read_b = [&](auto stc, auto cc) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, c = decltype(cc)::value, off = st * B_STAGE + c * BSUB;
        static_for<2 * BQ>([&](auto ic) {
          constexpr int ks = decltype(ic)::value / BQ, j = decltype(ic)::value % BQ;
          asm_lds_read16<off + j * 16 * ROWB>(fb[st][ks][c * BQ + j], br[ks]);
        });
      };
      // one read phase and the cluster it feeds
      auto phase = [&](auto stc, auto cc, int kt) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, c = decltype(cc)::value;
        using SN = std::integral_constant<int, st ^ 1>;
        using CP = std::integral_constant<int, (c + Q - 1) % Q>;
        using SA = std::integral_constant<int, c == 0 ? st ^ 1 : st>;
        using SB = std::integral_constant<int, c == 0 ? st : st ^ 1>;
        read_a(stc, cc);
        read_b(SN{}, cc);
        load_a(SA{}, CP{}, c == 0 ? kt + 1 : kt + 2);
        load_b(SB{}, CP{}, c == 0 ? kt + 2 : kt + 3);
        asm_lgkm_wait<0>();
        wait_vmcnt<(2 * Q - 2) * (LA + LB)>();
        asm volatile("s_barrier" ::: "memory");
        static_for<2 * AF * BF>([&](auto mc) {
          constexpr int m = decltype(mc)::value, ks = m / (AF * BF), i = m % (AF * BF) / BF, j = m % BF;
          asm_mfma16(acc16[c * AF + i][j], fa[ks][i], fb[st][ks][j]);
        });
        asm volatile("s_barrier" ::: "memory");
      };
#pragma unroll
      for (int i = 0; i < AM; ++i)
#pragma unroll
        for (int j = 0; j < AN; ++j) asm volatile("" : "+v"(acc16[i][j]));
      using S0 = std::integral_constant<int, 0>;
      using S1 = std::integral_constant<int, 1>;
      static_for<Q>([&](auto cc) { load_b(S0{}, cc, 0); });
      static_for<Q>([&](auto cc) {
        load_a(S0{}, cc, 0);
        load_b(S1{}, cc, 1);
      });
      wait_vmcnt<Q * (LA + LB)>();
      asm volatile("s_barrier" ::: "memory");
      static_for<Q>([&](auto cc) { read_b(S0{}, cc); });
      asm_lgkm_wait<0>();
      asm volatile("s_barrier" ::: "memory");
      static_for<Q - 1>([&](auto cc) {
        load_a(S1{}, cc, 1);
        load_b(S0{}, cc, 2);
      });
      wait_vmcnt<(2 * Q - 2) * (LA + LB)>();
      asm volatile("s_barrier" ::: "memory");
      if (wv >= 4) asm volatile("s_barrier" ::: "memory");
      int kt = 0;
      for (; kt + 1 < KT; kt += 2) {
        static_for<Q>([&](auto cc) { phase(S0{}, cc, kt); });
        static_for<Q>([&](auto cc) { phase(S1{}, cc, kt + 1); });
      }
      if (kt < KT) static_for<Q>([&](auto cc) { phase(S0{}, cc, kt); });
      if (wv < 4) asm volatile("s_barrier" ::: "memory");
      asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
      for (int i = 0; i < AM; ++i)
#pragma unroll
        for (int j = 0; j < AN; ++j) asm volatile("" : "+v"(acc16[i][j]));
    } else if constexpr (FM2 + FN2 <= FM * FN2) {
      // Every configuration whose phase holds at least one MFMA per fragment
      // read (all but the 128x64 skinny tile): the schedule below with every
      // MFMA, fragment read, LDS wait and barrier an asm statement, so the
      // instructions issue in exactly this order (0.5-2.5% faster than the
      // compiler's placement of the same schedule, bitwise the same results).
      // Phases of NMP MFMAs:
      //  P0  k-step 0, fragment rows 0 .. NA/2-1; one read of this tile's
      //      k-step-1 fragments after each of the first NR MFMAs
      //      -- lgkmcnt(0), barrier: no wave reads this stage any more
      //  P1  k-step 0, rows NA/2 ..; loads 0 .. Q1-1 of tile kt+2 spread over it
      //  P2  k-step 1, rows 0 .. NA/2-1; the other IPT - Q1 loads
      //  P3  k-step 1, rows NA/2 ..: NMP - NR MFMAs, then
      //      -- vmcnt(IPT), barrier: tile kt+1 visible
      //      the rest, each followed by one of the next tile's k-step-0 reads
      // LDS operations complete in order, so before each P0 MFMA the wait
      // allows every read issued after the P3 read that MFMA needs.
      constexpr int NA = FM2, NB = FN2, NR = NA + NB, NMP = (NA / 2) * NB;
      static_assert(NR <= NMP, "schedule");
      const int lds0 = (int)(unsigned)(size_t)(__attribute__((address_space(3))) char*)lbase;
      const int a0 = lds0 + fra[0], a1 = lds0 + fra[1], b0 = lds0 + frb[0], b1 = lds0 + frb[1];
      i32x4_t fa0[NA], fb0[NB], fa1[NA], fb1[NB];
      // k-step-0 fragment reads in the order A0, B0 .. B(NB-1), A1 .. A(NA-1)
      // (the order the first P0 MFMAs need them); k-step 1: A's, then B's
      auto rd0 = [&](auto stc, auto rc) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, r = decltype(rc)::value;
        if constexpr (r == 0) asm_lds_read16<st * A_STAGE>(fa0[0], a0);
        else if constexpr (r <= NB) asm_lds_read16<st * B_STAGE + (r - 1) * 16 * ROWB>(fb0[r - 1], b0);
        else asm_lds_read16<st * A_STAGE + (r - NB) * 16 * ROWB>(fa0[r - NB], a0);
      };
      auto rd1 = [&](auto stc, auto rc) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, r = decltype(rc)::value;
        if constexpr (r < NA) asm_lds_read16<st * A_STAGE + r * 16 * ROWB>(fa1[r], a1);
        else asm_lds_read16<st * B_STAGE + (r - NA) * 16 * ROWB>(fb1[r - NA], b1);
      };
      // loads [Q1) of a tile in P1 and [Q1, IPT) in P2, spread evenly over each phase's MFMAs
      constexpr int Q1 = (IPT + 1) / 2, Q2 = IPT - Q1;
      auto tile8 = [&](auto stc, int kt) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value;
        using SN = std::integral_constant<int, st ^ 1>;
        const int kt2 = min(kt + 2, KT - 1);
        static_for<NMP>([&](auto mc) {  // P0: k-step 0, rows 0 .. NA/2-1; this tile's k-step-1 reads
          constexpr int m = decltype(mc)::value, i = m / NB, j = m % NB;
          constexpr int ia = i == 0 ? 0 : NB + i, ib = 1 + j;
          constexpr int need = ia > ib ? ia : ib;
          asm_lgkm_wait<(NR - 1 - need) + (m < NR ? m : NR)>();
          asm_mfma16(acc16[i][j], fa0[i], fb0[j]);
          if constexpr (m < NR) rd1(stc, std::integral_constant<int, m>{});
        });
        asm_lgkm_wait<0>();
        asm volatile("s_barrier" ::: "memory");
        static_for<NMP>([&](auto mc) {  // P1: k-step 0, rows NA/2 ..; first half of the loads of tile kt+2
          constexpr int m = decltype(mc)::value, i = NA / 2 + m / NB, j = m % NB;
          asm_mfma16(acc16[i][j], fa0[i], fb0[j]);
          constexpr int q0 = m * Q1 / NMP, q1 = (m + 1) * Q1 / NMP;
          if constexpr (q1 > q0) load_part(st, kt2, q0, q1);
        });
        static_for<NMP>([&](auto mc) {  // P2: k-step 1, rows 0 .. NA/2-1; second half of the loads
          constexpr int m = decltype(mc)::value, i = m / NB, j = m % NB;
          asm_mfma16(acc16[i][j], fa1[i], fb1[j]);
          constexpr int q0 = m * Q2 / NMP, q1 = (m + 1) * Q2 / NMP;
          if constexpr (q1 > q0) load_part(st, kt2, Q1 + q0, Q1 + q1);
        });
        static_for<NMP>([&](auto mc) {  // P3: k-step 1, rows NA/2 ..; the next tile's k-step-0 reads
          constexpr int m = decltype(mc)::value, i = NA / 2 + m / NB, j = m % NB;
          if constexpr (m == NMP - NR) {  // the MFMAs before it need no LDS
            wait_vmcnt<IPT>();
            asm volatile("s_barrier" ::: "memory");
          }
          asm_mfma16(acc16[i][j], fa1[i], fb1[j]);
          if constexpr (m >= NMP - NR) rd0(SN{}, std::integral_constant<int, m - (NMP - NR)>{});
        });
      };
      // The zeroed accumulators pass through an empty asm statement here, so
      // their initialisation is issued before the prologue and not next to
      // the first asm MFMA (a VALU write just before an MFMA that reads it
      // needs wait states the compiler does not know to insert).
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc16[i][j]));
      load_part(0, 0, 0, IPT);
      load_part(1, min(1, KT - 1), 0, IPT);
      wait_vmcnt<IPT>();
      asm volatile("s_barrier" ::: "memory");
      static_for<NR>([&](auto rc) { rd0(std::integral_constant<int, 0>{}, rc); });
      int kt = 0;
      for (; kt + 1 < KT; kt += 2) {
        tile8(std::integral_constant<int, 0>{}, kt);
        tile8(std::integral_constant<int, 1>{}, kt + 1);
      }
      if (kt < KT) tile8(std::integral_constant<int, 0>{}, kt);
      asm_lgkm_wait<0>();
      // wait states between the last asm MFMAs and the accumulators' next
      // reader; each accumulator then passes through an empty asm statement,
      // which keeps every read of it after the wait states
      asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc16[i][j]));
    } else {
    bf16x8_t ha[2][FM2], hb[2][FN2];
      auto rd = [&](auto stc, auto ksc) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value, ks = decltype(ksc)::value;
  #pragma unroll
        for (int i = 0; i < FM2; ++i)
          ha[ks][i] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(lbase + fra[ks] + st * A_STAGE + i * 16 * ROWB));
  #pragma unroll
        for (int j = 0; j < FN2; ++j)
          hb[ks][j] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(lbase + frb[ks] + st * B_STAGE + j * 16 * ROWB));
      };
      // phase h of k-step ks: fragment rows h FM .. (h + 1) FM - 1
      auto mm = [&](auto ksc, auto hc) __attribute__((always_inline)) {
        constexpr int ks = decltype(ksc)::value, h = decltype(hc)::value;
  #pragma unroll
        for (int i = h * FM; i < (h + 1) * FM; ++i)
  #pragma unroll
          for (int j = 0; j < FN2; ++j)
            acc16[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ha[ks][i], hb[ks][j], acc16[i][j], 0, 0, 0);
      };
      // instruction order of a phase: each MFMA followed by its share of R LDS
      // reads and V buffer loads
      auto weave = [&](auto rc, auto vc) __attribute__((always_inline)) {
        constexpr int R = decltype(rc)::value, V = decltype(vc)::value;
        static_for<NMP>([&](auto mc) {
          constexpr int m = decltype(mc)::value;
          constexpr int r = (m + 1) * R / NMP - m * R / NMP, v = (m + 1) * V / NMP - m * V / NMP;
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                           // MFMA
          if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);      // DS read
          if constexpr (v > 0) __builtin_amdgcn_sched_group_barrier(0x020, v, 0);      // VMEM read
        });
      };
      constexpr int QH = IPT / 2;
      using J0 = std::integral_constant<int, 0>;
      using J1 = std::integral_constant<int, 1>;
      auto tile = [&](auto stc, int kt) __attribute__((always_inline)) {
        constexpr int st = decltype(stc)::value;
        using SN = std::integral_constant<int, st ^ 1>;
        // phase 0: this tile's k-step 1 fragments
        rd(stc, J1{});
        mm(J0{}, J0{});
        weave(std::integral_constant<int, NR2>{}, J0{});
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): own reads of this stage done
        asm volatile("s_barrier" ::: "memory");
        // phases 1, 2: the loads of tile kt + 2 into this stage
        load_part(st, min(kt + 2, KT - 1), 0, QH);
        mm(J0{}, J1{});
        weave(J0{}, std::integral_constant<int, QH>{});
        __builtin_amdgcn_sched_barrier(0);
        load_part(st, min(kt + 2, KT - 1), QH, IPT);
        mm(J1{}, J0{});
        weave(J0{}, std::integral_constant<int, IPT - QH>{});
        __builtin_amdgcn_sched_barrier(0);
        // tile kt + 1 landed (only the loads of kt + 2 may still be in flight)
        wait_vmcnt<IPT>();
        asm volatile("s_barrier" ::: "memory");
        // phase 3: the next tile's k-step 0 fragments
        rd(SN{}, J0{});
        mm(J1{}, J1{});
        weave(std::integral_constant<int, NR2>{}, J0{});
        __builtin_amdgcn_sched_barrier(0);
      };
      // Loads past the last K tile fetch it again into a stage nobody reads any
      // more (no branches, constant wait counts).  The barriers are bare
      // s_barriers: a __syncthreads() fence would also drain the loads still in
      // flight for later tiles.
      load_part(0, 0, 0, IPT);
      load_part(1, min(1, KT - 1), 0, IPT);
      wait_vmcnt<IPT>();
      asm volatile("s_barrier" ::: "memory");
      rd(J0{}, J0{});
      int kt = 0;
      for (; kt + 1 < KT; kt += 2) {
        tile(J0{}, kt);
        tile(J1{}, kt + 1);
      }
      if (kt < KT) tile(J0{}, kt);
    }
    // the refetches of the last tile must land before the epilogue reuses LDS
    wait_vmcnt<0>();
    __syncthreads();

    if (np > 1) {
      // Split K: publish this piece's partial sums, or -- for the last piece
      // of the tile to arrive -- add every piece's in piece order (the same
      // order whichever piece arrives last) and go on to the epilogue.  A
      // piece that finds all the others already counted skips publishing.
      // The sums move by agent-scope accesses (sc1): stores write through the
      // XCD's L2 and loads do not take lines it holds, so no block writes a
      // whole L2 back or invalidates it under the blocks still multiplying
      // there.  Every wave waits for its own stores before the block barrier,
      // and thread 0 counts after it.  With a release fence per publishing and
      // an acquire fence per merging block, and one load in flight at a time,
      // the split cost 22 us of 100 on 768 x 3072 x 15360 (3 pieces) and 38 of
      // 150 on 1536 x 3072 x 12288; now about half.
      constexpr int NV = AM * AN, NB = NV % 8 == 0 ? 8 : NV % 6 == 0 ? 6 : 1;
      int* const flag = (int*)&lds[STAGES * STAGE - 1];  // past the epilogue's LDS (asserted below)
      int* const cnt = P.sk_cnt + tile_id;
      auto slot = [&](int q) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((char*)P.sk_part + ((long)tile_id * np + q) * (NV * NT * 16), (short)0,
                                                 NV * NT * 16, kBufferWord3);
      };
      if (tid == 0) *flag = __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == np - 1;
      __syncthreads();
      if (!*flag) {
        const __amdgpu_buffer_rsrc_t mine = slot(piece);
#pragma unroll
        for (int i = 0; i < AM; ++i)
#pragma unroll
          for (int j = 0; j < AN; ++j)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc16[i][j]), mine, tid * 16,
                                                   (i * AN + j) * NT * 16, kAgentScope);
        wait_vmcnt<0>();
        __syncthreads();
        if (tid == 0) *flag = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == np - 1;
        __syncthreads();
        if (!*flag) return;  // uniform across the block
      }
      // NB accumulators at a time, a piece's loads for all of them in flight together
      static_for<NV / NB>([&](auto bc) {
        constexpr int b0 = decltype(bc)::value * NB;
        f32x4_t t[NB] = {};
        for (int q = 0; q < np; ++q) {
          if (q == piece) {
            static_for<NB>([&](auto ec) {
              constexpr int e = decltype(ec)::value, v = b0 + e;
              t[e] += acc16[v / AN][v % AN];
            });
          } else {
            const __amdgpu_buffer_rsrc_t r = slot(q);
            u32x4_t w[NB];
#pragma unroll
            for (int e = 0; e < NB; ++e)
              w[e] = __builtin_amdgcn_raw_buffer_load_b128(r, tid * 16, (b0 + e) * NT * 16, kAgentScope);
#pragma unroll
            for (int e = 0; e < NB; ++e) t[e] += __builtin_bit_cast(f32x4_t, w[e]);
          }
        }
        static_for<NB>([&](auto ec) {
          constexpr int e = decltype(ec)::value, v = b0 + e;
          acc16[v / AN][v % AN] = t[e];
        });
      });
      if (tid == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else {
    // ---- register path with zero-filled K tail (two LDS buffers).
    constexpr int A_CH = BM * CPR / NT, B_CH = BN * CPR / NT;
    static_assert((BM * CPR) % NT == 0 && (BN * CPR) % NT == 0 && A_CH >= 1 && B_CH >= 1, "tile config");
    uint4 ra[A_CH], rb[B_CH];
    auto gload = [&](int kt) {
      const int k0 = kt * BK;
#pragma unroll
      for (int c = 0; c < A_CH; ++c) {
        const int idx = tid + c * NT;
        const int row = idx / CPR, kc = idx % CPR;
        const int gr = m0 + row, gk = k0 + kc * 8;
        const bool ok = gr < M && gk < K;
        const uint4 v = *(const uint4*)(A + (long)min(gr, M - 1) * lda + min(gk, K - 8));
        ra[c] = ok ? v : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int c = 0; c < B_CH; ++c) {
        const int idx = tid + c * NT;
        const int row = idx / CPR, kc = idx % CPR;
        const int gr = n0 + row, gk = k0 + kc * 8;
        const bool ok = gr < N && gk < K;
        const uint4 v = *(const uint4*)(W + (long)min(gr, N - 1) * ldw + min(gk, K - 8));
        rb[c] = ok ? v : make_uint4(0, 0, 0, 0);
      }
    };
    auto lstore = [&](int st) {
      uint4* S = lds + st * STAGE;
#pragma unroll
      for (int c = 0; c < A_CH; ++c) {
        const int idx = tid + c * NT;
        S[lds_slot<CPR>(idx / CPR, idx % CPR)] = ra[c];
      }
#pragma unroll
      for (int c = 0; c < B_CH; ++c) {
        const int idx = tid + c * NT;
        S[lds_slot<CPR>(BM + idx / CPR, idx % CPR)] = rb[c];
      }
    };
    gload(0);
    lstore(0);
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
      if (kt + 1 < KT) gload(kt + 1);
      compute(kt & 1);
      if (kt + 1 < KT) lstore((kt + 1) & 1);
      __syncthreads();
    }
  }

  // epilogue.  Row facts (request, padded position, grid position) are computed
  // once per tile row into LDS, so the loop never indexes the batch metadata.
  // The wave tile leaves in groups of 32 rows, each staged through a per-wave
  // LDS buffer.
  RowEntry* rows = (RowEntry*)&lds[0];
  constexpr int SP = WTN + 4;  // staging row pitch in floats (16-byte aligned rows)
  float* stg = (float*)&lds[0] + BM * (sizeof(RowEntry) / 4) + wave * 32 * SP;
  static_assert(WTN <= 64 && BM * sizeof(RowEntry) + NWAVES * 32 * SP * 4 <= sizeof(lds) - 16,
                "epilogue LDS (the last 16 bytes hold the split flag)");
  const EpiArgs E = gi ? P.g[1].epi : P.g[0].epi;
  if (E.mode == EPI_RESID || E.mode == EPI_QKV) {
    for (int t = tid; t < BM; t += NT)
      if (m0 + t < M) rows[t] = make_row_entry(P.meta, E.row_base + m0 + t);
    __syncthreads();
  }
  const bf16_t* bias = (const bf16_t*)E.bias;
  // The bias of every column this lane stages, loaded before the first output
  // store: loads and stores share one in-order counter, so a bias load issued
  // after a group's stores would wait for them.
  constexpr int NBC = DTL ? FN16 : FN;
  float bcol[NBC];
#pragma unroll
  for (int q = 0; q < NBC; ++q) {
    const int n = n0 + wn * WTN + (DTL ? q * 16 + (lane & 15) : q * 32 + (lane & 31));
    bcol[q] = (bias != nullptr && n < N) ? bf2f(bias[n]) : 0.f;
  }
  // The group loop is rolled for wave tiles of more than two groups: only the
  // staging writes, which name accumulator registers, have a copy per group.
  // Unrolled over its groups, modes and tails the epilogue was 240 KB of code for
  // the 256x256 tile, run once per tile from an instruction cache (64 KB for two
  // CUs) that the launches of a step, each another kernel, leave cold.  Rolled
  // (the kernel is 21 KB), and with whole rows of the wave tile stored per wave
  // access, one single block at 256 px takes 229 us instead of 239, one double
  // block at 512 px 504 instead of 520, the 57-block 1024 px step 62.4 ms instead
  // of 63.4.
  // kFast: wave tiles of one or two groups are unrolled (31 KB for 128x128).  In
  // the rolled form their launches of one round or less lost 1 - 2 us to its
  // second turn and to the branches and addresses of every mode (512 x 3072 x 64
  // to bf16 8.7 us between events before, 10.5 rolled, 8.9 now; 1024 cubed 13.3,
  // 15.1, 13.4), and its 218 VGPRs left the 128x128 register path one block per
  // CU (7907 x 2304 x 696: 53, 79, 53 us).  The register path unrolls every tile:
  // no block of a served model takes it (16384 x 1536 x 200: 33.8, 38.2, 33.5).
  // On the 256x256 tile kFast's forms are slower inside a step (one single block
  // at 1024 px by 0.5 - 3%), whichever of them is left out.
  constexpr bool kFast = FM <= 2 || !DTL;
  const int ew = kFast ? __builtin_amdgcn_readfirstlane(wave) : wave;
#pragma unroll (kFast ? FM : 1)
  for (int g = 0; g < FM; ++g) {
    static_for<FM>([&](auto gc) {
      constexpr int i = decltype(gc)::value;
      if (g == i) {
        if constexpr (DTL) {
          static_for<FN16>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            static_for<2>([&](auto aa) {
              constexpr int a = decltype(aa)::value;
              static_for<4>([&](auto rr) {
                constexpr int r = decltype(rr)::value;
                stg[(a * 16 + 4 * (lane >> 4) + r) * SP + j * 16 + (lane & 15)] = acc16[2 * i + a][j][r] + bcol[j];
              });
            });
          });
        } else {
          static_for<FN>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            static_for<16>([&](auto rr) {
              constexpr int r = decltype(rr)::value;
              stg[((r / 4) * 8 + (lane >> 5) * 4 + (r % 4)) * SP + j * 32 + (lane & 31)] = acc[i][j][r] + bcol[j];
            });
          });
        }
      }
    });
    const int ml = ew / NWN * WTM + g * 32;
    epilogue_group<WTN, kFast>(E, rows + ml, stg, m0 + ml, n0 + ew % NWN * WTN, M, N, lane);
  }
}

// direct-to-LDS path: whole K tiles, 16-byte aligned rows, and operands
// small enough for the 32-bit offsets of buffer loads
template <int BM, int BN, int BK>
bool dtl_ok(const GemmProblem& p) {
  for (int g = 0; g < p.n_groups; ++g) {
    const GemmGroup& G = p.g[g];
    const bool ok = G.K % BK == 0 && G.lda % 8 == 0 && G.ldw % 8 == 0 && (long)(G.M + BM) * G.lda * 2 < (1L << 31) &&
                    (long)(p.N + BN) * G.ldw * 2 < (1L << 31);
    if (!ok) return false;
  }
  return true;
}

template <int BM, int BN>
long tile_count(const GemmProblem& p) {
  const int tiles_n = (p.N + BN - 1) / BN;
  long tiles = (long)((p.g[0].M + BM - 1) / BM) * tiles_n;
  if (p.n_groups > 1) tiles += (long)((p.g[1].M + BM - 1) / BM) * tiles_n;
  return tiles;
}

template <int BM, int BN, int NWM, int NWN, int BK, int STAGES, bool DTL>
hipError_t launch_kernel(const GemmProblem& p, int sk, hipStream_t s) {
  const long tiles = tile_count<BM, BN>(p);
  if (tiles == 0) return hipSuccess;
  GemmProblem q = p;
  q.sk_p = DTL ? sk : 1;
  hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, NWM, NWN, BK, STAGES, DTL>), dim3((unsigned)(tiles * q.sk_p)),
                     dim3(NWM * NWN * 64), 0, s, q);
  return hipGetLastError();
}

template <int BM, int BN, int NWM, int NWN, int BK, int STAGES>
hipError_t launch_cfg(const GemmProblem& p, int sk, hipStream_t s) {
  if (dtl_ok<BM, BN, BK>(p)) return launch_kernel<BM, BN, NWM, NWN, BK, STAGES, true>(p, sk, s);
  return launch_kernel<BM, BN, NWM, NWN, BK, STAGES, false>(p, 1, s);
}

// direct-to-LDS-only configurations (wave tiles of an odd number of 16-column
// fragments have no register path): the 256x256 register path otherwise
template <int BM, int BN, int NWM, int NWN, int BK, int STAGES>
hipError_t launch_cfg_dtl_only(const GemmProblem& p, int sk, hipStream_t s) {
  if (dtl_ok<BM, BN, BK>(p)) return launch_kernel<BM, BN, NWM, NWN, BK, STAGES, true>(p, sk, s);
  return launch_cfg<256, 256, 2, 4, 64, 2>(p, 1, s);
}

enum GemmCfg { CFG_128x64 = 0, CFG_256x256 = 1, CFG_128x128 = 2, CFG_256x128 = 3, CFG_128x256 = 4, CFG_288x192 = 5 };

// Launch-time model of the tile configurations, fitted to dit_linear timings
// on MI355X over the step's GEMM shapes (M 768 .. 16896, N 1536 .. 21504,
// K 1536 .. 15360): one CU works through ceil(tiles / 256) tiles one after
// another, a tile costing its FLOPs at a per-CU rate plus a fixed prologue /
// epilogue time.  Large tiles have the higher rate (fewer operand bytes per
// FLOP); small tiles fill the 256 CUs when the big ones would leave most idle.
struct TileModel {
  GemmCfg cfg;
  int bm, bn;
  double tflops_per_cu;
  double fixed_us;
};
// 256x128's rate is raised from its fitted 6.11 to 128x256's 6.23: inside the
// step the two tie on FLOPs per tile and 256x128 measured faster wherever the
// two competed (M 768 .. 6144, the 256 / 512 px and SD3-shaped steps 0.7 - 2.4%
// faster, the rest unchanged).
// 256x256's rate is its fitted 7.31 raised by the 5% that its turn-taking
// schedule gained on one-round launches.  Launches of more than one round hold
// 256 busy CUs long enough for power to set the clock, and there the 256x128
// and 128x256 tiles, which move 1.5 times the operand bytes per FLOP, fall
// further behind than their one-round rates say (7622 x 3072 x 12288 inside a
// step: 540 us in 3 rounds of 256x128, 500 us in 2 of 256x256; 8056 x 3072 x
// 15360: 55 us more with the narrower tile): kSustainedLoss.
// With both, one single block at 1024 px 1064 -> 1051 us (linear2 on 256x256
// instead of 288x192), a packed 7622-row double block 1991 -> 1948 us, the
// 57-block 1024 px step 63.4 -> 63.0 ms, other sizes unchanged.
// 288x192 (12 waves of 96x48) divides 4608 x 3072 into exactly 256 tiles;
// its rate is set from the same large shapes on which 256x256 was measured
// (0.915 of 256x256's when both fill the GPU).  It is considered only for
// launches it covers in one round (see pick).
constexpr TileModel kTileModels[] = {
    {CFG_256x256, 256, 256, 7.7, 11.7},
    {CFG_256x128, 256, 128, 6.23, 8.4},
    {CFG_128x256, 128, 256, 6.23, 8.7},
    {CFG_128x128, 128, 128, 5.07, 4.1},
    {CFG_288x192, 288, 192, 6.31, 8.0},
};
constexpr double kSustainedLoss = 1.1;
// Split K: the merge adds, on the critical path, the write of a piece's
// partial sums and the last piece's read of the others' (fp32, bm x bn per
// piece) plus the arrival handshake.  A split is taken only when the model
// predicts it saves at least kSplitMinGain of the launch.
constexpr double kMergeFixedUs = 3.0;
constexpr double kMergeBytesPerUs = 40e3;
constexpr double kSplitMinGain = 0.05;
constexpr int kSplitMaxPieces = 8;

double model_us(const TileModel& t, const GemmProblem& p, int sk) {
  const long tn = (p.N + t.bn - 1) / t.bn;
  long tiles = 0;
  double work = 0.0;  // sum of piece times, microseconds
  for (int g = 0; g < p.n_groups; ++g) {
    const long tg = (long)((p.g[g].M + t.bm - 1) / t.bm) * tn;
    tiles += tg;
    work += tg * sk * (2.0 * t.bm * t.bn * p.g[g].K / sk / (t.tflops_per_cu * 1e6) + t.fixed_us);
  }
  if (tiles == 0) return 0.0;
  const long units = tiles * sk;
  double us = (double)((units + 255) / 256) * (work / units);
  if (units > 256 && (t.cfg == CFG_256x128 || t.cfg == CFG_128x256)) us *= kSustainedLoss;
  if (sk > 1) us += kMergeFixedUs + (sk - 1) * 4.0 * t.bm * t.bn / kMergeBytesPerUs;
  return us;
}

bool dtl_for(GemmCfg c, const GemmProblem& p) {
  switch (c) {
    case CFG_256x256: return dtl_ok<256, 256, 64>(p);
    case CFG_256x128: return dtl_ok<256, 128, 64>(p);
    case CFG_128x256: return dtl_ok<128, 256, 64>(p);
    case CFG_128x128: return dtl_ok<128, 128, 64>(p);
    case CFG_288x192: return dtl_ok<288, 192, 64>(p);
    default: return false;
  }
}

// K may be split when the caller gave split workspace, the direct-to-LDS path
// runs, both groups share K, every piece keeps at least 4 K tiles, and the
// counters and partial-sum slots suffice.
bool split_ok(const TileModel& t, const GemmProblem& p, int sk) {
  if (p.sk_part == nullptr || p.sk_cnt == nullptr || !dtl_for(t.cfg, p)) return false;
  if (p.n_groups > 1 && p.g[0].K != p.g[1].K) return false;
  if (p.g[0].K / 64 < 4 * sk) return false;
  const long tn = (p.N + t.bn - 1) / t.bn;
  long tiles = 0;
  for (int g = 0; g < p.n_groups; ++g) tiles += (long)((p.g[g].M + t.bm - 1) / t.bm) * tn;
  return tiles <= kSplitMaxTiles && tiles * sk * t.bm * t.bn * 4L <= kSplitPartBytes;
}

struct Choice {
  GemmCfg cfg;
  int sk;
};

// pick(): the configuration and K split with the shortest modelled launch
// (its time, in microseconds, in *us when asked for; 0 for the skinny-N path,
// which the model does not cover)
Choice pick(const GemmProblem& p, double* us_out = nullptr) {
  if (us_out) *us_out = 0.0;
  if (p.N <= 64) return {CFG_128x64, 1};
  Choice best{CFG_128x128, 1};
  double best_us = 1e300;
  for (const TileModel& t : kTileModels) {
    // 288x192 has no register path, and it measured faster inside the step
    // only where its tiles fit in one round
    if (t.cfg == CFG_288x192 && (!dtl_for(t.cfg, p) || tile_count<288, 192>(p) > 256)) continue;
    const double us = model_us(t, p, 1);
    if (us < best_us) {
      best_us = us;
      best = {t.cfg, 1};
    }
  }
  Choice split = best;
  double split_us = best_us;
  for (const TileModel& t : kTileModels)
    for (int sk = 2; sk <= kSplitMaxPieces; ++sk) {
      if (t.cfg == CFG_288x192 || !split_ok(t, p, sk)) continue;  // 288x192: one-round launches only
      const double us = model_us(t, p, sk);
      if (us < split_us) {
        split_us = us;
        split = {t.cfg, sk};
      }
    }
  const bool take_split = split_us <= (1.0 - kSplitMinGain) * best_us;
  if (us_out) *us_out = take_split ? split_us : best_us;
  return take_split ? split : best;
}

// Two groups as two launches: the image group of a double block often fills
// whole rounds of 256x256 tiles by itself (4096 rows x 12288 at 1024 px,
// 16384 x 3072 at 2048 px), and the text group's few tiles then open a last
// round that is mostly idle.  Run alone, the text group takes a tiling of its
// own (smaller tiles, split K) and finishes in a fraction of a round.  The
// second launch costs one kernel boundary.
constexpr double kLaunchGapUs = 4.0;
constexpr double kGroupSplitMinGain = 0.03;

}  // namespace

bool gemm_bf16_split_groups(const GemmProblem& p) {
  if (p.n_groups < 2 || p.N <= 64) return false;
  double both = 0.0, first = 0.0, second = 0.0;
  pick(p, &both);
  GemmProblem q = p;
  q.n_groups = 1;
  pick(q, &first);
  q.g[0] = p.g[1];
  pick(q, &second);
  return first + second + kLaunchGapUs <= (1.0 - kGroupSplitMinGain) * both;
}

const char* gemm_bf16_config_name(const GemmProblem& p) {
  // "gemm_bf16_<tile>" and, for a split of K into k pieces, "..._k<k>"
  struct Names {
    std::string n[6][kSplitMaxPieces + 1];
    Names() {
      const char* base[] = {"gemm_bf16_128x64", "gemm_bf16_256x256", "gemm_bf16_128x128", "gemm_bf16_256x128",
                            "gemm_bf16_128x256", "gemm_bf16_288x192"};
      for (int c = 0; c < 6; ++c)
        for (int k = 0; k <= kSplitMaxPieces; ++k) n[c][k] = k <= 1 ? base[c] : base[c] + std::string("_k") + std::to_string(k);
    }
  };
  static const Names names;
  const Choice c = pick(p);
  return names.n[c.cfg][c.sk].c_str();
}

hipError_t launch_gemm_bf16(const GemmProblem& p, hipStream_t s) {
  const Choice c = pick(p);
  switch (c.cfg) {
    case CFG_128x64:
      return launch_cfg<128, 64, 4, 1, 64, 2>(p, 1, s);
    case CFG_256x256:
      return launch_cfg<256, 256, 2, 4, 64, 2>(p, c.sk, s);
    case CFG_256x128:
      return launch_cfg<256, 128, 4, 2, 64, 2>(p, c.sk, s);
    case CFG_128x256:
      return launch_cfg<128, 256, 2, 4, 64, 2>(p, c.sk, s);
    case CFG_288x192:
      return launch_cfg_dtl_only<288, 192, 3, 4, 64, 2>(p, c.sk, s);
    default:
      return launch_cfg<128, 128, 2, 2, 64, 2>(p, c.sk, s);
  }
}

}  // namespace dit
