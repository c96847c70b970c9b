// fp32 GEMM on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 products
// and sums, no reduced precision), Y = A W^T + b with the same epilogues as the
// bf16 kernel.  Used by fp32 models.
//
// The fp32 models are small: their launches hold a few hundred rows and wait
// for memory, not for the matrix cores.  So operands go straight from memory to
// registers, 16 bytes per lane, with no LDS round trip or barrier before the
// end.  A lane's four consecutive K values feed four MFMAs (K is summed in the
// order 0 4 8 12, 1 5 9 13, ... inside a chunk, on both operands alike).  A
// block owns 32 x 32 outputs; its four waves split the K range, and the partial
// sums meet in LDS and are added in wave order.  That many small blocks also
// win where there is work for 64 x 64 tiles without a split (M 1100, N 1024,
// K 1024: 42 against 63 us; M 4096, N 3072, K 1024: 366 against 391 us).
// M 288, N 16 - 1536, K 16 - 1536 (the six launches of the small model's step
// at 256 px): 12.1 us per launch between events, launch included, against 43 us
// for 64 x 64 tiles on the vector ALUs.
//
// G is the number of 16-wide K chunks in each of a wave's two register buffers.
// With a block or more for each CU, waves hide each other's latency and G = 1
// wins (5 waves per SIMD, with G = 4 it is 3): M 288, N 1152, K 384 G = 1, 2, 4:
// 9.1, 9.9, 12.7 us.  Below that a wave has to hide it alone: M 288, N 384,
// K 1536 (108 blocks) 17.1, 16.0, 16.9 us; M 7, N 1024, K 4096 (32 blocks, 64
// chunks per wave) 33.3, 30.2, 28.9 us.
// G changes no order of sums, so a row's result does not depend on the batch.
#include "device_common.h"

namespace dit {

namespace {

constexpr int WT = 32;       // a wave's tile
constexpr int SP = WT + 4;   // LDS row pitch of a staged tile

// Four consecutive outputs n .. n+3 (n a multiple of 4) of row m, bias added.
__device__ __forceinline__ void store4(float* dst, int left, float4 y) {
  if (left >= 4 && ((uintptr_t)dst & 15) == 0) {
    *(float4*)dst = y;
    return;
  }
  dst[0] = y.x;
  if (left > 1) dst[1] = y.y;
  if (left > 2) dst[2] = y.z;
  if (left > 3) dst[3] = y.w;
}

__device__ __forceinline__ float4 gelu4(float4 y) {
  return make_float4(gelu_tanh(y.x), gelu_tanh(y.y), gelu_tanh(y.z), gelu_tanh(y.w));
}

__device__ __forceinline__ void epilogue4(const GemmProblem& P, const EpiArgs& E, int m, int n, float4 y) {
  const int left = P.N - n;
  switch (E.mode) {
    case EPI_STORE_F32:
    case EPI_STORE_T:
      store4((float*)E.out + (long)m * E.ldo + n, left, y);
      break;
    case EPI_GELU:
      store4((float*)E.out + (long)m * E.ldo + E.col0 + n, left, gelu4(y));
      break;
    case EPI_RESID: {  // N is the model width, a multiple of 64
      const RowInfo ri = row_info(P.meta, E.row_base + m);
      const float4 g = *(const float4*)(E.mods + (long)ri.req * E.mods_ld + E.gate_off + n);
      float4* xo = (float4*)((float*)E.out + (long)m * E.ldo + n);
      const float4 x = *xo;
      *xo = make_float4(x.x + g.x * y.x, x.y + g.y * y.y, x.z + g.z * y.z, x.w + g.w * y.w);
      break;
    }
    case EPI_QKV: {
      if (n >= E.n_qkv) {
        store4((float*)E.gelu_out + (long)m * E.gelu_ld + E.gelu_col0 + (n - E.n_qkv), left, gelu4(y));
        break;
      }
      const RowEntry re = make_row_entry(P.meta, E.row_base + m);
      const int H = E.hidden, d = E.head_dim, which = n / H, hn = n - which * H, h = hn / d, dd = hn - h * d;
      if (which == 2) {
        float* vt = (float*)E.vt + ((long)h * d + dd) * E.vt_ld + vt_slot(re.pos);
        vt[0] = y.x;
        vt[E.vt_ld] = y.y;
        vt[2 * E.vt_ld] = y.z;
        vt[3 * E.vt_ld] = y.w;
        break;
      }
      if (re.gi >= 0) {
        const int half = d >> 1, pos = dd < half ? re.gi : re.gj;
        const float4 t = *(const float4*)(E.rope + pos * (d >> 2) + ((dd < half ? dd : dd - half) >> 1));
        y = make_float4(y.x * t.x - y.y * t.y, y.x * t.y + y.y * t.x, y.z * t.z - y.w * t.w, y.z * t.w + y.w * t.z);
      }
      *(float4*)((float*)(which == 0 ? E.q : E.k) + ((long)h * E.T + re.pos) * d + dd) = y;
      break;
    }
  }
}

// ROWS: the grid has more than one row of blocks (see grid_of); the others skip its
// block numbering (0.2 us of a 9 us launch)
template <int G, bool ROWS>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmProblem P) {
  __shared__ float red[4][WT * SP];

  const int tiles_n = (P.N + WT - 1) / WT;
  const int tm0 = (P.g[0].M + WT - 1) / WT;
  int id = ROWS ? block_id() : blockIdx.x;
  if (ROWS && id >= (tm0 + (P.n_groups > 1 ? (P.g[1].M + WT - 1) / WT : 0)) * tiles_n) return;
  int gi = 0;
  if (id >= tm0 * tiles_n) {
    gi = 1;
    id -= tm0 * tiles_n;
  }
  const float* __restrict__ A = (const float*)(gi ? P.g[1].A : P.g[0].A);
  const float* __restrict__ W = (const float*)(gi ? P.g[1].W : P.g[0].W);
  const long lda = gi ? P.g[1].lda : P.g[0].lda;
  const long ldw = gi ? P.g[1].ldw : P.g[0].ldw;
  const int M = gi ? P.g[1].M : P.g[0].M;
  const int K = gi ? P.g[1].K : P.g[0].K;
  const int N = P.N;

  const int tid = threadIdx.x, lane = tid & 63;
  // with a scalar wave number the loop's guards are branches, otherwise lane
  // masks.  Branches win where a wave hides its own latency (M 7, N 1024,
  // K 4096: 28.2 against 28.9 us), masks with G = 1 (M 1100, N 1024, K 1024:
  // 41.9 against 43.9 us; M 8192, N 9216, K 1024: 2209 against 2418 us)
  const int wave = G == 1 ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = id / tiles_n * WT, n0 = id % tiles_n * WT;

  // lane: row lane % 16 of a 16-row fragment, K values 4 (lane / 16) .. + 3 of
  // a chunk.  Rows past the edge re-read the last one (their products reach
  // discarded outputs only); K values past the edge are zero on both sides.
  const int kq = (lane >> 4) * 4;
  const float* pa[2];
  const float* pb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    pa[i] = A + (long)min(m0 + i * 16 + (lane & 15), M - 1) * lda;
    pb[i] = W + (long)min(n0 + i * 16 + (lane & 15), N - 1) * ldw;
  }
  const int chunks = (K + 15) / 16;
  const int c0 = wave * chunks / 4, c1 = (wave + 1) * chunks / 4;
  f32x4_t acc[2][2] = {};
  float4 fa[2][G][2], fb[2][G][2];
  auto load = [&](auto bufc, int c) __attribute__((always_inline)) {
    constexpr int buf = decltype(bufc)::value;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int k = (c + g) * 16 + kq, ka = min(k, K - 4);
      const bool ok = k < K;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float4 a = *(const float4*)(pa[i] + ka), b = *(const float4*)(pb[i] + ka);
        fa[buf][g][i] = ok ? a : make_float4(0.f, 0.f, 0.f, 0.f);
        fb[buf][g][i] = ok ? b : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  };
  auto multiply = [&](auto bufc, int c) __attribute__((always_inline)) {
    constexpr int buf = decltype(bufc)::value;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (c + g >= c1) break;
      static_for<4>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        auto at = [](const float4& v) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; };
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(at(fa[buf][g][i]), at(fb[buf][g][j]), acc[i][j], 0, 0, 0);
      });
    }
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  load(B0{}, c0);
  for (int c = c0; c < c1; c += 2 * G) {
    if (c + G < c1) load(B1{}, c + G);
    multiply(B0{}, c);
    if (c + 2 * G < c1) load(B0{}, c + 2 * G);
    if (c + G < c1) multiply(B1{}, c + G);
  }

  // stage: column lane % 16 of a 16 x 16 block, rows 4 (lane / 16) .. + 3
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[wave][(i * 16 + (lane >> 4) * 4 + r) * SP + j * 16 + (lane & 15)] = acc[i][j][r];
  __syncthreads();

  const EpiArgs E = gi ? P.g[1].epi : P.g[0].epi;
  const float* bias = (const float*)E.bias;
  // a thread writes 4 columns, consecutive lanes along a row; for V columns along
  // the rows, which are consecutive in V^T
  const bool vcols = E.mode == EPI_QKV && n0 >= 2 * E.hidden && n0 < E.n_qkv;
  const int r = vcols ? tid & 31 : tid >> 3, c = vcols ? (tid >> 5) * 4 : (tid & 7) * 4;
  const int m = m0 + r, n = n0 + c;
  if (m >= M || n >= N) return;
  float4 y = *(const float4*)&red[0][r * SP + c];
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    const float4 t = *(const float4*)&red[w][r * SP + c];
    y.x += t.x;
    y.y += t.y;
    y.z += t.z;
    y.w += t.w;
  }
  if (bias) {
    y.x += bias[n];
    if (n + 1 < N) y.y += bias[n + 1];
    if (n + 2 < N) y.z += bias[n + 2];
    if (n + 3 < N) y.w += bias[n + 3];
  }
  epilogue4(P, E, m, n, y);
}

}  // namespace

hipError_t launch_gemm_f32(const GemmProblem& p, hipStream_t s) {
  long tiles = 0;
  int kmax = 0;
  for (int g = 0; g < p.n_groups; ++g) {
    tiles += (long)((p.g[g].M + WT - 1) / WT) * ((p.N + WT - 1) / WT);
    kmax = p.g[g].K > kmax ? p.g[g].K : kmax;
  }
  if (tiles == 0) return hipSuccess;
  const dim3 grid = grid_of(tiles), block(256);
  // K 2048: 32 chunks per wave.  Below a block per CU the two buffers of 2
  // chunks do for K up to there, longer K want the 8 chunks in flight
  if (grid.y > 1)
    hipLaunchKernelGGL((gemm_f32_kernel<1, true>), grid, block, 0, s, p);
  else if (tiles >= 256)
    hipLaunchKernelGGL((gemm_f32_kernel<1, false>), grid, block, 0, s, p);
  else if (kmax <= 2048)
    hipLaunchKernelGGL((gemm_f32_kernel<2, false>), grid, block, 0, s, p);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<4, false>), grid, block, 0, s, p);
  return hipGetLastError();
}

}  // namespace dit
