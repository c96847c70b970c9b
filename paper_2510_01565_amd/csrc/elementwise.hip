// HBM-bound kernels of the step: adaLN LayerNorm, the modulation GEMV over
// all blocks' adaLN weights (whose launch also carries the timestep embedding
// and a call's setup), the Euler update and the V relayout of the stand-alone
// attention call.
// Rows are processed one per wavefront with 16-byte accesses; all reductions
// are fixed butterfly trees (bitwise deterministic).
#include <math.h>

#include <algorithm>

#include "device_common.h"

namespace dit {

namespace {

// ---------------------------------------------------------------- timestep embedding
// e[r] = [cos(1000 t f_j) | sin(1000 t f_j)], f_j = 1e4^(-j/half), in fp64.
struct TimeArgs {
  float t[kMaxReq];
};
__device__ __forceinline__ float timestep_value(float t, int k, int dim) {
  const int half = dim / 2, j = k < half ? k : k - half;
  const double ang = 1000.0 * (double)t * exp(-log(10000.0) * (double)j / half);
  return (float)(k < half ? cos(ang) : sin(ang));
}
__global__ void timestep_kernel(float* e, int n_req, TimeArgs ta, int dim) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_req * dim) e[i] = timestep_value(ta.t[i / dim], i % dim, dim);
}

// ---------------------------------------------------------------- setup
// What a call prepares in its workspace ahead of the first GEMM, spread over
// `nblocks` blocks of 256 threads:
//  the RoPE table, table[pos][k] = (cos, sin)(pos * theta^(-2k / (d/2))), in fp64;
//  the split GEMMs' arrival counters, zeroed;
//  the V^T columns of every request's padding keys, zeroed.
__device__ __forceinline__ void setup_block(const SetupArgs& a, int block, int nblocks) {
  const int t0 = block * 256 + threadIdx.x, stride = nblocks * 256;
  const int quarter = a.head_dim / 4, axis = a.head_dim / 2;
  for (int i = t0; i < DIT_MAX_GRID * quarter; i += stride) {
    const int pos = i / quarter, k = i % quarter;
    const double ang = (double)pos * pow(a.theta, -2.0 * k / axis);
    a.rope[i] = make_float2((float)cos(ang), (float)sin(ang));
  }
  for (int i = t0; i < a.n_zero; i += stride) a.zero[i] = 0;
  const int rows = a.heads * a.head_dim;
  for (int r = 0; r < a.meta.n_req; ++r) {
    const int L = a.meta.joint_off[r + 1] - a.meta.joint_off[r];
    const int pad = a.meta.pad_off[r + 1] - a.meta.pad_off[r] - L;  // < 64
    for (int i = t0; i < rows * 64; i += stride) {
      const int k = i & 63;
      if (k >= pad) continue;
      const long at = (long)(i >> 6) * a.vt_ld + vt_slot(a.meta.pad_off[r] + L + k);
      if (a.es == 2) ((uint16_t*)a.vt)[at] = 0;
      else ((float*)a.vt)[at] = 0.f;
    }
  }
}

// ---------------------------------------------------------------- GEMV
// y[r, o] = sum_k W[o, k] act(x[r, k]) + b[o] for up to GV_R requests per
// pass; activations staged in LDS, weights streamed once with 16-byte loads.
// Each wavefront takes GemvShape::V output rows at a time and requests all of
// their chunks (a lane holds chunks lane, lane + 64, ... of each row) before
// any arithmetic, so V rows of loads are in flight per wave.  The weights are
// read once per step and never reused, so the loads are nontemporal (they do
// not displace cached data); on MI355X this streams the 6.5 GB of the FLUX
// modulation weights at about 6.8 TB/s against 5.5 TB/s for one row per wave
// with ordinary loads.
// FIRST: a call's first launch, whose first `sblocks` blocks run the call's
// setup (see setup_block, nothing in this launch reads it) and whose
// activations may be the timestep embedding.  Both are fp64 code that needs
// 80 VGPRs and 104 SGPRs by itself, so it stays out of the other launches.
constexpr int GV_R = 4;
constexpr int LN_MAX_H = 4096;  // widest hidden size (also the LayerNorm's limit)

template <typename WT>
struct GemvShape {
  static constexpr int EPC = 16 / sizeof(WT);        // elements per 16-byte chunk
  static constexpr int V = sizeof(WT) == 2 ? 4 : 2;  // rows per wave in flight
};

// MAXC: 16-byte chunks per lane and row the registers hold (K <= 64 EPC MAXC)
template <typename WT, int MAXC, bool FIRST>
__global__ __launch_bounds__(256) void gemv_kernel(const WT* __restrict__ W, const WT* __restrict__ b,
                                                   const float* __restrict__ x, long ldx, int n_req, int K,
                                                   int N, int act, float* __restrict__ y, long ldy, TimeArgs ta,
                                                   int sblocks, const SetupArgs su) {
  if constexpr (FIRST) {
    if ((int)blockIdx.x < sblocks) {
      setup_block(su, blockIdx.x, sblocks);
      return;
    }
  }
  const int block = FIRST ? blockIdx.x - sblocks : blockIdx.x;
  using S = GemvShape<WT>;
  constexpr int EPC = S::EPC, V = S::V;
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  extern __shared__ float xs[];  // [n_req][K]
  const int nr = min(n_req, GV_R);
  const int lane = threadIdx.x & 63;
  // The activations are staged after the chunk indices are formed (fewer VGPRs,
  // so more waves), except for the widest rows, whose two waves per SIMD gain
  // nothing from it and whose spilled scalars grow (K 4096, four requests: 2-4%).
  constexpr bool kStageFirst = MAXC >= 8;
  auto stage = [&]() __attribute__((always_inline)) {
    for (int i = threadIdx.x; i < nr * K; i += blockDim.x) {
      const int r = i / K, k = i % K;
      if constexpr (FIRST) {
        if (act == GEMV_TIMESTEP) {
          xs[i] = timestep_value(ta.t[r], k, K);
          continue;
        }
      }
      const float v = x[(long)r * ldx + k];
      xs[i] = act == GEMV_SILU ? silu(v) : v;
    }
    __syncthreads();
  };
  if constexpr (kStageFirst) stage();
  const int nwaves = (FIRST ? gridDim.x - sblocks : gridDim.x) * (blockDim.x >> 6);
  const int chunks = K / EPC;
  // Chunk i of a lane is chunk lane + 64 i of the row; lanes past the row's
  // last chunk load that chunk again (no branch around a load: a branch would
  // end the run of loads in flight) and weigh it by zero.
  int cidx[MAXC];
  float keep[MAXC];
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    cidx[i] = min(lane + 64 * i, chunks - 1);
    keep[i] = lane + 64 * i < chunks ? 1.f : 0.f;
  }
  if constexpr (!kStageFirst) stage();
  for (int o0 = (block * (blockDim.x >> 6) + (threadIdx.x >> 6)) * V; o0 < N; o0 += nwaves * V) {
    u32x4 u[V][MAXC];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const u32x4* wr = (const u32x4*)(W + (long)min(o0 + v, N - 1) * K);
#pragma unroll
      for (int i = 0; i < MAXC; ++i) u[v][i] = __builtin_nontemporal_load(wr + cidx[i]);
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      float acc[GV_R] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < MAXC; ++i) {
        float wv[EPC];
        if constexpr (sizeof(WT) == 2) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            wv[2 * e] = __uint_as_float(u[v][i][e] << 16) * keep[i];
            wv[2 * e + 1] = __uint_as_float(u[v][i][e] & 0xFFFF0000u) * keep[i];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) wv[e] = __uint_as_float(u[v][i][e]) * keep[i];
        }
#pragma unroll
        for (int r = 0; r < GV_R; ++r) {
          if (r < nr) {
            // 16-byte aligned: K and the chunk offset are multiples of 4 floats
            const float4* xr = (const float4*)(xs + r * K + cidx[i] * EPC);
#pragma unroll
            for (int q = 0; q < EPC / 4; ++q) {
              const float4 xv = xr[q];
              acc[r] = fmaf(wv[4 * q], xv.x, acc[r]);
              acc[r] = fmaf(wv[4 * q + 1], xv.y, acc[r]);
              acc[r] = fmaf(wv[4 * q + 2], xv.z, acc[r]);
              acc[r] = fmaf(wv[4 * q + 3], xv.w, acc[r]);
            }
          }
        }
      }
      const int o = o0 + v;
#pragma unroll
      for (int r = 0; r < GV_R; ++r) {
        if (r < nr) {
          const float sum = wave_sum(acc[r]);
          if (lane == 0 && o < N) y[(long)r * ldy + o] = sum + (b ? to_f32<WT>(b[o]) : 0.f);
        }
      }
    }
  }
}

// ---------------------------------------------------------------- adaLN LayerNorm
// out = LN(x) * (1 + scale[req]) + shift[req], LN with biased variance and no
// affine; statistics in fp32 with a two-pass (mean, then centred squares)
// evaluation from registers.  One wavefront per row, NV float4 per lane
// (H <= 256 NV, at most LN_MAX_H), NV fixed at compile time so the row uses
// no more registers than it needs and more rows stay in flight.

template <typename OT, int NV>
__global__ __launch_bounds__(256) void ln_mod_kernel(const float* __restrict__ X, int H, int row_begin,
                                                     int row_end, const BatchMeta meta,
                                                     const float* __restrict__ mods, int mods_ld, int sh_t,
                                                     int sc_t, int sh_i, int sc_i, float eps, OT* __restrict__ out,
                                                     long ldo) {
  const int lane = threadIdx.x & 63;
  const int R = row_begin + blockIdx.x * 4 + (threadIdx.x >> 6);
  if (R >= row_end) return;
  const int H4 = H >> 2;
  const float4* xr = (const float4*)(X + (long)R * H);
  const RowInfo ri = row_info(meta, R);
  const float* mrow = mods + (long)ri.req * mods_ld;
  const float4* shv = (const float4*)(mrow + (ri.is_img ? sh_i : sh_t));
  const float4* scv = (const float4*)(mrow + (ri.is_img ? sc_i : sc_t));
  // float4 i of a lane is float4 lane + 64 i of the row; lanes past the row
  // load its last float4 again and weigh it by zero (no load behind a branch,
  // so all of them are in flight at once)
  int cidx[NV];
  float keep[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    cidx[i] = min(lane + i * 64, H4 - 1);
    keep[i] = lane + i * 64 < H4 ? 1.f : 0.f;
  }
  float4 v[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = xr[cidx[i]];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) s += keep[i] * ((v[i].x + v[i].y) + (v[i].z + v[i].w));
  const float mean = wave_sum(s) / (float)H;
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i].x -= mean;
    v[i].y -= mean;
    v[i].z -= mean;
    v[i].w -= mean;
    ss += keep[i] * ((v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w));
  }
  const float rstd = 1.0f / sqrtf(wave_sum(ss) / (float)H + eps);
  OT* orow = out + (long)(R - row_begin) * ldo;
  // Every lane stores: a lane past the row's end writes the row's last
  // float4 with exactly the bytes the lane that owns it writes (same inputs,
  // same arithmetic), so no store needs a branch and the shift / scale loads
  // all leave before the first store.
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = cidx[i];
    const float4 sh = shv[c], sc = scv[c];
    const float y0 = v[i].x * rstd * (1.f + sc.x) + sh.x;
    const float y1 = v[i].y * rstd * (1.f + sc.y) + sh.y;
    const float y2 = v[i].z * rstd * (1.f + sc.z) + sh.z;
    const float y3 = v[i].w * rstd * (1.f + sc.w) + sh.w;
    if constexpr (sizeof(OT) == 2) {
      uint2 w;
      w.x = pack_bf16x2(y0, y1);
      w.y = pack_bf16x2(y2, y3);
      *(uint2*)(orow + c * 4) = w;
    } else {
      *(float4*)(orow + c * 4) = make_float4(y0, y1, y2, y3);
    }
  }
}

// ---------------------------------------------------------------- Euler
struct DtArgs {
  float dt[kMaxReq];
};
template <typename T>
__global__ void euler_kernel(T* __restrict__ x, const T* __restrict__ v, long n, int channels, const BatchMeta meta,
                             DtArgs da) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int row = (int)(i / channels);
  int r = 0;
  while (r + 1 < meta.n_req && row >= meta.img_off[r + 1]) ++r;
  const float xv = to_f32<T>(x[i]), vv = to_f32<T>(v[i]);
  x[i] = from_f32<T>(xv - da.dt[r] * vv);
}

// ---------------------------------------------------------------- V relayout
// v [T_joint][heads][d] -> V^T [heads][d][padded positions], columns in
// vt_slot order, a request's padding keys zero.  A block moves 64 padded
// positions x 64 dimensions of a head through LDS, with 16-byte loads along d
// and 16-byte stores along the keys (a thread stores one 16-key group of one
// row).  At 16 896 tokens and 6 heads of 128 (26 MB each way) 15 us with its
// launch, against 43 us for element-wise accesses and a second launch for the
// padding.
template <typename T>
__global__ __launch_bounds__(256) void v_transpose_kernel(const T* __restrict__ v, const BatchMeta meta, int heads,
                                                          int d, T* __restrict__ vt, long ld) {
  constexpr int E = 16 / sizeof(T);            // elements of a 16-byte piece
  constexpr int WORDS = 64 * sizeof(T) / 4;    // 4-byte words of a tile row
  constexpr int PITCH = WORDS + 1;             // odd: a column's rows fall on different banks
  __shared__ uint32_t tile[64 * PITCH];
  const int p0 = blockIdx.x * 64, d0 = blockIdx.y * 64, h = blockIdx.z;
  int r = 0;  // pad_off are multiples of 64: the positions belong to one request
  while (r + 1 < meta.n_req && p0 >= meta.pad_off[r + 1]) ++r;
  const int q0 = p0 - meta.pad_off[r];
  const int left = meta.joint_off[r + 1] - meta.joint_off[r] - q0;  // keys of the request from here on
  const T* src = v + ((long)(meta.joint_off[r] + q0) * heads + h) * d + d0;
#pragma unroll
  for (int u = 0; u < 64 * 64 / E / 256; ++u) {
    const int i = threadIdx.x + u * 256, row = i / (64 / E), c = i % (64 / E);
    uint4 w = make_uint4(0, 0, 0, 0);
    if (row < left) w = *(const uint4*)(src + (long)row * heads * d + c * E);
    uint32_t* t = &tile[row * PITCH + c * 4];
    t[0] = w.x;
    t[1] = w.y;
    t[2] = w.z;
    t[3] = w.w;
  }
  __syncthreads();
  const int dd = threadIdx.x >> 2, g = (threadIdx.x & 3) * 16;
  T o[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) o[q] = ((const T*)&tile[(g + vt_slot(q)) * PITCH])[dd];
  T* dst = vt + ((long)h * d + d0 + dd) * ld + p0 + g;
#pragma unroll
  for (int q = 0; q < 16 / E; ++q) *(uint4*)(dst + q * E) = *(const uint4*)(o + q * E);
}

}  // namespace

hipError_t launch_timestep_embed(float* e, int n_req, const float* t_host, int dim, hipStream_t s) {
  TimeArgs ta{};
  for (int r = 0; r < n_req; ++r) ta.t[r] = t_host[r];
  const int n = n_req * dim;
  hipLaunchKernelGGL(timestep_kernel, dim3((n + 255) / 256), dim3(256), 0, s, e, n_req, ta, dim);
  return hipGetLastError();
}

template <typename WT, int MAXC>
void gemv_launch(int blocks, int sblocks, size_t shmem, hipStream_t s, const void* W, const void* b, const float* x,
                 long ldx, int nr, int K, int N, int act, float* y, long ldy, const TimeArgs& ta, const SetupArgs& su) {
  if (sblocks > 0 || act == GEMV_TIMESTEP)
    hipLaunchKernelGGL((gemv_kernel<WT, MAXC, true>), dim3(blocks + sblocks), dim3(256), shmem, s, (const WT*)W,
                       (const WT*)b, x, ldx, nr, K, N, act, y, ldy, ta, sblocks, su);
  else
    hipLaunchKernelGGL((gemv_kernel<WT, MAXC, false>), dim3(blocks), dim3(256), shmem, s, (const WT*)W, (const WT*)b, x,
                       ldx, nr, K, N, act, y, ldy, ta, 0, su);
}

// 256-thread blocks per CU that the registers of each instance allow (its waves
// per SIMD), by its MAXC and FIRST
constexpr int kGemvMaxC[] = {1, 2, 3, 4, 6, 8, 16};
constexpr int kGemvPerCuBf16[2][7] = {{8, 7, 5, 4, 3, 2, 1}, {6, 6, 5, 4, 3, 2, 1}};
constexpr int kGemvPerCuF32[2][7] = {{8, 8, 8, 7, 4, 3, 2}, {6, 6, 6, 6, 5, 3, 2}};
constexpr size_t kLdsPerCu = 160 * 1024;

// 16-byte chunks per lane of a row of K weights
template <typename WT>
int gemv_chunks(int K) {
  return (K / GemvShape<WT>::EPC + 63) / 64;
}
int gemv_blocks_per_cu(int wdtype, int K, bool first) {
  const int c = wdtype == DIT_BF16 ? gemv_chunks<bf16_t>(K) : gemv_chunks<float>(K);
  int i = 0;
  while (kGemvMaxC[i] < c) ++i;
  return (wdtype == DIT_BF16 ? kGemvPerCuBf16 : kGemvPerCuF32)[first][i];
}

template <typename WT, class... A>
void gemv_dispatch(int K, A&&... a) {
  const int c = gemv_chunks<WT>(K);
  if (c <= 1) gemv_launch<WT, 1>(a...);
  else if (c <= 2) gemv_launch<WT, 2>(a...);
  else if (c <= 3) gemv_launch<WT, 3>(a...);
  else if (c <= 4) gemv_launch<WT, 4>(a...);
  else if (c <= 6) gemv_launch<WT, 6>(a...);
  else if (c <= 8) gemv_launch<WT, 8>(a...);
  else gemv_launch<WT, 16>(a...);
}

hipError_t launch_gemv(int wdtype, const void* W, const void* b, const float* x, long ldx, int n_req, int K,
                       int N, int act, const float* t_host, float* y, long ldy, const SetupArgs* setup,
                       hipStream_t s) {
  if (K > LN_MAX_H) return hipErrorInvalidValue;
  const size_t shmem = (size_t)(n_req < GV_R ? n_req : GV_R) * K * sizeof(float);
  const int V = wdtype == DIT_BF16 ? GemvShape<bf16_t>::V : GemvShape<float>::V;
  int blocks = (N + 4 * V - 1) / (4 * V);
  // Launches of a few rounds of resident blocks take one round of blocks that
  // loop evenly instead: each new block waits for its activations before it asks
  // for weights (cold weights, us between events, one block per 4 V rows against
  // one even round; bf16, 36 864 rows: K 3072 47.0 -> 41.4 and with four requests
  // 92 -> 69, K 4096 72 -> 56, K 2048 31.3 -> 29.6; fp32, 36 864 rows of 1024
  // 26.7 -> 26.5, four requests 48 -> 38).  The round is what the instance's own
  // registers and the activations' LDS hold: with three blocks per CU for every
  // K, launches of 30 720 rows of 512 take 11.5 us instead of 9.0.  Longer
  // launches hide that wait (262 144 rows: equal), and below two rounds the loop
  // would leave CUs idle.
  const int per_cu = std::min(gemv_blocks_per_cu(wdtype, K, setup || act == GEMV_TIMESTEP), (int)(kLdsPerCu / shmem));
  const int resident = 256 * per_cu;
  constexpr int kMaxBlocks = 256 * 32;
  if (blocks > kMaxBlocks) {
    blocks = kMaxBlocks;
  } else if (blocks > 2 * resident) {
    const int rounds = (blocks + resident - 1) / resident;
    blocks = (blocks + rounds - 1) / rounds;
  }
  SetupArgs su{};
  if (setup) su = *setup;
  for (int r0 = 0; r0 < n_req; r0 += GV_R) {
    const int nr = n_req - r0 < GV_R ? n_req - r0 : GV_R;
    TimeArgs ta{};
    if (act == GEMV_TIMESTEP)
      for (int r = 0; r < nr; ++r) ta.t[r] = t_host[r0 + r];
    const int sblocks = setup && r0 == 0 ? kSetupBlocks : 0;
    const float* xr = x ? x + (long)r0 * ldx : nullptr;
    float* yr = y + (long)r0 * ldy;
    if (wdtype == DIT_BF16)
      gemv_dispatch<bf16_t>(K, blocks, sblocks, shmem, s, W, b, xr, ldx, nr, K, N, act, yr, ldy, ta, su);
    else
      gemv_dispatch<float>(K, blocks, sblocks, shmem, s, W, b, xr, ldx, nr, K, N, act, yr, ldy, ta, su);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_ln_modulate(int out_dtype, const float* X, int H, int row_begin, int row_end,
                              const BatchMeta& meta, const float* mods, int mods_ld, int shift_txt, int scale_txt,
                              int shift_img, int scale_img, float eps, void* out, long ldo, hipStream_t s) {
  const int rows = row_end - row_begin;
  if (rows <= 0) return hipSuccess;
  if (H > LN_MAX_H) return hipErrorInvalidValue;
  const dim3 grid((rows + 3) / 4);
  const int nv = (H / 4 + 63) / 64;
#define DIT_LN_LAUNCH(OT, NV)                                                                                 \
  hipLaunchKernelGGL((ln_mod_kernel<OT, NV>), grid, dim3(256), 0, s, X, H, row_begin, row_end, meta, mods, mods_ld, \
                     shift_txt, scale_txt, shift_img, scale_img, eps, (OT*)out, ldo)
#define DIT_LN_DISPATCH(OT)          \
  if (nv <= 2) DIT_LN_LAUNCH(OT, 2);  \
  else if (nv <= 4) DIT_LN_LAUNCH(OT, 4); \
  else if (nv <= 8) DIT_LN_LAUNCH(OT, 8); \
  else if (nv <= 12) DIT_LN_LAUNCH(OT, 12); \
  else DIT_LN_LAUNCH(OT, 16);
  if (out_dtype == DIT_BF16) {
    DIT_LN_DISPATCH(bf16_t)
  } else {
    DIT_LN_DISPATCH(float)
  }
#undef DIT_LN_DISPATCH
#undef DIT_LN_LAUNCH
  return hipGetLastError();
}

hipError_t launch_euler(int dtype, void* x, const void* v, int channels, const BatchMeta& meta,
                        const float* dt_host, hipStream_t s) {
  DtArgs da{};
  for (int r = 0; r < meta.n_req; ++r) da.dt[r] = dt_host[r];
  const long n = (long)meta.T_img * channels;
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)((n + 255) / 256));
  if (dtype == DIT_BF16)
    hipLaunchKernelGGL(euler_kernel<bf16_t>, grid, dim3(256), 0, s, (bf16_t*)x, (const bf16_t*)v, n, channels, meta,
                       da);
  else
    hipLaunchKernelGGL(euler_kernel<float>, grid, dim3(256), 0, s, (float*)x, (const float*)v, n, channels, meta,
                       da);
  return hipGetLastError();
}

hipError_t launch_v_transpose(int dtype, const void* v, const BatchMeta& meta, int heads, int d, void* vt,
                              hipStream_t s) {
  const long ld = meta.pad_off[meta.n_req];
  if (meta.T == 0) return hipSuccess;
  if (d % 64 != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(ld / 64), d / 64, heads);
  if (dtype == DIT_BF16)
    hipLaunchKernelGGL(v_transpose_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)v, meta, heads, d,
                       (bf16_t*)vt, ld);
  else
    hipLaunchKernelGGL(v_transpose_kernel<float>, grid, dim3(256), 0, s, (const float*)v, meta, heads, d, (float*)vt,
                       ld);
  return hipGetLastError();
}

}  // namespace dit
