// float32 GEMM for float32 stages (fully-connected layers) on the matrix
// cores: v_mfma_f32_32x32x2_f32, float32 operands and accumulation, any M, N,
// K and leading dimension, plain operand modes.
//
// Two kernels, chosen by pick():
//
// Tile kernel (gemm_f32_kernel): 64 x 64 block tile, 4 waves each owning a
// 32 x 32 sub-tile, K step 32. The bound is the matrix cores (157 TFLOP/s):
// a K step is 16 MFMAs, 1024 cycles a wave, against 16 KB of loads and two
// 16-byte LDS reads per four MFMAs. What has to be hidden is the loads'
// latency: 16-byte global loads run two K steps ahead in registers, LDS holds
// two steps, one barrier a step, and K is split over blocks until every CU
// has two of them; a second pass sums the float32 partials in split order and
// applies the epilogue.
//
// Short kernel (gemm_f32_short_kernel): one 32 x 32 tile per block, K split
// over its 8 waves, operands loaded from global memory straight into MFMA
// fragments and the waves' partial tiles added in wave order in LDS. For
// products that are a launch and one round of loads long, where a K split
// over blocks would pay a second launch (about 5 us) to sum its partials.
#include <algorithm>
#include <cstdio>

#include "kernels.hpp"

namespace spx {
namespace {

constexpr int TB = 64, TK = 32, NT = 256;
constexpr int KP = TK + 4;           // K-mode LDS pitch: 16 rows' 16-byte chunks on distinct banks
constexpr int RP = TB + 8;           // R-mode LDS pitch: k and k + 4 on opposite halves of the 64 banks
constexpr int TARGET_BLOCKS = 512;   // split K until about this many blocks run (two per CU)
constexpr int MIN_SPLIT_STEPS = 4;   // K steps per split at least
constexpr int MAX_SPLITS = 64;
constexpr int SW = 8;                // waves of a short-kernel block
constexpr int SCH = 32;              // k per wave and round of the short kernel

struct F32Args {
  int M, N, K;
  int splits, k_per_split;   // splits > 1: raw partials [split][M][N] to `partial`
  float* partial;
  const float* A;
  long lda;
  const float* B;
  long ldb;
  float* out;
  long ldc;
  const float* bias;
  const float* res;
  const float* mask;
  float alpha;
  int relu, accumulate;
};

// A thread's two groups of four elements of a 64 x 32 operand tile:
// K-mode (X[r ld + k]): rows t / 8 + 32 i, k 4 (t % 8) ..; R-mode
// (X[k ld + r]): k t / 16 + 16 i, rows 4 (t % 16) .. . VEC: 16-byte loads
// (aligned pointer and leading dimension, contiguous extent a multiple of 4,
// so a group lies inside the operand or outside it); otherwise element loads.
template <int MODE, bool VEC>
struct TileLoader {
  float4 v[2];
  __device__ __forceinline__ void load(const float* X, long ld, int rows, int kend, int row0, int k0, int tid) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = row0 + (MODE == OP_K_PLAIN ? (tid >> 3) + 32 * i : 4 * (tid & 15));
      const int k = k0 + (MODE == OP_K_PLAIN ? 4 * (tid & 7) : (tid >> 4) + 16 * i);
      float4 x = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (r < rows && k < kend) {
        const float* p = MODE == OP_K_PLAIN ? X + static_cast<long>(r) * ld + k : X + static_cast<long>(k) * ld + r;
        if (VEC) {
          x = *reinterpret_cast<const float4*>(p);
        } else {
          const int left = MODE == OP_K_PLAIN ? kend - k : rows - r;
          x.x = p[0];
          if (left > 1) x.y = p[1];
          if (left > 2) x.z = p[2];
          if (left > 3) x.w = p[3];
        }
      }
      v[i] = x;
    }
  }
  __device__ __forceinline__ void store(float* S, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float* p = MODE == OP_K_PLAIN ? S + ((tid >> 3) + 32 * i) * KP + 4 * (tid & 7)
                                    : S + ((tid >> 4) + 16 * i) * RP + 4 * (tid & 15);
      *reinterpret_cast<float4*>(p) = v[i];
    }
  }
};

// Four of the eight k of group q (k 8 q .. 8 q + 7 of the step) for row
// `row`: the lanes of half h hold k 8 q + 4 h + j, and MFMA j takes element j
// of both halves. K-mode: one 16-byte read; R-mode: four.
template <int MODE>
__device__ __forceinline__ float4 frag(const float* S, int row, int q, int h) {
  if (MODE == OP_K_PLAIN) return *reinterpret_cast<const float4*>(S + row * KP + 8 * q + 4 * h);
  const float* p = S + (8 * q + 4 * h) * RP + row;
  return make_float4(p[0], p[RP], p[2 * RP], p[3 * RP]);
}

// value = acc * alpha + bias + residual, ReLU, mask, then stored or added.
__device__ __forceinline__ void epilogue_f32(const F32Args& a, int row, int col, float acc) {
  const long idx = static_cast<long>(row) * a.ldc + col;
  float v = acc * a.alpha;
  if (a.bias) v += a.bias[col];
  if (a.res) v += a.res[idx];
  if (a.relu) v = fmaxf(v, 0.0f);
  if (a.mask && !(a.mask[idx] > 0.0f)) v = 0.0f;
  if (a.accumulate) a.out[idx] += v;
  else a.out[idx] = v;
}

// The A fragment is the first MFMA operand: lane l holds column l % 32 of the
// wave's 32 x 32 tile, rows 8 (r / 4) + 4 (l / 32) + r % 4 in register r, so
// every store of a wave writes two whole 128-byte row segments.
template <int MA, int MB, bool VEC>
__global__ __launch_bounds__(NT) void gemm_f32_kernel(F32Args a) {
  constexpr int ASZ = MA == OP_K_PLAIN ? TB * KP : TK * RP, BSZ = MB == OP_K_PLAIN ? TB * KP : TK * RP;
  __shared__ __attribute__((aligned(16))) float As[2][ASZ];
  __shared__ __attribute__((aligned(16))) float Bs[2][BSZ];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.y * TB, col0 = blockIdx.x * TB;
  const int kbeg = blockIdx.z * a.k_per_split, kend = min(a.K, kbeg + a.k_per_split);
  const int ra = (wave >> 1) * 32 + (lane & 31), rb = (wave & 1) * 32 + (lane & 31), h = lane >> 5;
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

  TileLoader<MA, VEC> la0, la1;
  TileLoader<MB, VEC> lb0, lb1;
  auto fetch = [&](TileLoader<MA, VEC>& la, TileLoader<MB, VEC>& lb, int k0) {
    la.load(a.A, a.lda, a.M, kend, row0, k0, tid);   // a step past the end loads zeros
    lb.load(a.B, a.ldb, a.N, kend, col0, k0, tid);
  };
  auto compute = [&](const float* sa, const float* sb) {
#pragma unroll
    for (int q = 0; q < TK / 8; ++q) {
      const float4 fa = frag<MA>(sa, ra, q, h), fb = frag<MB>(sb, rb, q, h);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.x, fb.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.y, fb.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.z, fb.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.w, fb.w, acc, 0, 0, 0);
    }
  };
  // Register sets 0 / 1 carry the steps of even / odd index, LDS buffer b the
  // step being multiplied (index parity b).
  fetch(la0, lb0, kbeg);
  fetch(la1, lb1, kbeg + TK);
  la0.store(As[0], tid);
  lb0.store(Bs[0], tid);
  __syncthreads();
  const int nk = (kend - kbeg + TK - 1) / TK;
  for (int kt = 0; kt < nk; kt += 2) {
    fetch(la0, lb0, kbeg + (kt + 2) * TK);
    compute(As[0], Bs[0]);
    la1.store(As[1], tid);
    lb1.store(Bs[1], tid);
    __syncthreads();
    if (kt + 1 >= nk) break;
    fetch(la1, lb1, kbeg + (kt + 3) * TK);
    compute(As[1], Bs[1]);
    la0.store(As[0], tid);
    lb0.store(Bs[0], tid);
    __syncthreads();
  }
  const int col = col0 + rb;
  if (col >= a.N) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = row0 + (wave >> 1) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
    if (row >= a.M) continue;
    if (a.splits > 1)
      a.partial[(static_cast<long>(blockIdx.z) * a.M + row) * a.N + col] = acc[r];
    else
      epilogue_f32(a, row, col, acc[r]);
  }
}

// Four elements k .. k + 3 of one row (zero past kend or for a row outside the
// operand).
template <int MODE, bool VEC>
__device__ __forceinline__ void short_load(const float* X, long ld, bool ok, int row, int k, int kend, float4& v) {
  v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (!ok || k >= kend) return;
  if (MODE == OP_K_PLAIN) {
    const float* p = X + static_cast<long>(row) * ld + k;
    if (VEC) {
      v = *reinterpret_cast<const float4*>(p);
      return;
    }
    v.x = p[0];
    if (k + 1 < kend) v.y = p[1];
    if (k + 2 < kend) v.z = p[2];
    if (k + 3 < kend) v.w = p[3];
  } else {
    const float* p = X + static_cast<long>(k) * ld + row;
    v.x = p[0];
    if (k + 1 < kend) v.y = p[ld];
    if (k + 2 < kend) v.z = p[2 * ld];
    if (k + 3 < kend) v.w = p[3 * ld];
  }
}

template <int MA, int MB, bool VEC>
__global__ __launch_bounds__(64 * SW) void gemm_f32_short_kernel(F32Args a) {
  __shared__ float red[SW][32][33];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5;
  const int row0 = blockIdx.y * 32, col0 = blockIdx.x * 32;
  const int ra = row0 + (lane & 31), rb = col0 + (lane & 31);
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  // round j of wave w: k SCH (SW j + w) .. + SCH - 1; the next round's loads
  // are issued before this round's MFMAs
  constexpr int G = SCH / 8;
  float4 fa[2][G], fb[2][G];
  auto fetch = [&](float4 (&va)[G], float4 (&vb)[G], int k0) {
#pragma unroll
    for (int q = 0; q < G; ++q) {
      short_load<MA, VEC>(a.A, a.lda, ra < a.M, ra, k0 + 8 * q + 4 * h, a.K, va[q]);
      short_load<MB, VEC>(a.B, a.ldb, rb < a.N, rb, k0 + 8 * q + 4 * h, a.K, vb[q]);
    }
  };
  auto compute = [&](const float4 (&va)[G], const float4 (&vb)[G]) {
#pragma unroll
    for (int q = 0; q < G; ++q) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va[q].x, vb[q].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va[q].y, vb[q].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va[q].z, vb[q].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va[q].w, vb[q].w, acc, 0, 0, 0);
    }
  };
  constexpr int STEP = SW * SCH;
  int k0 = wave * SCH;
  fetch(fa[0], fb[0], k0);
  for (; k0 < a.K; k0 += 2 * STEP) {
    fetch(fa[1], fb[1], k0 + STEP);
    compute(fa[0], fb[0]);
    fetch(fa[0], fb[0], k0 + 2 * STEP);
    compute(fa[1], fb[1]);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][8 * (r >> 2) + 4 * h + (r & 3)][lane & 31] = acc[r];
  __syncthreads();
#pragma unroll
  for (int e = tid; e < 32 * 32; e += 64 * SW) {
    const int i = e >> 5, j = e & 31;
    float v = red[0][i][j];
#pragma unroll
    for (int w = 1; w < SW; ++w) v += red[w][i][j];
    if (row0 + i < a.M && col0 + j < a.N) epilogue_f32(a, row0 + i, col0 + j, v);
  }
}

// Sums the split partials of each output in split order, then the epilogue.
__global__ __launch_bounds__(256) void gemm_f32_reduce_kernel(F32Args a) {
  const long mn = static_cast<long>(a.M) * a.N;
  for (long t = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; t < mn; t += static_cast<long>(gridDim.x) * 256) {
    float s = a.partial[t];
#pragma unroll 8
    for (int sp = 1; sp < a.splits; ++sp) s += a.partial[sp * mn + t];
    const int row = static_cast<int>(t / a.N), col = static_cast<int>(t - static_cast<long>(row) * a.N);
    epilogue_f32(a, row, col, s);
  }
}

// Kernel and K split of a product. The short kernel serves grids of few waves
// whose blocks run few rounds one after the other: at most four rounds of
// SW SCH = 256 k (2 us each, which no idle CU shortens),
// and up to 256K (32 x 32 tile, k) pairs, past which the tile kernel's reuse of
// each load 64 times wins. us, short against tile kernel with its reduction:
//   32 x 10:   K = 256 7.9 / 11.5, 512 8.9 / 11.4, 1024 12.5 / 12.4,
//              2048 20.1 / 13.0, 8192 63 / 15.5, 65536 494 / 36, 262144 1970 / 110
//   256 x 128: K = 256 8.4 / 11.4, 1024 14.5 / 13.6, 2048 23.2 / 14.3
//   512 x 256: K = 256 8.4 / 11.7, 1024 14.9 / 14.6, 2048 25.8 / 19.1
// At 1024 the one launch saved decides. A product of 32 x 256 x 784 takes one
// launch instead of two (the three-layer classifier: 113 -> 88 us a
// mini-batch); 128 x 2048 x 3072, long since past the limits, took 105 us with
// the former 16-deep, element-loading tile (a step of three such layers 851 ->
// 229 us).
struct Pick {
  bool short_k;
  int splits, steps_per;
};

Pick pick(int M, int N, int K, bool ws, size_t ws_bytes) {
  const long t32 = static_cast<long>((M + 31) / 32) * ((N + 31) / 32);
  const long t64 = static_cast<long>((M + TB - 1) / TB) * ((N + TB - 1) / TB);
  const int ksteps = (K + TK - 1) / TK;
  Pick p{false, 1, std::max(1, ksteps)};
  if (K <= 4 * SW * SCH && t32 <= 1024 && K * t32 <= 256L * 1024) {
    p.short_k = true;
    return p;
  }
  if (ws && t64 < TARGET_BLOCKS && ksteps >= 2 * MIN_SPLIT_STEPS) {
    int splits = static_cast<int>(std::min<long>(TARGET_BLOCKS / t64, ksteps / MIN_SPLIT_STEPS));
    splits = std::min(splits, MAX_SPLITS);
    while (splits > 1 && static_cast<size_t>(splits) * M * N * 4 > ws_bytes) --splits;
    p.steps_per = std::max(1, (ksteps + splits - 1) / std::max(1, splits));
    p.splits = std::max(1, (ksteps + p.steps_per - 1) / p.steps_per);   // no empty split
  }
  return p;
}

bool vec_operand(const Operand& o, int rows, int K) {
  return (reinterpret_cast<uintptr_t>(o.ptr) & 15) == 0 && o.ld % 4 == 0 && (o.mode == OP_K_PLAIN ? K : rows) % 4 == 0;
}

template <int MA, int MB, bool VEC>
hipError_t launch(const F32Args& a, bool short_k, hipStream_t s) {
  if (short_k) {
    hipLaunchKernelGGL((gemm_f32_short_kernel<MA, MB, VEC>), dim3((a.N + 31) / 32, (a.M + 31) / 32), dim3(64 * SW), 0,
                       s, a);
    return hipGetLastError();
  }
  dim3 grid((a.N + TB - 1) / TB, (a.M + TB - 1) / TB, a.splits);
  hipLaunchKernelGGL((gemm_f32_kernel<MA, MB, VEC>), grid, dim3(NT), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.splits == 1) return e;
  const long mn = static_cast<long>(a.M) * a.N;
  const long blocks = std::min<long>((mn + 255) / 256, 4096);
  hipLaunchKernelGGL(gemm_f32_reduce_kernel, dim3(static_cast<int>(blocks)), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int MA, int MB>
hipError_t launch(const F32Args& a, bool short_k, bool vec, hipStream_t s) {
  return vec ? launch<MA, MB, true>(a, short_k, s) : launch<MA, MB, false>(a, short_k, s);
}

}  // namespace

const char* gemm_f32_kernel_name(const GemmDesc& d) {
  static thread_local char buf[48];
  const Pick p = pick(d.M, d.N, d.K, d.workspace != nullptr, d.workspace_bytes);
  const bool vec = vec_operand(d.A, d.M, d.K) && vec_operand(d.B, d.N, d.K);
  std::snprintf(buf, sizeof(buf), "gemm_f32_%skernel<%d, %d, %s>", p.short_k ? "short_" : "", d.A.mode, d.B.mode,
                vec ? "true" : "false");
  return buf;
}

hipError_t gemm_f32(const GemmDesc& d, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  if (d.batch != 1 || !d.epi.out_f32 || d.epi.out_bf16 || d.epi.res_bf16) return hipErrorInvalidValue;
  F32Args a{};
  a.M = d.M;
  a.N = d.N;
  a.K = d.K;
  a.A = static_cast<const float*>(d.A.ptr);
  a.lda = d.A.ld;
  a.B = static_cast<const float*>(d.B.ptr);
  a.ldb = d.B.ld;
  a.out = d.epi.out_f32;
  a.ldc = d.epi.ldc;
  a.bias = d.epi.bias;
  a.res = d.epi.res_f32;
  a.mask = static_cast<const float*>(d.epi.mask);
  a.alpha = d.epi.alpha;
  a.relu = d.epi.relu;
  a.accumulate = d.epi.accumulate;
  const Pick p = pick(d.M, d.N, d.K, d.workspace != nullptr, d.workspace_bytes);
  a.splits = p.splits;
  a.k_per_split = p.steps_per * TK;
  a.partial = d.workspace;
  const bool vec = vec_operand(d.A, d.M, d.K) && vec_operand(d.B, d.N, d.K);
  const int ma = d.A.mode, mb = d.B.mode;
  if (ma == OP_K_PLAIN && mb == OP_K_PLAIN) return launch<OP_K_PLAIN, OP_K_PLAIN>(a, p.short_k, vec, s);
  if (ma == OP_K_PLAIN && mb == OP_R_PLAIN) return launch<OP_K_PLAIN, OP_R_PLAIN>(a, p.short_k, vec, s);
  if (ma == OP_R_PLAIN && mb == OP_R_PLAIN) return launch<OP_R_PLAIN, OP_R_PLAIN>(a, p.short_k, vec, s);
  return hipErrorInvalidValue;
}

}  // namespace spx
