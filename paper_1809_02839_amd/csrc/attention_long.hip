// Fused multi-head attention core for any sequence length (head dimension 32
// or 64) on gfx950; attention.hip has the one-block form for 128 rows of 64.
//
// The score matrix never reaches memory: forward and backward recompute it in
// tiles from Q and K, so a layer keeps two floats per row instead of six bytes
// per score, and the nine launches of the batched-GEMM form (bound by moving 10
// bytes per score in each softmax pass at 3.3 TB/s) become three. What bounds
// these is the chain of small products and exponentials of a group (exp_neg).
// At S = 328, 24 x 8 heads of 64: forward 46 us (scores, softmax and P V were
// 30 + 63 + 30), backward 95 us (four products and the softmax backward were
// 4 x 28 + 60); an encoder layer's step 600 -> 433 us. A first version that
// passed P and dS through LDS with four barriers a tile took 54 and 167 us.
//
// Rounding is that of the batched form: scores, row maxima, probabilities and
// dP in float32; bf16(P) with P already normalised, so the forward makes two
// passes over the keys (row statistics, then P V) instead of rescaling
// unnormalised tiles; dS = bf16(P (dP - rowsum(P dP))).
//
// Forward and dQ: a block owns 128 query rows of one (batch, head) and walks
// the key tiles; dK and dV: a block owns 128 keys and walks the query tiles.
// Four waves, each with 32 of the block's rows. The fragment of the walked
// operand goes first into v_mfma_f32_32x32x16_bf16, so a lane ends with its
// own row's (lane % 32) scores against columns 8 (r / 4) + 4 (lane / 32) +
// r % 4 of a 32-column group. Those registers, rounded to bf16, are already
// an operand of the next product: its k order is free as long as both
// operands share it, so registers 8 c .. 8 c + 7 serve as the lane's eight k
// of step c and the other operand is read with the same k (frag_cols). So P
// and dS never go through LDS, a tile costs two barriers, and one 32-column
// group's values are all that is live: LDS holds the two staged tiles only and
// three blocks of the forward and dQ (two of dK and dV, which hold two
// results) share a CU.
// Rows past the sequence are staged as zeros and their probabilities set to 0.
#include "kernels.hpp"

namespace spx {
namespace {

constexpr int TS = 128, NT = 256;

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

__device__ __forceinline__ bf16x8_t gld8(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u16x8_t*>(p));
}
// 8 consecutive k of row `row` from an LDS tile [row][k] of pitch P.
template <int P>
__device__ __forceinline__ bf16x8_t frag_rows(const bf16_t* s, int row, int k) {
  return gld8(s + row * P + k);
}
// Operand for "row" m0 + lane % 32 from a tile stored [k][row], by two
// transposing reads (within a 16-lane group, lane i receives element i % 4 of
// the 8-byte chunk addressed by lane 4 q + i / 4, q < 4): the lanes of half h
// get k0 + 4 h + 0 .. 3 and k0 + 8 + 4 h + 0 .. 3, the k order of a score
// register group (see above).
template <int P>
__device__ __forceinline__ bf16x8_t frag_cols(const bf16_t* s, int m0, int k0, int lane) {
  const int g = lane >> 4, i = lane & 15;
  const bf16_t* p = s + (k0 + 4 * (g >> 1) + (i >> 2)) * P + m0 + 16 * (g & 1) + 4 * (i & 3);
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p + 8 * P));
  const u16x8_t v = {static_cast<uint16_t>(lo[0]), static_cast<uint16_t>(lo[1]), static_cast<uint16_t>(lo[2]),
                     static_cast<uint16_t>(lo[3]), static_cast<uint16_t>(hi[0]), static_cast<uint16_t>(hi[1]),
                     static_cast<uint16_t>(hi[2]), static_cast<uint16_t>(hi[3])};
  return __builtin_bit_cast(bf16x8_t, v);
}
__device__ __forceinline__ f32x16_t mfma(bf16x8_t b, bf16x8_t a, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0);
}
// exp(x) for x <= 0 in float32 accuracy: exp2 of x log2(e) carried in two
// floats (the product's rounding error enters through the first-order term).
// Eight instructions against the library function's twenty or more, and a
// layer's passes take five per score. Below -200 the result is zero either
// way; a NaN stays one.
__device__ __forceinline__ float exp_neg(float x) {
  constexpr float kLog2e = 1.44269502162933349609f, kLog2eLo = 1.92596299112661746887e-8f, kLn2 = 0.69314718055994530942f;
  x = x < -200.0f ? -200.0f : x;
  const float hi = x * kLog2e;
  const float lo = fmaf(x, kLog2eLo, fmaf(x, kLog2e, -hi));
  const float e = __builtin_amdgcn_exp2f(hi);
  return fmaf(e, lo * kLn2, e);
}
template <int N>
__device__ __forceinline__ void zero(f32x16_t (&a)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[j][r] = 0.0f;
}
// Column of register r inside a 32-column group.
__device__ __forceinline__ int col_of(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// A thread's share of a 128 x DH block of rows row0 .. (rows ld apart), zero
// past row S - 1, and its copy into an LDS tile [128][DH + 8].
template <int DH>
struct Rows {
  static constexpr int V = TS * DH / 8 / NT, C = DH / 8;
  uint4 v[V];
  __device__ __forceinline__ void load(const bf16_t* src, long ld, int row0, int S, int tid) {
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int e = tid + NT * i, row = row0 + e / C;
      v[i] = make_uint4(0, 0, 0, 0);
      if (row < S) v[i] = *reinterpret_cast<const uint4*>(src + row * ld + (e % C) * 8);
    }
  }
  __device__ __forceinline__ void store(bf16_t* dst, int tid) const {
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int e = tid + NT * i;
      *reinterpret_cast<uint4*>(dst + (e / C) * (DH + 8) + (e % C) * 8) = v[i];
    }
  }
};

// The wave's 32 rows (fragments fr) against rows c0 .. c0 + 31 of an LDS tile.
template <int DH>
__device__ __forceinline__ f32x16_t group_product(const bf16x8_t (&fr)[DH / 16], const bf16_t* tile, int c0,
                                                  int lane) {
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int q = 0; q < DH / 16; ++q)
    acc = mfma(frag_rows<DH + 8>(tile, c0 + (lane & 31), 16 * q + 8 * (lane >> 5)), fr[q], acc);
  return acc;
}

// acc += the group's values, rounded to bf16, times rows c0 .. of a [k][DH] tile.
template <int DH>
__device__ __forceinline__ void group_accumulate(const f32x16_t& v, const bf16_t* tile, int c0, int lane,
                                                 f32x16_t (&acc)[DH / 32]) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const uint4 u = make_uint4(pack_bf16x2(v[8 * c], v[8 * c + 1]), pack_bf16x2(v[8 * c + 2], v[8 * c + 3]),
                               pack_bf16x2(v[8 * c + 4], v[8 * c + 5]), pack_bf16x2(v[8 * c + 6], v[8 * c + 7]));
    const bf16x8_t fa = __builtin_bit_cast(bf16x8_t, u);
#pragma unroll
    for (int jn = 0; jn < DH / 32; ++jn)
      acc[jn] = mfma(frag_cols<DH + 8>(tile, 32 * jn, c0 + 16 * c, lane), fa, acc[jn]);
  }
}

template <int DH>
__device__ __forceinline__ void load_frags(const bf16_t* row, int lane, bf16x8_t (&f)[DH / 16]) {
#pragma unroll
  for (int q = 0; q < DH / 16; ++q) f[q] = gld8(row + 16 * q + 8 * (lane >> 5));
}

// Rows row0 + lane % 32 (below S) of a wave's 32 x DH result.
template <int DH>
__device__ __forceinline__ void store_rows(bf16_t* out, long ld, int row, int S, const f32x16_t (&acc)[DH / 32],
                                           float alpha, int lane) {
  if (row >= S) return;
#pragma unroll
  for (int jn = 0; jn < DH / 32; ++jn)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<uint2*>(out + row * ld + 32 * jn + col_of(4 * g, lane)) =
          make_uint2(pack_bf16x2(acc[jn][4 * g] * alpha, acc[jn][4 * g + 1] * alpha),
                     pack_bf16x2(acc[jn][4 * g + 2] * alpha, acc[jn][4 * g + 3] * alpha));
}

// One (batch, head): its packed qkv rows and the wave's place in the block.
template <int DH>
struct Place {
  const bf16_t *q, *k, *v;
  long ld;
  int b, h, lane, lrow;
  __device__ Place(const bf16_t* qkv, int S, int heads, int d)
      : ld(3L * d), b(blockIdx.y / heads), h(blockIdx.y - b * heads), lane(threadIdx.x & 63),
        lrow(32 * (threadIdx.x >> 6) + (lane & 31)) {
    q = qkv + static_cast<long>(b) * S * ld + h * DH;
    k = q + d;
    v = k + d;
  }
};

template <int DH>
__global__ __launch_bounds__(NT, 3) void attention_long_fwd_kernel(const bf16_t* qkv, int S, int heads, int d,
                                                                   float scale, float* stats, bf16_t* ctx) {
  __shared__ __attribute__((aligned(16))) bf16_t Vs[TS * (DH + 8)];
  __shared__ __attribute__((aligned(16))) bf16_t Ks[TS * (DH + 8)];
  const Place<DH> at(qkv, S, heads, d);
  const int tid = threadIdx.x, lane = at.lane, row = blockIdx.x * TS + at.lrow;
  const bool live = blockIdx.x * TS + 32 * (tid >> 6) < S;   // the wave has rows inside the sequence
  bf16x8_t fq[DH / 16];
  load_frags<DH>(at.q + min(row, S - 1) * at.ld, lane, fq);

  // row statistics: a row's group scores are in this lane and lane ^ 32
  float m = -INFINITY, sum = 0.0f;
  Rows<DH> kr, vr;
  kr.load(at.k, at.ld, 0, S, tid);
  for (int k0 = 0; k0 < S; k0 += TS) {
    __syncthreads();
    kr.store(Ks, tid);
    __syncthreads();
    kr.load(at.k, at.ld, k0 + TS, S, tid);
    if (!live) continue;
    for (int c0 = 0; c0 < TS && k0 + c0 < S; c0 += 32) {
      f32x16_t acc = group_product<DH>(fq, Ks, c0, lane);
      float t = m;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[r] = __fmul_rn(acc[r], scale);
        if (k0 + c0 + col_of(r, lane) < S) t = fmaxf(t, acc[r]);
      }
      t = fmaxf(t, __shfl_xor(t, 32));
      // scores of -infinity only so far count zero, as against any later maximum
      const float t0 = t == -INFINITY ? 0.0f : t;
      float e = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x = exp_neg(__fsub_rn(acc[r], t0));
        e += k0 + c0 + col_of(r, lane) < S ? x : 0.0f;
      }
      sum = k0 + c0 == 0 ? e : fmaf(sum, exp_neg(__fsub_rn(m, t0)), e);
      m = t;
    }
  }
  sum += __shfl_xor(sum, 32);
  const float inv = 1.0f / sum;
  if (lane < 32 && row < S) {
    float* st = stats + (static_cast<long>(blockIdx.y) * S + row) * 2;
    st[0] = m;
    st[1] = inv;
  }
  // ctx = bf16(P) V
  f32x16_t o[DH / 32];
  zero(o);
  kr.load(at.k, at.ld, 0, S, tid);
  vr.load(at.v, at.ld, 0, S, tid);
  for (int k0 = 0; k0 < S; k0 += TS) {
    __syncthreads();
    kr.store(Ks, tid);
    vr.store(Vs, tid);
    __syncthreads();
    kr.load(at.k, at.ld, k0 + TS, S, tid);
    vr.load(at.v, at.ld, k0 + TS, S, tid);
    if (!live) continue;
    for (int c0 = 0; c0 < TS && k0 + c0 < S; c0 += 32) {
      f32x16_t p = group_product<DH>(fq, Ks, c0, lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x = __fmul_rn(exp_neg(__fsub_rn(__fmul_rn(p[r], scale), m)), inv);
        p[r] = k0 + c0 + col_of(r, lane) < S ? x : 0.0f;
      }
      group_accumulate<DH>(p, Vs, c0, lane, o);
    }
  }
  store_rows<DH>(ctx + static_cast<long>(at.b) * S * d + at.h * DH, d, row, S, o, 1.0f, lane);
}

// dQ of 128 query rows, and the row sums of P dP for the other kernel.
template <int DH>
__global__ __launch_bounds__(NT, 3) void attention_long_dq_kernel(const bf16_t* qkv, const bf16_t* dctx,
                                                                  const float* stats, int S, int heads, int d,
                                                                  float scale, float* dots, bf16_t* dqkv) {
  __shared__ __attribute__((aligned(16))) bf16_t Vs[TS * (DH + 8)];
  __shared__ __attribute__((aligned(16))) bf16_t Ks[TS * (DH + 8)];
  const Place<DH> at(qkv, S, heads, d);
  const int tid = threadIdx.x, lane = at.lane, row = blockIdx.x * TS + at.lrow, rc = min(row, S - 1);
  const bool live = blockIdx.x * TS + 32 * (tid >> 6) < S;
  bf16x8_t fq[DH / 16], fo[DH / 16];
  load_frags<DH>(at.q + rc * at.ld, lane, fq);
  load_frags<DH>(dctx + (static_cast<long>(at.b) * S + rc) * d + at.h * DH, lane, fo);
  const long srow = static_cast<long>(blockIdx.y) * S + rc;
  const float m = stats[2 * srow], inv = stats[2 * srow + 1];

  // f(group's P, dP, first column) for every staged group inside the sequence
  Rows<DH> kr, vr;
  auto walk = [&](auto&& f) {
    kr.load(at.k, at.ld, 0, S, tid);
    vr.load(at.v, at.ld, 0, S, tid);
    for (int k0 = 0; k0 < S; k0 += TS) {
      __syncthreads();
      kr.store(Ks, tid);
      vr.store(Vs, tid);
      __syncthreads();
      kr.load(at.k, at.ld, k0 + TS, S, tid);
      vr.load(at.v, at.ld, k0 + TS, S, tid);
      if (!live) continue;
      for (int c0 = 0; c0 < TS && k0 + c0 < S; c0 += 32) {
        f32x16_t p = group_product<DH>(fq, Ks, c0, lane);
        const f32x16_t dp = group_product<DH>(fo, Vs, c0, lane);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x = __fmul_rn(exp_neg(__fsub_rn(__fmul_rn(p[r], scale), m)), inv);
          p[r] = k0 + c0 + col_of(r, lane) < S ? x : 0.0f;
        }
        f(p, dp, c0);
      }
    }
  };
  float dot = 0.0f;
  walk([&](f32x16_t& p, const f32x16_t& dp, int) {
#pragma unroll
    for (int r = 0; r < 16; ++r) dot += p[r] * dp[r];
  });
  dot += __shfl_xor(dot, 32);
  if (lane < 32 && row < S) dots[srow] = dot;

  f32x16_t o[DH / 32];
  zero(o);
  walk([&](f32x16_t& p, const f32x16_t& dp, int c0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = p[r] * (dp[r] - dot);
    group_accumulate<DH>(p, Ks, c0, lane, o);
  });
  store_rows<DH>(dqkv + static_cast<long>(at.b) * S * at.ld + at.h * DH, at.ld, row, S, o, scale, lane);
}

// dK and dV of 128 keys: the wave's rows are keys, the walked columns queries,
// whose statistics are staged with them.
template <int DH>
__global__ __launch_bounds__(NT, 2) void attention_long_dkv_kernel(const bf16_t* qkv, const bf16_t* dctx,
                                                                   const float* stats, const float* dots, int S,
                                                                   int heads, int d, float scale, bf16_t* dqkv) {
  __shared__ __attribute__((aligned(16))) bf16_t Os[TS * (DH + 8)];
  __shared__ __attribute__((aligned(16))) bf16_t Qs[TS * (DH + 8)];
  __shared__ __attribute__((aligned(16))) float ms[TS], is[TS], ds[TS];   // max, 1 / sum (0 past the sequence), dot
  const Place<DH> at(qkv, S, heads, d);
  const int tid = threadIdx.x, lane = at.lane, key = blockIdx.x * TS + at.lrow, kc = min(key, S - 1);
  const bool live = blockIdx.x * TS + 32 * (tid >> 6) < S;
  const bf16_t* dOg = dctx + static_cast<long>(at.b) * S * d + at.h * DH;
  bf16x8_t fk[DH / 16], fv[DH / 16];
  load_frags<DH>(at.k + kc * at.ld, lane, fk);
  load_frags<DH>(at.v + kc * at.ld, lane, fv);
  f32x16_t dk[DH / 32], dv[DH / 32];
  zero(dk);
  zero(dv);
  Rows<DH> qr, dor;
  float sm = 0.0f, si = 0.0f, sd = 0.0f;
  auto fetch = [&](int q0) {
    qr.load(at.q, at.ld, q0, S, tid);
    dor.load(dOg, d, q0, S, tid);
    sm = si = sd = 0.0f;
    if (tid < TS && q0 + tid < S) {
      const long srow = static_cast<long>(blockIdx.y) * S + q0 + tid;
      sm = stats[2 * srow];
      si = stats[2 * srow + 1];
      sd = dots[srow];
    }
  };
  fetch(0);
  for (int q0 = 0; q0 < S; q0 += TS) {
    __syncthreads();
    qr.store(Qs, tid);
    dor.store(Os, tid);
    if (tid < TS) {
      ms[tid] = sm;
      is[tid] = si;
      ds[tid] = sd;
    }
    __syncthreads();
    fetch(q0 + TS);
    if (!live) continue;
    for (int c0 = 0; c0 < TS && q0 + c0 < S; c0 += 32) {
      f32x16_t p = group_product<DH>(fk, Qs, c0, lane);
      f32x16_t dp = group_product<DH>(fv, Os, c0, lane);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = c0 + col_of(4 * g, lane);
        const float4 mv = *reinterpret_cast<const float4*>(ms + c), iv = *reinterpret_cast<const float4*>(is + c),
                     dv4 = *reinterpret_cast<const float4*>(ds + c);
        const float mq[4] = {mv.x, mv.y, mv.z, mv.w}, iq[4] = {iv.x, iv.y, iv.z, iv.w},
                    dq[4] = {dv4.x, dv4.y, dv4.z, dv4.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = 4 * g + q;
          const float x = __fmul_rn(exp_neg(__fsub_rn(__fmul_rn(p[r], scale), mq[q])), iq[q]);
          p[r] = q0 + c + q < S ? x : 0.0f;   // every lane's key below S is stored, the others' rows are not
          dp[r] = p[r] * (dp[r] - dq[q]);
        }
      }
      group_accumulate<DH>(p, Os, c0, lane, dv);
      group_accumulate<DH>(dp, Qs, c0, lane, dk);
    }
  }
  bf16_t* out = dqkv + static_cast<long>(at.b) * S * at.ld + at.h * DH;
  store_rows<DH>(out + d, at.ld, key, S, dk, scale, lane);
  store_rows<DH>(out + 2 * d, at.ld, key, S, dv, 1.0f, lane);
}

// Probabilities of 32 query rows of one (batch, head) for a reader, formed from
// the stored statistics by the operations of the passes above, so they are the
// values those passes use: the float32 P (Pf) or bf16(P) (Pb). Unit u covers
// rows 32 (u % units) .. of head u / units; the output starts at unit u0's.
template <int DH>
__global__ __launch_bounds__(64) void attention_long_probs_kernel(const bf16_t* qkv, const float* stats, int S,
                                                                  int heads, int d, float scale, long u0, float* Pf,
                                                                  bf16_t* Pb) {
  const int lane = threadIdx.x, units = (S + 31) / 32;
  const long u = u0 + blockIdx.x, z = u / units, z0 = u0 / units;
  const int row0 = static_cast<int>(u - z * units) * 32, row = row0 + (lane & 31), rc = min(row, S - 1);
  const long ld = 3L * d, b = z / heads;
  const bf16_t* q = qkv + b * S * ld + (z - b * heads) * DH;
  const bf16_t* k = q + d;
  bf16x8_t fq[DH / 16];
  load_frags<DH>(q + rc * ld, lane, fq);
  const float m = stats[2 * (z * S + rc)], inv = stats[2 * (z * S + rc) + 1];
  const long first = z0 * S + 32L * (u0 - z0 * units);   // row of the output's first
  for (int c0 = 0; c0 < S; c0 += 32) {
    bf16x8_t fk[DH / 16];
    load_frags<DH>(k + min(c0 + (lane & 31), S - 1) * ld, lane, fk);
    f32x16_t p;
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = 0.0f;
#pragma unroll
    for (int e = 0; e < DH / 16; ++e) p = mfma(fk[e], fq[e], p);
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = __fmul_rn(exp_neg(__fsub_rn(__fmul_rn(p[r], scale), m)), inv);
    if (row >= S) continue;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = c0 + col_of(4 * g, lane);   // S is a multiple of 8: the four columns are inside or outside
      if (c >= S) continue;
      const long at = (z * S + row - first) * S + c;
      if (Pf) *reinterpret_cast<float4*>(Pf + at) = make_float4(p[4 * g], p[4 * g + 1], p[4 * g + 2], p[4 * g + 3]);
      else *reinterpret_cast<uint2*>(Pb + at) = make_uint2(pack_bf16x2(p[4 * g], p[4 * g + 1]),
                                                           pack_bf16x2(p[4 * g + 2], p[4 * g + 3]));
    }
  }
}

}  // namespace

// Head dimensions the tiles are compiled for; the grid's second dimension
// holds every (batch, head).
bool attention_long_supported(int batch, int heads, int head_dim) {
  return (head_dim == 32 || head_dim == 64) && static_cast<long>(batch) * heads <= 65535;
}

// Where the tiles are faster than the batched GEMMs with stored probabilities.
// A block walks the whole sequence, so few blocks of a long sequence leave most
// CUs idle for long, while the GEMMs spread the score matrix over the chip.
// Both measured, us of an encoder layer's step, tiles / GEMMs, by blocks of 128
// rows: S = 1024: 64 blocks 363 / 345, 96 349 / 367, 128 354 / 400; S = 2048:
// 16 466 / 327, 32 411 / 310, 80 486 / 457, 96 490 / 504; S = 4096: 32 758 /
// 417, 64 765 / 576, 96 775 / 811; S = 10240: 80 1629 / 1646. Up to S = 768 the
// nine launches are the longer side at any count: S = 640: 10 268 / 308, 40
// 278 / 298; S = 768: 24 290 / 311.
bool attention_long_preferred(int batch, int S, int heads) {
  return S <= 768 || static_cast<long>(batch) * heads * ((S + TS - 1) / TS) >= 88;
}

hipError_t attention_long_fwd(const bf16_t* qkv, int batch, int S, int heads, int d, float scale, float* stats,
                              bf16_t* ctx, hipStream_t s) {
  if (!attention_long_supported(batch, heads, d / heads) || S < 1 || S % 8) return hipErrorInvalidValue;
  const dim3 grid((S + TS - 1) / TS, batch * heads);
  auto* kernel = d / heads == 64 ? attention_long_fwd_kernel<64> : attention_long_fwd_kernel<32>;
  hipLaunchKernelGGL(kernel, grid, dim3(NT), 0, s, qkv, S, heads, d, scale, stats, ctx);
  return hipGetLastError();
}

hipError_t attention_long_probs(const bf16_t* qkv, const float* stats, int batch, int S, int heads, int d, float scale,
                                long u0, long u1, float* Pf, bf16_t* Pb, hipStream_t s) {
  const long units = static_cast<long>(batch) * heads * ((S + 31) / 32);
  if (!attention_long_supported(batch, heads, d / heads) || S < 1 || S % 8 || u0 < 0 || u1 <= u0 || u1 > units ||
      u1 - u0 > 0x7fffffff)
    return hipErrorInvalidValue;
  auto* kernel = d / heads == 64 ? attention_long_probs_kernel<64> : attention_long_probs_kernel<32>;
  hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(u1 - u0)), dim3(64), 0, s, qkv, stats, S, heads, d, scale, u0,
                     Pf, Pb);
  return hipGetLastError();
}

hipError_t attention_long_bwd(const bf16_t* qkv, const bf16_t* dctx, const float* stats, int batch, int S, int heads,
                              int d, float scale, float* dots, bf16_t* dqkv, hipStream_t s) {
  if (!attention_long_supported(batch, heads, d / heads) || S < 1 || S % 8) return hipErrorInvalidValue;
  const dim3 grid((S + TS - 1) / TS, batch * heads);
  const bool wide = d / heads == 64;
  auto* dq = wide ? attention_long_dq_kernel<64> : attention_long_dq_kernel<32>;
  hipLaunchKernelGGL(dq, grid, dim3(NT), 0, s, qkv, dctx, stats, S, heads, d, scale, dots, dqkv);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto* dkv = wide ? attention_long_dkv_kernel<64> : attention_long_dkv_kernel<32>;
  hipLaunchKernelGGL(dkv, grid, dim3(NT), 0, s, qkv, dctx, stats, dots, S, heads, d, scale, dqkv);
  return hipGetLastError();
}

}  // namespace spx
