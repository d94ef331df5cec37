// One step of the draft's semi-autoregressive layer (SpecFLASH Sec. 3.1
// and Algorithm 1: the textual input FC(concat(F_T, E)); Sec. 3.3: one pass
// of one transformer layer gives the K placeholder states; Sec. 4.3: one
// layer of 32 heads):
//   x0 = [F_T, E] W_fc^T + b_fc
//   x1 = x0 + Attn(RoPE(RMSNorm(x0) Wqkv^T)) Wo^T      (cached context)
//   out = x1 + (silu(h Wg^T) * (h Wu^T)) Wdown^T,  h = RMSNorm(x1)
// for the r new rows of each sequence, over the draft's KV cache.
//
// A drafting step has few rows (R = B r <= 128 per pass), so every
// projection streams its weight once and is bound by HBM.  All five are
// built around the weight stream of skinny_stream.hpp: a work-group of eight
// waves, of which up to seven own 32 output columns each over a range of
// 256-channel chunks of the reduction and one copies the input rows (int8
// weights: sixteen waves, up to fourteen of 16 columns).  A
// compute unit streams weights at a bounded rate, so the planner sizes the
// column groups and reduction splits to give every unit the same load; each
// split writes fp32 partial sums, and one epilogue launch per projection
// adds the splits and applies what follows it: bias + norm weight, RoPE +
// cache append, residual + norm weight, SwiGLU (in the gate / up projection
// itself where it needs no split), or the final residual (an RMSNorm's row
// factor commutes with the projection after it, so it is applied to that
// projection's result).  The attention is the
// verification kernel (writing the bf16 input of Wo itself): the new
// rows are a block of r queries, causal inside the block, over the cache.
#include <math.h>

#include <algorithm>

#include "device_common.hpp"
#include "launch.hpp"
#include "skinny_stream.hpp"

namespace sd {
namespace {

// Projection work-groups own up to 224 output columns: seven waves of 32
// (two 16-column blocks), or, for int8 rows, fourteen waves of 16, and one
// more wave that copies the input.  Int8 rows spend vector instructions on
// the conversion, which twice the waves overlap better (few column units
// would leave matrix cores idle: 80 rows, 512 x 1024 13.4 us with waves of 32
// columns, 9.7 us with waves of 16).
// Columns per work-group, splits and order of the sums are the same for
// both, so bf16 and int8 weights of the same values give the same bits.
constexpr int kLinearCols = 32;        // the plan's column unit
constexpr int kLinearMaxUnits = 7;
template <int RB, bool Q8>
struct LinearCfg {
  static constexpr int CB = Q8 ? 1 : 2;        // 16-column blocks per wave
  static constexpr int NW = Q8 ? 16 : 8;       // waves
};
constexpr int kEpiThreads = 256;
typedef floatx4 floatx4_u __attribute__((aligned(4)));   // four floats at any float's alignment

// part[ks][r][n] = sum over split ks's chunks of x[r][k] w[n][k], for the
// rows r0 .. r0 + 16 RB - 1 of this pass.  Q8: the weight holds int8 rows
// with one fp32 scale per row (output column), applied to the accumulators.
// A work-group owns a.cols output columns; waves past them only meet the
// barriers, so the planner can size the groups to fill every compute unit
// evenly.
template <int RB, bool Q8>
__global__ __launch_bounds__((LinearCfg<RB, Q8>::NW * 64)) void linear_partial(LinearArgs a) {
  constexpr int NW = LinearCfg<RB, Q8>::NW, CB = LinearCfg<RB, Q8>::CB;
  __shared__ __align__(16) unsigned char ring[stream_ring_bytes(RB)];
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), G = lane >> 4, c = lane & 15;
  const int n0 = blockIdx.x * a.cols + w * 16 * CB;
  const int ks = blockIdx.y;
  const int r0 = blockIdx.z * RB * 16;
  const int K = a.K, N = a.N, R = a.R;
  const int nch = K / kStreamChunk;
  const int ch0 = (int)((unsigned)nch * (unsigned)ks / (unsigned)a.ksplit);   // nch < 2^18, ksplit <= 16
  const int ch1 = (int)((unsigned)nch * (unsigned)(ks + 1) / (unsigned)a.ksplit);
  // Work-groups in step would read the same channels of every row, rows a
  // multiple of a kilobyte apart, which keeps few channels of their XCD's L2
  // busy.  With up to four splits, consecutive work-groups of one XCD (every
  // eighth) start at consecutive chunks (6 rows: 57344 x 8192, one split,
  // 179.6 -> 162 us; 8192 x 8192, four, 31.5 -> 25.4 us).  More splits spread
  // the starts by themselves, and share the input chunks in L2 better in
  // step (112 rows, 4096 x 14336, eight splits: 33.0 us, rotated 34.8 us).
  const int rot = a.ksplit <= 4 && ch0 < ch1 ? (int)((blockIdx.x >> 3) % (unsigned)(ch1 - ch0)) : 0;
  const bool active = w < NW - 1 && w * 16 * CB < a.cols;   // wave-uniform
  floatx4 acc[CB][RB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[cb][rb] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (ch0 < ch1) {
    const size_t row_bytes = (size_t)K * (Q8 ? 1 : 2);
    int valid[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) valid[cb] = N - n0 - 16 * cb;
    stream_product<RB, CB, NW, Q8>(static_cast<const unsigned char*>(a.w) + n0 * row_bytes, 16 * row_bytes, valid,
                                   active, static_cast<const uint16_t*>(a.x) + (size_t)r0 * K, min(R - r0, RB * 16),
                                   K, ch0, ch1, rot, ring, acc);
  }
  if (!active) return;
  // accumulator element i of lane (c, G): input row rb*16 + c, column n0 +
  // 16 cb + 4G + i
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int n = n0 + 16 * cb + 4 * G;
    if constexpr (Q8) {
      floatx4 sc;
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[i] = a.wscale[min(n + i, N - 1)];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[cb][rb] *= sc;
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = r0 + rb * 16 + c;
      if (r >= R || n >= N) continue;
      float* dst = a.part + ((size_t)ks * R + r) * N + n;
      if (n + 3 < N && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
        *reinterpret_cast<floatx4*>(dst) = acc[cb][rb];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < N) dst[i] = acc[cb][rb][i];
      }
    }
  }
}

__device__ __forceinline__ float split_sum(const float* part, int ksplit, size_t stride, size_t idx) {
  float s = 0.f;
  for (int ks = 0; ks < ksplit; ++ks) s += part[(size_t)ks * stride + idx];
  return s;
}

// The same for four consecutive values at a 16-byte aligned index, added in
// the same order: every split's load is issued before the first is used
// (one after the other they cost a memory latency each).
template <int M>
__device__ __forceinline__ void split_sum4(const float* part, int ksplit, size_t stride, const size_t (&idx)[M],
                                           floatx4 (&s)[M]) {
  floatx4 v[M][kLinearMaxSplits];
#pragma unroll
  for (int ks = 0; ks < kLinearMaxSplits; ++ks)
    if (ks < ksplit) {
#pragma unroll
      for (int i = 0; i < M; ++i) v[i][ks] = *reinterpret_cast<const floatx4*>(part + ks * stride + idx[i]);
    }
#pragma unroll
  for (int i = 0; i < M; ++i) s[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < kLinearMaxSplits; ++ks)
    if (ks < ksplit) {
#pragma unroll
      for (int i = 0; i < M; ++i) s[i] += v[i][ks];
    }
}

__device__ __forceinline__ void store_bf16x4(__bf16* dst, const floatx4& v) {
  Pack8 pk;
#pragma unroll
  for (int e = 0; e < 4; ++e) pk.b[e] = float_to_bf16(v[e]);
  *reinterpret_cast<u32x2*>(dst) = u32x2{pk.u[0], pk.u[1]};
}

__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  return t;
}

// y = sum of splits (+ bias) (+ residual), written as fp32 `out` [R, N];
// grid (ceil(N / kEpiCols), R), kEpiThreads threads of four columns each.
// Every split of a thread's columns is loaded before any is added (the
// splits are added in split order), so a row's partials stream from many
// compute units at once.  With `h`, it also prepares the next projection's
// input under an RMSNorm: h = bf16(y * norm_w), and block x of row r writes
// the sum of squares of its columns to ss[r * gridDim.x + x].  The factor
// 1 / sqrt(mean(y^2) + eps), one per row, commutes with the projection, whose
// epilogue applies it (row_scale); a launch of its own for it took 3.8 us (6
// rows) to 4.8 us (112 rows) in the layer, twice.
// The factor is 0 where the mean square overflows.  A value whose square
// overflows enters h as 0 y, as the factor would make it: 0 if it is finite,
// so that no product of the row overflows (and 0 times it stays 0), NaN if it
// is infinite, so that every normalised value of its row is NaN.
constexpr int kEpiCols = 4 * kEpiThreads;
__device__ __forceinline__ float norm_input(float y) { return y * y == INFINITY ? 0.f * y : y; }
__global__ __launch_bounds__(kEpiThreads) void epi_add_cols(const float* part, int ksplit, int R, int N,
                                                            const float* bias, const float* residual,
                                                            float* out, const float* norm_w, __bf16* h,
                                                            float* ss) {
  __shared__ float red[kEpiThreads / 64];
  const int r = blockIdx.y;
  const size_t stride = (size_t)R * N;
  const size_t row = (size_t)r * N;
  const int n0 = blockIdx.x * kEpiCols + threadIdx.x * 4;
  auto a16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const bool vec = (N & 3) == 0 && a16(part) && a16(out) && (!bias || a16(bias)) && (!residual || a16(residual));
  float s2 = 0.f;
  if (vec) {
    if (n0 < N) {
      floatx4 v[kLinearMaxSplits];
#pragma unroll
      for (int ks = 0; ks < kLinearMaxSplits; ++ks)
        if (ks < ksplit) v[ks] = *reinterpret_cast<const floatx4*>(part + ks * stride + row + n0);
      floatx4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < kLinearMaxSplits; ++ks)
        if (ks < ksplit) y += v[ks];
      if (bias) y += *reinterpret_cast<const floatx4*>(bias + n0);
      if (residual) y += *reinterpret_cast<const floatx4*>(residual + row + n0);
      *reinterpret_cast<floatx4*>(out + row + n0) = y;
      if (h != nullptr) {
        Pack8 pk;
#pragma unroll
        for (int j = 0; j < 4; ++j) pk.b[j] = float_to_bf16(norm_input(y[j]) * norm_w[n0 + j]);
        *reinterpret_cast<u32x2*>(h + row + n0) = u32x2{pk.u[0], pk.u[1]};
      }
      s2 = y[0] * y[0] + y[1] * y[1] + y[2] * y[2] + y[3] * y[3];
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + j;
      if (n >= N) break;
      float y = split_sum(part, ksplit, stride, row + n);
      if (bias) y += bias[n];
      if (residual) y += residual[row + n];
      out[row + n] = y;
      if (h != nullptr) h[row + n] = float_to_bf16(norm_input(y) * norm_w[n]);
      s2 += y * y;
    }
  }
  if (h == nullptr) return;
  const float t = block_sum(s2, red);
  if (threadIdx.x == 0) ss[(size_t)r * gridDim.x + blockIdx.x] = t;
}

// 1 / sqrt(mean(y^2) + eps) of row r of width d from epi_add_cols' nblk block
// sums (added in block order, eight loads in flight).
__device__ __forceinline__ float row_scale(const float* ss, int nblk, int r, int d, float eps) {
  float t = 0.f;
  for (int i0 = 0; i0 < nblk; i0 += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = i0 + i < nblk ? ss[(size_t)r * nblk + i0 + i] : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) t += v[i];
  }
  return 1.f / sqrtf(t / (float)d + eps);
}
static int epi_blocks(int N) { return (N + kEpiCols - 1) / kEpiCols; }

// Fused projection output of row r (sequence b = r / rows, j = r % rows,
// position p = pos[b] + j): query heads rotated into q [R, Hq, D] (bf16),
// key heads rotated and value heads copied into the caches at position p
// (skipped when p is outside 0 .. Lmax - 1).  Half-split pairs (i, i + D/2)
// turn by p theta^(-2i/D): the frequencies are formed once per work-group
// in float64, the angle p f in float64 is reduced to [-pi, pi] in float64,
// and only the sine and cosine of the reduced angle are taken in float32
// (an error of a few float32 ulp at any position).  Row 0 of each sequence
// also writes kv_len[b] = pos[b] + rows for the attention.
__global__ __launch_bounds__(kEpiThreads) void epi_rope_qkv(const float* part, int ksplit, int R, int N,
                                                            const int32_t* pos, int rows, int Hq, int Hkv,
                                                            int D, double log_theta, int Lmax, __bf16* q,
                                                            __bf16* kc, __bf16* vc, int32_t* kv_len,
                                                            const float* ss, int nblk, int d, float eps) {
  __shared__ float2 rot[64];                   // (cos, sin) of each pair's angle
  const int r = blockIdx.y;
  const int b = r / rows, j = r - b * rows;
  const int p = pos[b] + j;
  const bool store = p >= 0 && p < Lmax;
  if (j == 0 && blockIdx.x == 0 && threadIdx.x == 0) kv_len[b] = pos[b] + rows;
  const float inv = row_scale(ss, nblk, r, d, eps);
  const size_t stride = (size_t)R * N;
  const int half = D / 2;
  if (threadIdx.x < half) {
    const double f = exp(-2.0 * (double)threadIdx.x / (double)D * log_theta);
    const double ang = (double)p * f;
    const double twopi = 6.283185307179586476925286766559;
    const float red = (float)(ang - twopi * rint(ang / twopi));
    float sn, cs;
    sincosf(red, &sn, &cs);
    rot[threadIdx.x] = make_float2(cs, sn);
  }
  __syncthreads();
  // thread t of the row: pairs 4 t .. 4 t + 3 (query and key heads), then
  // four value elements (D is a multiple of 64, so both stay in one head)
  const int quads = (Hq + Hkv) * half / 4;
  const int t = blockIdx.x * kEpiThreads + threadIdx.x;
  if (t < quads) {
    const int hh = t * 4 / half, i = t * 4 - hh * half;
    const size_t base = (size_t)r * N + (size_t)hh * D + i;
    const size_t idx[2] = {base, base + half};
    floatx4 x[2];
    split_sum4(part, ksplit, stride, idx, x);
    const floatx4 x0 = x[0] * inv, x1 = x[1] * inv;
    floatx4 y0, y1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float cs = rot[i + e].x, sn = rot[i + e].y;
      y0[e] = x0[e] * cs - x1[e] * sn;
      y1[e] = x1[e] * cs + x0[e] * sn;
    }
    if (hh < Hq) {
      __bf16* dst = q + ((size_t)r * Hq + hh) * D + i;
      store_bf16x4(dst, y0);
      store_bf16x4(dst + half, y1);
    } else if (store) {
      __bf16* dst = kc + (((size_t)b * Lmax + p) * Hkv + (hh - Hq)) * D + i;
      store_bf16x4(dst, y0);
      store_bf16x4(dst + half, y1);
    }
  } else if (store && t < quads + Hkv * D / 4) {
    const int e4 = (t - quads) * 4;               // element of the row's value heads
    const size_t idx[1] = {(size_t)r * N + (size_t)(Hq + Hkv) * D + e4};
    floatx4 v[1];
    split_sum4(part, ksplit, stride, idx, v);
    store_bf16x4(vc + ((size_t)b * Lmax + p) * Hkv * D + e4, v[0] * inv);
  }
}

// act[r][i] = silu(g) * u with g, u the split sums of columns i and I + i
// times the row's norm factor
__global__ __launch_bounds__(kEpiThreads) void epi_swiglu(const float* part, int ksplit, int R, int I,
                                                          __bf16* act, const float* ss, int nblk, int d, float eps) {
  const int r = blockIdx.y;
  const int i = (blockIdx.x * kEpiThreads + threadIdx.x) * 4;   // I is a multiple of 256
  if (i >= I) return;
  const size_t N = 2 * (size_t)I;
  const size_t idx[2] = {(size_t)r * N + i, (size_t)r * N + I + i};
  floatx4 x[2], y;
  split_sum4(part, ksplit, (size_t)R * N, idx, x);
  const float inv = row_scale(ss, nblk, r, d, eps);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float g = x[0][e] * inv, u = x[1][e] * inv;
    y[e] = g / (1.f + expf(-g)) * u;
  }
  store_bf16x4(act + (size_t)r * I + i, y);
}

// The gate / up projection with SwiGLU as its epilogue, for the whole
// reduction in one split: act[r][i] = silu(g) * u, bf16, g and u the products
// with weight rows i and I + i times the row's norm factor.  A unit is 16
// gate rows and their 16 up rows: the two blocks of a wave, or two waves
// that meet through LDS (the waves of int8 rows, see LinearCfg).  The same
// products as linear_partial's, without the partials' way through memory and
// the second launch, but summed from another chunk on (the start follows the
// work-group's index, and a column lies in another one) and never in splits,
// so the float32 sums may round differently.  Bf16 and int8 weights of the
// same values share the order and give the same bits.
struct SwigluArgs {
  __bf16* act;
  const float* ss;
  int nblk, d, I, units;   // units per work-group
  float eps;
};
template <int RB, bool Q8>
__global__ __launch_bounds__((LinearCfg<RB, Q8>::NW * 64)) void linear_swiglu(LinearArgs a, SwigluArgs g) {
  constexpr int NW = LinearCfg<RB, Q8>::NW, CB = LinearCfg<RB, Q8>::CB;
  __shared__ __align__(16) unsigned char ring[stream_ring_bytes(RB)];
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), G = lane >> 4, c = lane & 15;
  const int unit = CB == 2 ? w : w >> 1, up = CB == 2 ? 0 : w & 1;
  const int p0 = (blockIdx.x * g.units + unit) * 16;
  const int r0 = blockIdx.z * RB * 16;
  const int K = a.K, I = g.I, R = a.R;
  const int nch = K / kStreamChunk;
  const int rot = (int)((blockIdx.x >> 3) % (unsigned)nch);
  const bool active = w < NW - 1 && unit < g.units && p0 < I;   // wave-uniform
  floatx4 acc[CB][RB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[cb][rb] = floatx4{0.f, 0.f, 0.f, 0.f};
  const size_t row_bytes = (size_t)K * (Q8 ? 1 : 2);
  int valid[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) valid[cb] = I - p0;
  stream_product<RB, CB, NW, Q8>(static_cast<const unsigned char*>(a.w) + (p0 + (size_t)up * I) * row_bytes,
                                 I * row_bytes, valid, active, static_cast<const uint16_t*>(a.x) + (size_t)r0 * K,
                                 min(R - r0, RB * 16), K, 0, nch, rot, ring, acc);
  const int n = p0 + 4 * G;
  if constexpr (Q8) {
    if (active) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const floatx4 sc = *reinterpret_cast<const floatx4_u*>(a.wscale + (size_t)(up + cb) * I + n);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[cb][rb] *= sc;
      }
    }
  }
  floatx4 uv[RB];
  if constexpr (CB == 2) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) uv[rb] = acc[1][rb];
  } else {
    // every wave is done with the ring: the up products go through it
    floatx4* xu = reinterpret_cast<floatx4*>(ring);
    static_assert(kLinearMaxUnits * RB * 1024 <= stream_ring_bytes(RB), "up products fit the ring");
    __syncthreads();
    if (active && up) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) xu[(unit * RB + rb) * 64 + lane] = acc[0][rb];
    }
    __syncthreads();
    if (active && !up) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) uv[rb] = xu[(unit * RB + rb) * 64 + lane];
    }
  }
  if (!active || up) return;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = r0 + rb * 16 + c;
    if (r >= R) continue;
    const float inv = row_scale(g.ss, g.nblk, r, g.d, g.eps);
    floatx4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gv = acc[0][rb][e] * inv, u = uv[rb][e] * inv;
      y[e] = gv / (1.f + expf(-gv)) * u;
    }
    store_bf16x4(g.act + (size_t)r * I + n, y);
  }
}

// ------------------------------------------------- K drafts in K / k' passes
// Before the head: the k' placeholder rows of a pass's output (rows
// r - k' .. r - 1 of each sequence) rounded to bf16 as the LM head's input
// rows (b, j), and this pass's uniforms u[b][t k' + j] gathered.
__global__ __launch_bounds__(kEpiThreads) void kp_prep(const float* out, int r, int kp, int d, const float* u,
                                                       int K, int t, __bf16* hid, float* ut) {
  const int row = blockIdx.x;
  const int b = row / kp, j = row - b * kp;
  const float* src = out + ((size_t)b * r + (r - kp + j)) * d;
  for (int e = threadIdx.x; e < d; e += kEpiThreads) hid[(size_t)row * d + e] = float_to_bf16(src[e]);
  if (threadIdx.x == 0) ut[row] = u[(size_t)b * K + (size_t)t * kp + j];
}

// After the draw: row (b, j)'s token and distribution to the outputs at
// draft t k' + j; with another pass to come, the next pass's rows of
// sequence b (the drafted token, concat(bf16(F'), E[token]), then a
// placeholder row) and its positions pos_out[b] = pos_in[b] + advance.
// Token ids outside the vocabulary read the nearest embedding row.
__global__ __launch_bounds__(kEpiThreads) void kp_post(const float* probs, const int32_t* tok, int kp, int K,
                                                       int t, int V, int d, const __bf16* hid, const __bf16* emb,
                                                       const __bf16* ph, int32_t* tokens, float* q, __bf16* unext,
                                                       const int32_t* pos_in, int advance, int32_t* pos_out,
                                                       int more) {
  const int row = blockIdx.x;
  const int b = row / kp, j = row - b * kp;
  const int token = tok[row];
  const size_t dst = (size_t)b * K + (size_t)t * kp + j;
  if (threadIdx.x == 0) tokens[dst] = token;
  const float* src = probs + (size_t)row * V;
  float* qd = q + dst * V;
  for (int v = threadIdx.x; v < V; v += kEpiThreads) qd[v] = src[v];
  if (!more) return;
  const int tk = min(max(token, 0), V - 1);
  __bf16* text = unext + ((size_t)b * 2 * kp + j) * 2 * d;
  __bf16* place = unext + ((size_t)b * 2 * kp + kp + j) * 2 * d;
  for (int e = threadIdx.x; e < d; e += kEpiThreads) {
    text[e] = hid[(size_t)row * d + e];
    text[d + e] = emb[(size_t)tk * d + e];
  }
  for (int e = threadIdx.x; e < 2 * d; e += kEpiThreads) place[e] = ph[e];
  if (j == 0 && threadIdx.x == 0) pos_out[b] = pos_in[b] + advance;
}

template <int RB, bool Q8>
hipError_t launch_partial_rb(const LinearArgs& a, int passes, hipStream_t st) {
  hipLaunchKernelGGL((linear_partial<RB, Q8>), dim3((a.N + a.cols - 1) / a.cols, a.ksplit, passes),
                     dim3(LinearCfg<RB, Q8>::NW * 64), 0, st, a);
  return hipGetLastError();
}

template <int RB, bool Q8>
hipError_t launch_swiglu_rb(const LinearArgs& a, const SwigluArgs& g, int passes, hipStream_t st) {
  hipLaunchKernelGGL((linear_swiglu<RB, Q8>), dim3((g.I / 16 + g.units - 1) / g.units, 1, passes),
                     dim3(LinearCfg<RB, Q8>::NW * 64), 0, st, a, g);
  return hipGetLastError();
}

template <bool Q8>
hipError_t launch_swiglu(const LinearArgs& a, const SwigluArgs& g, int rb, int passes, hipStream_t st) {
  switch (rb) {
    case 1: return launch_swiglu_rb<1, Q8>(a, g, passes, st);
    case 2: return launch_swiglu_rb<2, Q8>(a, g, passes, st);
    case 3: return launch_swiglu_rb<3, Q8>(a, g, passes, st);
    case 4: return launch_swiglu_rb<4, Q8>(a, g, passes, st);
    case 5: return launch_swiglu_rb<5, Q8>(a, g, passes, st);
    case 6: return launch_swiglu_rb<6, Q8>(a, g, passes, st);
    case 7: return launch_swiglu_rb<7, Q8>(a, g, passes, st);
    default: return launch_swiglu_rb<8, Q8>(a, g, passes, st);
  }
}

template <bool Q8>
hipError_t launch_partial(const LinearArgs& a, int rb, int passes, hipStream_t st) {
  switch (rb) {
    case 1: return launch_partial_rb<1, Q8>(a, passes, st);
    case 2: return launch_partial_rb<2, Q8>(a, passes, st);
    case 3: return launch_partial_rb<3, Q8>(a, passes, st);
    case 4: return launch_partial_rb<4, Q8>(a, passes, st);
    case 5: return launch_partial_rb<5, Q8>(a, passes, st);
    case 6: return launch_partial_rb<6, Q8>(a, passes, st);
    case 7: return launch_partial_rb<7, Q8>(a, passes, st);
    default: return launch_partial_rb<8, Q8>(a, passes, st);
  }
}

}  // namespace

LinearPlan plan_linear(int R, int K, int N, int cus) {
  LinearPlan p{};
  const int pass_rows = 16 * std::max(1, stream_row_blocks(K));   // the caller refuses a K without a row block
  const int rows = std::min(R, pass_rows);
  p.row_blocks = (rows + 15) / 16;
  p.passes = (R + pass_rows - 1) / pass_rows;
  constexpr int wide = kLinearCols;
  // one work-group per compute unit: its registers hold no second one
  const long long cap = std::max(cus, 1);
  const int nch = K / kStreamChunk;
  const long long ncu = std::max(cus, 1);
  // A compute unit streams its weight rows at a bounded rate, so the time
  // follows the most loaded unit: (work-groups it runs) x (chunks per
  // work-group) x (bytes per chunk: its weight rows, and the input rows,
  // which come from L2 and cost about half as much each).  For 2..7 column
  // units, split the reduction to fill the device in one round (at least
  // four chunks per split) and keep the count with the least such load; ties
  // go to more units (more weight loads in flight).  One unit fewer than
  // possible fills every compute unit evenly where wider groups would leave
  // some with one group less than others.
  long long best = -1;
  for (int nwa = kLinearMaxUnits; nwa >= 2; --nwa) {
    const long long g = (long long)((N + nwa * wide - 1) / (nwa * wide)) * p.passes;
    long long ks = std::max(1LL, cap / g);
    ks = std::min<long long>(ks, std::max(1, nch / 4));
    ks = std::max(1LL, std::min<long long>(ks, kLinearMaxSplits));
    const long long per_cu = (g * ks + ncu - 1) / ncu;
    const long long load = per_cu * ((nch + ks - 1) / ks) * (2 * nwa * wide + p.row_blocks * 16);
    if (best < 0 || load < best) {
      best = load;
      p.cols = nwa * wide;
      p.ksplit = (int)ks;
    }
  }
  p.load = best;
  p.part_bytes = (size_t)p.ksplit * R * N * sizeof(float);
  return p;
}

hipError_t launch_linear_partial(const LinearArgs& args, const LinearPlan& p, hipStream_t st) {
  LinearArgs a = args;
  a.cols = p.cols;
  if (a.wscale != nullptr) return launch_partial<true>(a, p.row_blocks, p.passes, st);
  return launch_partial<false>(a, p.row_blocks, p.passes, st);
}

hipError_t launch_epi_add(const float* part, int ksplit, int R, int N, const float* bias, const float* residual,
                          float* out, hipStream_t st) {
  hipLaunchKernelGGL(epi_add_cols, dim3(epi_blocks(N), R), dim3(kEpiThreads), 0, st, part, ksplit, R, N, bias,
                     residual, out, (const float*)nullptr, (__bf16*)nullptr, (float*)nullptr);
  return hipGetLastError();
}

// ------------------------------------------------------- the whole layer
static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

SemiArPlan plan_semi_ar(int B, int r, int d, int Hq, int Hkv, int I, int Lmax, int cus) {
  SemiArPlan p{};
  const int R = B * r, D = d / Hq;
  const int nqkv = (Hq + 2 * Hkv) * D;
  p.fc = plan_linear(R, 2 * d, d, cus);
  p.qkv = plan_linear(R, d, nqkv, cus);
  p.o = plan_linear(R, Hq * D, d, cus);
  p.gu = plan_linear(R, d, 2 * I, cus);
  p.down = plan_linear(R, I, d, cus);
  // The gate / up projection in one split with SwiGLU as its epilogue, when
  // the most loaded compute unit then streams at most 8% more than in the
  // plan above (plan_linear's load; units of 16 gate and 16 up rows).  Fused
  // against unfused: one sequence of 6 rows with its head (d = 4096, I =
  // 11008) 166.4 against 170.2 us, a layer of 4 sequences at d = 8192, I =
  // 28672 391 against 396 us (bf16) and within 0.4% of each other (int8; 8
  // sequences of 9 rows 292 against 299).  Where
  // the load would grow by a third (16 sequences, d = 4096, I = 14336) it
  // gains nothing: 182.8 against 182.9 us.
  const long long ncu = std::max(cus, 1);
  long long best = -1;
  for (int u = kLinearMaxUnits; u >= 1; --u) {
    const long long g = (long long)((I / 16 + u - 1) / u) * p.gu.passes;
    const long long load = (g + ncu - 1) / ncu * (d / kStreamChunk) * (2 * u * kLinearCols + p.gu.row_blocks * 16);
    if (best < 0 || load < best) {
      best = load;
      p.gu_units = u;
    }
  }
  if (best * 100 > p.gu.load * 108) p.gu_units = 0;
  p.verify = plan_verify(B, r, Hq, Hkv, D, Lmax, 1, cus);
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += align256(bytes); return o; };
  const size_t part = std::max({p.fc.part_bytes, p.qkv.part_bytes, p.o.part_bytes, p.gu.part_bytes,
                                p.down.part_bytes});
  p.off_part = take(part);
  p.off_x0 = take((size_t)R * d * 4);
  p.off_h = take((size_t)R * d * 2);
  p.off_q = take((size_t)R * Hq * D * 2);
  p.off_attn16 = take((size_t)R * Hq * D * 2);
  p.off_x1 = take((size_t)R * d * 4);
  p.off_act = take((size_t)R * I * 2);
  p.off_kvlen = take((size_t)B * 4);
  p.off_ss = take((size_t)R * epi_blocks(d) * 4);
  p.off_verify = take(p.verify.workspace_bytes);
  p.workspace_bytes = off;
  p.ok = p.verify.ok;
  return p;
}

hipError_t launch_semi_ar(const SemiArArgs& a, const SemiArPlan& p, hipStream_t st) {
  unsigned char* ws = static_cast<unsigned char*>(a.workspace);
  float* part = reinterpret_cast<float*>(ws + p.off_part);
  float* x0 = reinterpret_cast<float*>(ws + p.off_x0);
  __bf16* h = reinterpret_cast<__bf16*>(ws + p.off_h);
  __bf16* q = reinterpret_cast<__bf16*>(ws + p.off_q);
  __bf16* attn16 = reinterpret_cast<__bf16*>(ws + p.off_attn16);
  float* x1 = reinterpret_cast<float*>(ws + p.off_x1);
  __bf16* act = reinterpret_cast<__bf16*>(ws + p.off_act);
  int32_t* kv_len = reinterpret_cast<int32_t*>(ws + p.off_kvlen);
  float* ss = reinterpret_cast<float*>(ws + p.off_ss);
  const int R = a.B * a.r, d = a.d, D = d / a.Hq;
  const dim3 eg(epi_blocks(d), R);
  const int nqkv = (a.Hq + 2 * a.Hkv) * D;
  hipError_t e;
  auto lin = [&](const void* x, const void* w, const float* scale, int K, int N, const LinearPlan& lp) {
    LinearArgs la{x, w, part, R, K, N, lp.ksplit, scale};
    return launch_linear_partial(la, lp, st);
  };
  // x0 = FC(u), h = x0 ln1 (the norm's row factors follow the projection)
  if ((e = lin(a.u, a.fc_w, a.fc_s, 2 * d, d, p.fc)) != hipSuccess) return e;
  hipLaunchKernelGGL(epi_add_cols, eg, dim3(kEpiThreads), 0, st, part, p.fc.ksplit, R, d, a.fc_b,
                     (const float*)nullptr, x0, a.ln1, h, ss);
  // q, k, v with RoPE; k, v appended to the cache
  if ((e = lin(h, a.wqkv, a.wqkv_s, d, nqkv, p.qkv)) != hipSuccess) return e;
  const int rope_threads = ((a.Hq + a.Hkv) * (D / 2) + a.Hkv * D) / 4;
  hipLaunchKernelGGL(epi_rope_qkv, dim3((rope_threads + kEpiThreads - 1) / kEpiThreads, R), dim3(kEpiThreads), 0, st, part, p.qkv.ksplit, R, nqkv, a.pos, a.r,
                     a.Hq, a.Hkv, D, log((double)a.theta), a.Lmax, q,
                     static_cast<__bf16*>(a.k_cache), static_cast<__bf16*>(a.v_cache), kv_len, ss, (int)eg.x, d, a.eps);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // attention of the r new rows over the cache, causal inside them
  VerifyArgs va{};
  va.q = q;
  va.kc = a.k_cache;
  va.vc = a.v_cache;
  va.kv_len = kv_len;
  va.page_table = nullptr;
  va.Lmax = a.Lmax;
  va.out = nullptr;
  va.out_bf16 = attn16;                        // the merge writes the bf16 input of Wo
  va.lse = nullptr;
  va.B = a.B;
  va.k = a.r;
  va.Hq = a.Hq;
  va.Hkv = a.Hkv;
  va.D = D;
  va.scale = 1.f / sqrtf((float)D);
  va.scale_log2 = va.scale * kLog2e;
  va.part_o = reinterpret_cast<float*>(ws + p.off_verify);
  va.part_lse = va.part_o + p.verify.part_rows * D;
  if ((e = launch_verify(va, p.verify, 1, st)) != hipSuccess) return e;
  // x1 = x0 + attn Wo^T, h = x1 ln2
  if ((e = lin(attn16, a.wo, a.wo_s, a.Hq * D, d, p.o)) != hipSuccess) return e;
  hipLaunchKernelGGL(epi_add_cols, eg, dim3(kEpiThreads), 0, st, part, p.o.ksplit, R, d,
                     (const float*)nullptr, x0, x1, a.ln2, h, ss);
  // act = SwiGLU(h), out = x1 + act Wdown^T
  if (p.gu_units > 0) {
    LinearArgs la{h, a.wgu, nullptr, R, d, 2 * a.I, 1, a.wgu_s};
    const SwigluArgs sg{act, ss, (int)eg.x, d, a.I, p.gu_units, a.eps};
    e = a.wgu_s != nullptr ? launch_swiglu<true>(la, sg, p.gu.row_blocks, p.gu.passes, st)
                           : launch_swiglu<false>(la, sg, p.gu.row_blocks, p.gu.passes, st);
    if (e != hipSuccess) return e;
  } else {
    if ((e = lin(h, a.wgu, a.wgu_s, d, 2 * a.I, p.gu)) != hipSuccess) return e;
    hipLaunchKernelGGL(epi_swiglu, dim3((a.I / 4 + kEpiThreads - 1) / kEpiThreads, R), dim3(kEpiThreads), 0, st, part,
                       p.gu.ksplit, R, a.I, act, ss, (int)eg.x, d, a.eps);
  }
  if ((e = lin(act, a.wdown, a.wdown_s, a.I, d, p.down)) != hipSuccess) return e;
  return launch_epi_add(part, p.down.ksplit, R, d, nullptr, x1, a.out, st);
}

}  // namespace sd

namespace sd {

SemiArDraftPlan plan_semi_ar_draft(int B, int r0, int d, int Hq, int Hkv, int I, int Lmax, int V, int K, int kp,
                                   int cus) {
  SemiArDraftPlan p{};
  p.first = plan_semi_ar(B, r0, d, Hq, Hkv, I, Lmax, cus);
  p.later = K > kp ? plan_semi_ar(B, 2 * kp, d, Hq, Hkv, I, Lmax, cus) : p.first;
  const int rmax = std::max(r0, 2 * kp), R = B * kp;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += align256(bytes); return o; };
  p.off_layer = take(std::max(p.first.workspace_bytes, p.later.workspace_bytes));
  p.off_out = take((size_t)B * rmax * d * 4);
  p.off_unext = take((size_t)B * 2 * kp * 2 * d * 2);
  p.off_hid = take((size_t)R * d * 2);
  p.off_probs = take((size_t)R * V * 4);
  p.off_lmstats = take(lm_head_workspace_bytes(R, V));
  p.off_sample = take(accept_workspace_bytes(R, 0, V, 1));
  p.off_nacc = take((size_t)R * 4);
  p.off_ut = take((size_t)R * 4);
  p.off_tok = take((size_t)R * 4);
  p.off_pos = take((size_t)2 * B * 4);
  p.workspace_bytes = off;
  p.cus = cus;
  p.ok = p.first.ok && p.later.ok;
  return p;
}

hipError_t launch_semi_ar_draft(const SemiArDraftArgs& a, const SemiArDraftPlan& p, hipStream_t st) {
  unsigned char* ws = static_cast<unsigned char*>(a.workspace);
  float* out = reinterpret_cast<float*>(ws + p.off_out);
  __bf16* unext = reinterpret_cast<__bf16*>(ws + p.off_unext);
  __bf16* hid = reinterpret_cast<__bf16*>(ws + p.off_hid);
  float* probs = reinterpret_cast<float*>(ws + p.off_probs);
  float* ut = reinterpret_cast<float*>(ws + p.off_ut);
  int32_t* tok = reinterpret_cast<int32_t*>(ws + p.off_tok);
  int32_t* posbuf = reinterpret_cast<int32_t*>(ws + p.off_pos);
  const int B = a.layer.B, d = a.layer.d, kp = a.kp, R = B * kp;
  const int passes = a.K / kp;
  hipError_t e;
  for (int t = 0; t < passes; ++t) {
    SemiArArgs la = a.layer;
    la.r = t == 0 ? a.layer.r : 2 * kp;
    la.u = t == 0 ? a.layer.u : unext;
    la.pos = t == 0 ? a.layer.pos : posbuf + (t & 1) * B;
    la.out = out;
    la.workspace = ws + p.off_layer;
    if ((e = launch_semi_ar(la, t == 0 ? p.first : p.later, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(kp_prep, dim3(R), dim3(kEpiThreads), 0, st, out, la.r, kp, d, a.u, a.K, t, hid, ut);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    LmHeadArgs lh{};
    lh.hidden = hid;
    lh.weight = a.lm_w;
    lh.probs = probs;
    lh.R = R;
    lh.d = d;
    lh.V = a.V;
    lh.scale_log2 = kLog2e / a.temperature;
    lh.stats = reinterpret_cast<float*>(ws + p.off_lmstats);
    lh.cus = p.cus;
    if ((e = launch_lm_head(lh, 1, st)) != hipSuccess) return e;
    AcceptArgs sa{};
    sa.p = probs;
    sa.u = ut;
    sa.n_accepted = reinterpret_cast<int32_t*>(ws + p.off_nacc);
    sa.tokens = tok;
    sa.B = R;
    sa.k = 0;
    sa.V = a.V;
    sa.mode = 1;
    if ((e = launch_accept(sa, ws + p.off_sample, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(kp_post, dim3(R), dim3(kEpiThreads), 0, st, probs, tok, kp, a.K, t, a.V, d, hid,
                       static_cast<const __bf16*>(a.emb), static_cast<const __bf16*>(a.ph), a.tokens, a.q, unext,
                       la.pos, la.r - kp, posbuf + ((t + 1) & 1) * B, (int)(t + 1 < passes));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sd
