// The weight stream shared by the skinny products (few input rows against
// every row of a large weight): z^T = W x^T on bf16 matrix cores, the
// weight read once from HBM straight into registers, the input rows staged
// through LDS.
#pragma once

#include <type_traits>

#include "device_common.hpp"

namespace sd {

typedef __attribute__((address_space(3))) void stream_lds_void;

constexpr int kStreamStep = 128;    // reduction channels per step
constexpr int kStreamChunk = 256;   // granularity of a range of the reduction
constexpr int stream_slot_bytes(int rb) { return rb * 16 * kStreamStep * 2; }
constexpr int stream_ring_bytes(int rb) { return 4 * stream_slot_bytes(rb); }

// Two int8 values (bytes k, k + 1 of v) as two bf16 values, exactly (every
// int8 value has at most 8 significant bits): sign-extend, convert to
// float32, keep the upper halves.
__device__ __forceinline__ uint32_t i8x2_to_bf16x2(uint32_t v, int k) {
  const float f0 = (float)(int)(int8_t)(v >> (8 * k));
  const float f1 = (float)(int)(int8_t)(v >> (8 * k + 8));
  return __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
}

// A buffer resource over [p, p + bytes) held in scalar registers (both
// arguments are wave-uniform; the compiler cannot always see it).
__device__ __forceinline__ auto stream_rsrc(const void* p, uint32_t bytes) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uintptr_t)hi << 32) | lo), (short)0,
                                           __builtin_amdgcn_readfirstlane((int)bytes), 0x00027000);
}

template <int B, int E, typename F>
__device__ __forceinline__ void stream_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    stream_for<B + 1, E>(f);
  }
}

// acc[cb][rb] += W rows x input rows over the 256-channel chunks ch0 ..
// ch1 - 1 (ch0 < ch1), by a work-group of NW waves: wave NW - 1 copies the
// input, the others multiply.  Accumulator element i of lane (c, G) is row
// 16 cb + 4 G + i of the wave's weight rows, input row 16 rb + c of the pass.
//
//   w0      the wave's first weight row (wave-uniform); block cb starts
//           cb * block_bytes further on and has valid[cb] rows, the others
//           read as zero
//   active  false (wave-uniform): a wave without weight rows, which only
//           meets the barriers
//   x       first input row of the pass; `rows` of them exist, the other
//           rows of the RB blocks read as zero
//   ring    stream_ring_bytes(RB) of LDS
//
//   rot     0 .. ch1 - ch0 - 1: the chunk the range starts from (it wraps)
//
// The stream is bound by HBM, so everything else has to stay out of the way
// of the weight loads.  The reduction advances in steps of 128 channels.
// Weights go to registers in groups of two steps: eight 16-byte loads per
// lane and 16-row block for bf16, 512 bytes of each row, four and 256 bytes
// for int8.  Two groups of registers take turns: one is loaded while the
// other is multiplied, its loads back to back at the group's start, one
// 16-row block after the other, so that a row's bytes reach HBM together
// (issued piece by piece over both blocks, bf16 is up to 24% slower: 6 rows,
// 8192 x 28672 82 -> 102 us).  The lanes' share of a group is such that both
// types sum the same products in the same order, and that a load touches one
// 128-byte line per row.
//
// Groups of four int8 steps (eight loads) leave idle steps at the end of
// short ranges, and registers for sixteen waves only up to 64 input rows.
// Calls of sd_linear_q8 in a graph, weights from HBM, four steps (seven waves
// of 32 columns above 64 rows; under 16 and 65 to 112 rows every load issued
// as its registers came free) -> two steps: 24 rows, 4096 x 11008 20.6 -> 17.0
// us; 80 rows, 2048 x 5632 20.7 -> 14.0; 80 rows, 4096 x 11008 33.4 -> 24.2; 6
// rows, 57344 x 8192 92.0 -> 89.3; 48 rows there 108.3 -> 101.1; 112 rows
// 140.5 -> 142.5; 128 rows 164.4 -> 157.8.
//
// The input rows of a step are copied L2 -> LDS by the buffer_load ... lds
// DMA into a ring of four slots, three steps ahead.  The copying wave waits
// (a counted wait) for the copies of step t, meets the work-group and issues
// those of step t + 3 into the slot that every wave has just finished.
// Copies and weight loads count on one counter that retires in order, so a
// wave with both would have to wait for its weights whenever it waits for
// newer copies; with the copies in a wave of their own, the others wait for
// nothing but the registers they multiply next.
//
// Loads past the range or past the last row fail the buffer bounds check:
// they count like the others, so the steps need no branches and every wait
// is a compile-time constant, but move no data.
//
// The fragments are read by inline asm, four at a time, one such unit ahead
// of the matrix cores: LDS reads that the compiler sees, it orders behind
// every load in flight (s_waitcnt vmcnt(0) before a chunk's first product),
// which left HBM idle under the products.
//
// Two blocks of 16 weight rows per wave (CB = 2, bf16) take half the fragment
// reads and half the input copies per weight byte.  Measured (kernel trace,
// medians, weights from HBM; before: one block per wave, a single register
// group in flight under the products, copies in every wave): 112 rows,
// 28672 x 4096 68.0 -> 52.5 us; 4096 x 14336 39.0 -> 33.0 us; 36 rows, 57344 x
// 8192 185.6 -> 168.7 us (5.6 TB/s); 6 rows, 28672 x 4096 45.0 -> 40.8 us
// (5.75 TB/s).
template <int RB, int CB, int NW, bool Q8>
__device__ __forceinline__ void stream_product(const void* w0, size_t block_bytes, const int (&valid)[CB],
                                               bool active, const uint16_t* x, int rows,
                                               int K, int ch0, int ch1, int rot, unsigned char* ring,
                                               floatx4 (&acc)[CB][RB]) {
  constexpr int COPIES = RB * 4;                // 1 KB copies per step
  constexpr int GS = 2;                         // steps per weight group
  constexpr int WS = Q8 ? 2 : 4;                // weight loads per step, lane and 16-row block
  constexpr int GL = GS * WS;                   // and per group
  constexpr int SLOT = stream_slot_bytes(RB);
  constexpr uint32_t PAST = 0x80000000u;        // beyond every buffer's range
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), G = lane >> 4,
            c = lane & 15;
  const int t0 = ch0 * 2, t1 = ch1 * 2;         // steps of the range
  auto at = [&](int t) {                         // t-th step in this work-group's order
    t += 2 * rot;
    return t >= t1 ? t - (t1 - t0) : t;
  };
  // every wave runs whole turns of both rings; steps past the range
  // multiply zeros
  if (w == NW - 1) {
    // Copy j moves 1 KB: rows 4 j .. 4 j + 3, whose 16 pieces of a step (8
    // channels each) lie in the order p = 4 i + G of the products (i the
    // product, G the lane group that takes it), piece p at slot
    // p ^ ((row & 7) << 1), which keeps the fragment reads free of bank
    // conflicts.  Product i of a step takes channels 64 (i / 2) + 16 G +
    // 8 (i & 1) .. + 7: half of a lane's 16-byte load of int8 rows, a whole
    // one of bf16 rows, so that both sum the products in the same order.
    const auto xrsrc = stream_rsrc(x, (uint32_t)rows * (uint32_t)K * 2u);
    uint32_t xoff[2];                           // copies of even and odd j
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = j * 4 + G, p = c ^ ((row & 7) << 1);
      const int piece = (p >> 3) * 8 + (p & 3) * 2 + ((p >> 2) & 1);
      xoff[j] = (uint32_t)G * (uint32_t)K * 2u + (uint32_t)piece * 16u;
    }
    auto xcopy = [&](int t, int slot) {         // step t of the whole reduction
      const uint32_t off = t < t1 ? (uint32_t)at(t) * (kStreamStep * 2) : PAST;
#pragma unroll
      for (int j = 0; j < COPIES; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xrsrc, (stream_lds_void*)(ring + slot * SLOT + j * 1024), 16,
                                                 (int)(xoff[j & 1] + (off + (uint32_t)j * (uint32_t)K * 8u)), 0, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < 3; ++s) xcopy(t0 + s, s);
#pragma unroll 1
    for (int t = t0; t < t1; t += 2 * GS)
#pragma unroll
      for (int s = 0; s < 2 * GS; ++s) {
        wait_vm_then_barrier<(2 * COPIES < 63 ? 2 * COPIES : 63)>();
        xcopy(t + s + 3, (s + 3) & 3);
      }
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0): no copy outlives the work-group
    return;
  }
  auto meet = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  if (!active) {
#pragma unroll 1
    for (int t = t0; t < t1; t += 2 * GS)
#pragma unroll
      for (int s = 0; s < 2 * GS; ++s) meet();
    return;
  }

  const uint32_t row_bytes = (uint32_t)K * (Q8 ? 1u : 2u);
  decltype(stream_rsrc(w0, 0u)) wrsrc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
    wrsrc[cb] = stream_rsrc(static_cast<const unsigned char*>(w0) + cb * block_bytes,
                            (uint32_t)min(max(valid[cb], 0), 16) * row_bytes);
  const uint32_t woff = (uint32_t)c * row_bytes + (uint32_t)G * (Q8 ? 16u : 32u);
  u32x4 wf[2][CB][GL];
  // the group of steps t .. t + GS - 1, block by block
  auto wload = [&](u32x4 (&f)[CB][GL], int t) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i = 0; i < GL; ++i) {
        const int ts = t + i / WS;
        const uint32_t off = ts < t1 ? (uint32_t)at(ts) * (Q8 ? 128u : 256u) : PAST;
        const uint32_t in_step = Q8 ? 64u * (i & 1) : 128u * ((i & 3) >> 1) + 16u * (i & 1);
        f[cb][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc[cb], (int)(woff + off + in_step), 0, 0));
      }
  };
  uint32_t xa[4];                               // fragment addresses of the four products, slot 0
#pragma unroll
  for (int j = 0; j < 4; ++j) xa[j] = lds_addr(ring) + c * 256 + (((4 * j + G) ^ ((c & 7) << 1)) * 16);

  // products of one step: s its index within the weight group.  The step's
  // 4 RB fragments are read four at a time, one such unit ahead.
  auto multiply = [&](u32x4 (&f)[CB][GL], auto stag, auto slot_tag) {
    constexpr int s = decltype(stag)::value, SO = decltype(slot_tag)::value * SLOT;
    u32x4 xf[2][4];
    Pack8 p[CB];
    auto read = [&](auto ut) {
      constexpr int u = decltype(ut)::value;
      stream_for<0, 4>([&](auto it) {
        constexpr int i = decltype(it)::value, fr = 4 * u + i, j = fr / RB, off = SO + (fr % RB) * 4096;
        if constexpr (off < 65536)
          xf[u & 1][i] = lds_read_b128_off<off>(xa[j]);
        else
          xf[u & 1][i] = lds_read_b128_off<off - 65536>(xa[j] + 65536u);
      });
    };
    read(std::integral_constant<int, 0>{});
    stream_for<0, RB>([&](auto ut) {
      constexpr int u = decltype(ut)::value;
      if constexpr (u + 1 < RB) {
        read(std::integral_constant<int, u + 1>{});
        lds_wait_n<4>();
      } else {
        lds_wait_n<0>();
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) tie(xf[u & 1][i]);
      stream_for<0, 4>([&](auto it) {
        constexpr int i = decltype(it)::value, fr = 4 * u + i, j = fr / RB, rb = fr % RB;
        if constexpr (rb == 0) {
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) {
            if constexpr (Q8) {
              const u32x4& v = f[cb][s * WS + (j >> 1)];
              const uint32_t lo = v[(j & 1) * 2], hi = v[(j & 1) * 2 + 1];
              p[cb].u =
                  u32x4{i8x2_to_bf16x2(lo, 0), i8x2_to_bf16x2(lo, 2), i8x2_to_bf16x2(hi, 0), i8x2_to_bf16x2(hi, 2)};
            } else {
              p[cb].u = f[cb][s * WS + j];
            }
          }
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          Pack8 y;
          y.u = xf[u & 1][i];
          acc[cb][rb] = mfma_bf16(p[cb].b, y.b, acc[cb][rb]);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  wload(wf[0], t0);
#pragma unroll 1
  for (int t = t0; t < t1; t += 2 * GS)
    stream_for<0, 2 * GS>([&](auto st) {
      constexpr int s = decltype(st)::value, gs = s % GS;
      meet();
      if constexpr (gs == 0) wload(wf[(s / GS + 1) & 1], t + s + GS);
      multiply(wf[s / GS], std::integral_constant<int, gs>{}, std::integral_constant<int, s & 3>{});
    });
}

}  // namespace sd
