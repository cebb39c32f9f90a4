// Moments that a convolution's epilogue gathers from the values it stores, shared by the matrix-core kernels.
#pragma once
#include "conv_device.hpp"

namespace wmdec {

// MODE of a matrix-core kernel: kRows4 and kQuarters are forms between which and another kernel the batch decides, while a sample's
// bits must not depend on that choice; so both keep the activation's roundings apart (PIN).
//   kRows4     one of a pair of tiles, 4x16 and 8x16 (see four_row_slots): moments per four rows.
//   kQuarters  the batched form of kernels_conv_ksplit.hip, with its order of summation: of every 64 input channels the
//              k-th 16 belong to partial sum k, each of them is summed on its own, 16 channels and their nine taps at a
//              time, and the four are added in order.  Here one after the other into a second set of accumulators, on M tiles of 4 x 8
//              pixels, the blocks of that kernel's moments.
enum ConvMode { kPlain = 0, kRows4 = 1, kQuarters = 2 };

// Moments of a wavefront's stored values in the making: per channel of the lane's octet sums shifted by the lane's first value,
// over n pixels.
struct LaneMoments { float n, shift[8], s[8], q[8]; };

// ... merged per group and written.  A lane merges its channels of a group (PARTS groups per octet, or its part of a larger one),
// then the lanes that hold the same octet, and those of the group's other octets, are summed in the vector ALU: the mean first,
// then the squares about it.  (Through LDS, with a lane per channel that walked the others' sums and re-centred them one by
// one, this was 13 of the 122 us of 128 -> 128 channels at 480x720, and 1.5 of 36 at 60x90.)  OCTETS: octets of channels of the wavefront;
// LANE_ROWS: a row of 16 lanes holds one of four octets, otherwise lane l holds octet l % OCTETS.
template <int OCTETS, int PARTS, bool LANE_ROWS>
__device__ __forceinline__ void emit_moments(const LaneMoments& st, int lane, int co_w, Moments* dst, int cpg, int stats_stride, bool handed_over) {
  static_assert(!LANE_ROWS || OCTETS == 4, "a row of lanes per octet");
  constexpr int PC = 8 / PARTS;
  auto lanes = [&](float v) {
    if constexpr (LANE_ROWS) {
      v += row_rotate<1>(v);
      v += row_rotate<2>(v);
      v += row_rotate<4>(v);
      v += row_rotate<8>(v);
      if (cpg > 8) v = swap_sum<16>(v);
      if (cpg > 16) v = swap_sum<32>(v);
    } else {
      if constexpr (OCTETS <= 4) v += row_rotate<4>(v);
      v += row_rotate<8>(v);
      v = swap_sum<32>(swap_sum<16>(v));
      if (cpg > 8) v += quad_xor<1>(v);
      if (cpg > 16) v += quad_xor<2>(v);
    }
    return v;
  };
  const float inv = st.n > 0.f ? __builtin_amdgcn_rcpf(st.n) : 0.f;
  const float n = lanes(st.n), ninv = n > 0.f ? __builtin_amdgcn_rcpf(n) : 0.f;   // 1 ulp: `rest` corrects the mean
#pragma unroll
  for (int g = 0; g < PARTS; ++g) {
    float mean[PC], m = 0.f, q = 0.f;
#pragma unroll
    for (int e = 0; e < PC; ++e) {
      const int c = g * PC + e;
      const float ds = quotient(st.s[c], st.n, inv), m2 = st.q[c] - st.s[c] * ds;
      mean[e] = st.shift[c] + ds;
      m += mean[e];
      q += m2 < 0.f ? 0.f : m2;     // (NaN stays NaN)
    }
    m = st.n > 0.f ? m * (1.f / PC) : 0.f;     // the shift of a lane without pixels has no meaning
    float dev = 0.f;
#pragma unroll
    for (int e = 0; e < PC; ++e) { const float d = mean[e] - m; dev = fmaf(d, d, dev); }
    const float mid = lanes(st.n * m) * ninv;
    const float d = m - mid, nd = st.n * d;
    const float rest = lanes(nd) * ninv;       // what the roundings of mid left
    q = lanes(st.n > 0.f ? fmaf(st.n, dev, fmaf(nd * PC, d, q)) : 0.f) - n * PC * rest * rest;
    const Moments out{n * PC, mid + rest, q < 0.f ? 0.f : q};
    const int octet = LANE_ROWS ? lane >> 4 : lane;
    if ((LANE_ROWS ? (lane & 15) == 0 : lane < OCTETS) && ((octet * 8) & (cpg - 1)) == 0) {
      Moments* at = dst + (size_t)((co_w + octet * 8 + g * PC) / cpg) * stats_stride;
      if (handed_over) store_device(at, out);   // another workgroup of this launch may merge them, see the row hand-over of the kernels
      else *at = out;
    }
  }
}

template <int OCTETS, bool LANE_ROWS>
__device__ __forceinline__ void emit_groups(const LaneMoments& st, int lane, int co_w, Moments* dst, int cpg, int stats_stride, bool handed_over) {
  if (cpg >= 8) emit_moments<OCTETS, 1, LANE_ROWS>(st, lane, co_w, dst, cpg, stats_stride, handed_over);
  else if (cpg == 4) emit_moments<OCTETS, 2, LANE_ROWS>(st, lane, co_w, dst, cpg, stats_stride, handed_over);
  else if (cpg == 2) emit_moments<OCTETS, 4, LANE_ROWS>(st, lane, co_w, dst, cpg, stats_stride, handed_over);
  else emit_moments<OCTETS, 8, LANE_ROWS>(st, lane, co_w, dst, cpg, stats_stride, handed_over);
}

}  // namespace wmdec
