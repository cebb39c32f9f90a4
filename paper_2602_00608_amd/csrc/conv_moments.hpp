// Moments that a convolution's epilogue gathers from the values it stores, shared by the matrix-core kernels.
#pragma once
#include "conv_device.hpp"

namespace wmdec {

// MODE of a matrix-core kernel: kRows4, kQuarters and kSixEight are forms between which and another kernel the batch decides, while a sample's
// bits must not depend on that choice; so they keep the activation's roundings apart (PIN).
//   kRows4     one of a pair of tiles, 4x16 and 8x16 (see four_row_slots): moments per four rows.
//   kQuarters  the batched form of kernels_conv_ksplit.hip, with its order of summation: of every 64 input channels the
//              k-th 16 belong to partial sum k, each of them is summed on its own, 16 channels and their nine taps at a
//              time, and the four are added in order.  Here one after the other into a second set of accumulators, on M tiles of 4 x 8
//              pixels, the blocks of that kernel's moments.
//   kSixEight  one of a pair of tiles, 6x16 and 8x16 (see six_eight_pair): moments per run of rows between multiples of six and of eight, one or two
//              runs a tile of either kind.
enum ConvMode { kPlain = 0, kRows4 = 1, kQuarters = 2, kSixEight = 3 };

// kSixEight: of every 24 rows the runs begin at 0, 6, 8, 12, 16 and 18.  The run that a row belongs to, and the rows from it to the next run.
__host__ __device__ constexpr int six_eight_run(int row) {
  const int r = row % 24;
  return row / 24 * 6 + (r >= 6) + (r >= 8) + (r >= 12) + (r >= 16) + (r >= 18);
}
__host__ __device__ constexpr int six_eight_rows_left(int row) {
  const int six = 6 - row % 6, eight = 8 - row % 8;
  return six < eight ? six : eight;
}

// Moments of a wavefront's stored values in the making: per channel of the lane (CH neighbouring ones) shifted sums over n pixels.
template <int CH> struct LaneMoments { float n, shift[CH], s[CH], q[CH]; };
struct RelMoments { float n, mean, m2, about; };   // (the mean lacks `about`)

// ... merged per group and written, N of them side by side (each is a chain of dependent lane moves).  A lane merges its channels of a
// group (PARTS groups, or its part of a larger one), then the lanes that hold the same channels, and those of the group's other
// channels, are summed in the vector ALU (lanes): the mean first,
// then the squares about it.  (Through LDS, with a lane per channel that walked the others' sums and re-centred them one by
// one, this was 13 of the 122 us of 128 -> 128 channels at 480x720, and 1.5 of 36 at 60x90.)  co: the lane's first channel; writes: whether
// it is the lane that writes its groups; SOME: dst is null where there are none; all_n: pixels times lanes of a group where that is known, otherwise 0; REL: for lanes of few
// pixels.  Means, and the one written, are differences to that of one lane where the values lie far from zero (from_lane chooses, the same for all lanes that are summed): a few pixels' own mean is
// rounded at its exponent, which the squares about the group's mean would count.
template <int CH, int PARTS, bool SOME, bool REL = false, int N, typename Out, typename Lanes, typename Lane>
__device__ __forceinline__ void emit_moments(const LaneMoments<CH> (&st)[N], Out* const (&dst)[N], int co, bool writes, int cpg, int stats_stride, bool handed_over,
                                             float all_n, Lanes&& lanes, Lane&& from_lane) {
  constexpr int PC = CH / PARTS;
  float inv[N], n[N], ninv[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    inv[k] = st[k].n > 0.f ? __builtin_amdgcn_rcpf(st[k].n) : 0.f;
    n[k] = all_n > 0.f ? all_n : lanes(st[k].n);
    ninv[k] = n[k] > 0.f ? __builtin_amdgcn_rcpf(n[k]) : 0.f;   // 1 ulp: `rest` corrects the mean
  }
  float about[PARTS][N];
  if constexpr (REL) {
#pragma unroll
    for (int g = 0; g < PARTS; ++g)   // (of all groups at once: what the lanes are asked for is under way together)
#pragma unroll
      for (int k = 0; k < N; ++k) about[g][k] = from_lane(st[k].n > 0.f ? fmaf(st[k].s[g * PC], inv[k], st[k].shift[g * PC]) : __builtin_inff());
  }
#pragma unroll
  for (int g = 0; g < PARTS; ++g) {
    float m[N], q[N], dev[N], mid[N], rest[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      float mean[PC];
      m[k] = 0.f; q[k] = 0.f; dev[k] = 0.f;
#pragma unroll
      for (int e = 0; e < PC; ++e) {
        const int c = g * PC + e;
        const float ds = quotient(st[k].s[c], st[k].n, inv[k]), m2 = st[k].q[c] - st[k].s[c] * ds;
        mean[e] = REL ? (st[k].shift[c] - about[g][k]) + ds : st[k].shift[c] + ds;
        m[k] += mean[e];
        q[k] += m2 < 0.f ? 0.f : m2;     // (NaN stays NaN)
      }
      m[k] = st[k].n > 0.f ? m[k] * (1.f / PC) : 0.f;     // the shift of a lane without pixels has no meaning
#pragma unroll
      for (int e = 0; e < PC; ++e) { const float d = mean[e] - m[k]; dev[k] = fmaf(d, d, dev[k]); }
    }
#pragma unroll
    for (int k = 0; k < N; ++k) mid[k] = lanes(st[k].n * m[k]) * ninv[k];
#pragma unroll
    for (int k = 0; k < N; ++k) rest[k] = REL ? 0.f : lanes(st[k].n * (m[k] - mid[k])) * ninv[k];       // what the roundings of mid left (nothing of a difference)
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const float d = m[k] - mid[k], nd = st[k].n * d;
      q[k] = lanes(st[k].n > 0.f ? fmaf(st[k].n, dev[k], fmaf(nd * PC, d, q[k])) : 0.f) - n[k] * PC * rest[k] * rest[k];
    }
    if (writes) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        if (SOME && !dst[k]) continue;
        Out* at = dst[k] + (size_t)((co + g * PC) / cpg) * stats_stride;
        if constexpr (REL) *at = RelMoments{n[k] * PC, mid[k] + rest[k], q[k] < 0.f ? 0.f : q[k], about[g][k]};
        else {
          const Moments out{n[k] * PC, mid[k] + rest[k], q[k] < 0.f ? 0.f : q[k]};
          if (handed_over) store_device(at, out);   // another workgroup of this launch may merge them, see the row hand-over of the kernels
          else *at = out;
        }
      }
    }
  }
}

// Lane l holds vector l % VECTORS of the wavefront's channels, CH of them each.
template <int VECTORS, int CH, bool REL = false, typename Out>
__device__ __forceinline__ void emit_vectors(const LaneMoments<CH> (&st)[1], int lane, int co_w, Out* const (&dst)[1], int cpg, int stats_stride, bool handed_over) {
  static_assert(CH == 4 || CH == 8, "16 bytes");
  auto lanes = [&](float v) {
    if constexpr (VECTORS <= 4) v += row_rotate<4>(v);
    v += row_rotate<8>(v);
    v = swap_sum<32>(swap_sum<16>(v));
    if (cpg > CH) v += quad_xor<1>(v);
    if (cpg > 2 * CH) v += quad_xor<2>(v);
    return v;
  };
  const int co = co_w + lane * CH;
  // of a channel's mean in two lanes that are half a wavefront apart the one nearer to zero, if it is far from zero for how far they are from each other; otherwise there is nothing to take off, or
  // one of them has an outlier among its pixels
  auto from_lane = [&](float v) {
    const int head = lane % VECTORS & ~(max(cpg / CH, 1) - 1);   // the lanes of the group's first channels
    const float low = __shfl(v, head), high = __shfl(v, head + 32), near = fabsf(low) <= fabsf(high) ? low : high;
    return fabsf(near) > 8.f * fabsf(low - high) || fabsf(high) == __builtin_inff() ? near : 0.f;   // (infinite: a lane without pixels)
  };
  const bool writes = lane < VECTORS && ((lane * CH) & (cpg - 1)) == 0;
  if (cpg >= CH) emit_moments<CH, 1, false, REL>(st, dst, co, writes, cpg, stats_stride, handed_over, 0.f, lanes, from_lane);
  else if (cpg == CH / 2) emit_moments<CH, 2, false, REL>(st, dst, co, writes, cpg, stats_stride, handed_over, 0.f, lanes, from_lane);
  else if (cpg == CH / 4) emit_moments<CH, 4, false, REL>(st, dst, co, writes, cpg, stats_stride, handed_over, 0.f, lanes, from_lane);
  else if constexpr (CH == 8) emit_moments<8, 8, false, REL>(st, dst, co, writes, cpg, stats_stride, handed_over, 0.f, lanes, from_lane);
}

// Lane l holds channels 2 (l % 16) and the next of 32, of the pixels of quarter l / 16; full: all lanes hold the same number of them.
// A form for every size of a group: with the size looked at between the lane moves, the branches took longer than they do.
template <int N>
__device__ __forceinline__ void emit_pairs(const LaneMoments<2> (&st)[N], bool full, int lane, int co_w, Moments* const (&dst)[N], int cpg, int stats_stride, bool handed_over) {
  auto emit = [&](auto cpg_c) __attribute__((always_inline)) {
    constexpr int CPG = decltype(cpg_c)::value, PARTS = CPG == 1 ? 2 : 1, WIDTH = CPG == 1 ? 1 : CPG / 2;   // lanes of a group
    auto lanes = [&](float v) {
      v = swap_sum<32>(swap_sum<16>(v));
      return lane_group_sum<WIDTH>(v);
    };
    emit_moments<2, PARTS, (N > 1)>(st, dst, co_w + 2 * (lane & 15), lane < 16 && lane % WIDTH == 0, CPG, stats_stride, handed_over, full ? st[0].n * (4.f * WIDTH) : 0.f, lanes, [](float v) { return v; });
  };
  if (cpg == 16) emit(std::integral_constant<int, 16>{});
  else if (cpg == 8) emit(std::integral_constant<int, 8>{});
  else if (cpg == 4) emit(std::integral_constant<int, 4>{});
  else if (cpg == 2) emit(std::integral_constant<int, 2>{});
  else if (cpg == 1) emit(std::integral_constant<int, 1>{});
  else emit(std::integral_constant<int, 32>{});
}

}  // namespace wmdec
