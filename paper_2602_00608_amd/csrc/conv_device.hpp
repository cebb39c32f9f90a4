// Pieces shared by the matrix-core convolution kernels: launch parameters, operand loads, the activation on the load
// path and the row hand-over of the output statistics.
#pragma once
#include <algorithm>
#include <type_traits>
#include <utility>

#include "mfma.hpp"
#include "moments.hpp"
#include "pack_layout.hpp"
#include "quotient.hpp"
#include "sample_offsets.hpp"

namespace wmdec {

struct MfmaParams {
  const void* x; const float* mean; const float* rstd; const float* gamma; const float* beta;
  const void* w; const float* bias; const void* res; void* y;
  int silu, groups, norm;
  int n, h, w_out, cin, cout;
  int tiles_x, tiles_y, ntiles, total;
  int cin_blocks, cout_blocks;   // packed-layout extents: ceil(cin/16), ceil(cout/32)
  int w_bytes;                   // size of the packed weights the kernel may read
  int y_nchw;                    // 1: y is planar [n][cout][h][w] (the frame), else NHWC
  Moments* stats;                // non-null: moments of y per (sample, group, slot); slot = spatial tile * WM + wave row
  int stats_cpg, stats_groups, stats_slots;
  // Statistics hand-over without a merge launch.  rows_out: the last workgroup of every (sample, tile row, channel
  // tile) merges that row's triples into one triple per group, [n][stats_groups][tiles_y]; tickets: one counter per
  // (sample, tile row, channel tile), zero before the launch and zero again after it.  rows_in: the statistics of x
  // arrive as such row triples, [n][groups][rows_in_count], and are merged while the scale/shift table is built.
  Moments* rows_out; unsigned* tickets;
  const Moments* rows_in; int rows_in_count; float eps;
  // 1x1 shortcut folded into the contraction (3x3 only): y += W2 * x2 + bias2, x2 [n,h,w,cin2] taken as stored
  const void* x2; const void* w2; const float* bias2;
  int cin2, w2_bytes;
  NextWeights next;              // next.w non-null: workgroups from `total` on only bring these weights into the L2s
  unsigned inv_tiles_n, inv_tiles, inv_tiles_x;   // see div_rem: of tiles_x * tiles_y * n, tiles_x * tiles_y, tiles_x
  unsigned cpg_in, inv_cpg_in;                    // channels of a group of x, their reciprocal
};

// a / d and its remainder, inv = reciprocal(d): the product's high half is the quotient or one less.  (The compiler's division is some
// thirty dependent instructions, and a workgroup starts with a chain of them.)
inline unsigned reciprocal(unsigned d) { return d == 1 ? 0xffffffffu : (unsigned)((1ull << 32) / d); }
__device__ __forceinline__ int div_rem(unsigned a, unsigned d, unsigned inv, int& rem) {
  unsigned q = __umulhi(a, inv), r = a - q * d;
  if (r >= d) { ++q; r -= d; }
  rem = (int)r;
  return (int)q;
}
__device__ __forceinline__ int quotient_of(unsigned a, unsigned d, unsigned inv) { int rem; return div_rem(a, d, inv, rem); }
// Brings the arguments of the kernel (BYTES of them) into the scalar cache in one round trip.  The compiler loads them where they are first
// needed, and every 64 bytes that were not asked for before are a trip of their own to memory, 500 cycles each in front of everything else: a workgroup
// of 512 channels at 60x90 had its tile after 2530 cycles, now 1100.
template <int BYTES> __device__ __forceinline__ void fetch_arguments() {
  static_assert(BYTES > 4 * 64 && BYTES <= 5 * 64, "five lines, wherever the first begins");
  const auto* at = (const uint32_t __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" :: "s"(at[0]), "s"(at[16]), "s"(at[32]), "s"(at[48]), "s"(at[64]), "s"(at[BYTES / 4 - 1]));
}
// workgroup id -> (channel tile, sample, spatial tile, its row and column); the ids of one XCD (id % 8) cover neighbouring tiles of
// one channel range, so that its L2 fetches an eighth of the weights
struct WorkTile { int nt, n, tile, y, x; };
__device__ __forceinline__ WorkTile workgroup_tile(const MfmaParams& p) {
  const unsigned i = blockIdx.x, per = (unsigned)p.total / 8, rem = (unsigned)p.total % 8;
  const unsigned x = i % 8, j = i / 8, tiles = p.tiles_x * p.tiles_y;
  WorkTile t;
  int in_nt;
  t.nt = div_rem(x * per + (x < rem ? x : rem) + j, tiles * p.n, p.inv_tiles_n, in_nt);
  t.n = div_rem(in_nt, tiles, p.inv_tiles, t.tile);
  t.y = div_rem(t.tile, p.tiles_x, p.inv_tiles_x, t.x);
  return t;
}

// Whether the workgroup is one of those behind the launch's own that only bring weights (see warm_weights).  The answer's code belongs at the end of the
// kernel (__builtin_expect): 1x1 layers of few tiles lost 0.1 to 0.2 us of 4.5 to 11 otherwise.
__device__ __forceinline__ bool carries_weights(const MfmaParams& p) { return p.next.w && (int)blockIdx.x >= p.total; }

template <typename T> __device__ __forceinline__ void unpack8(const u32x4& v, float* f) {
  f[0] = unpack_lo<T>(v.x); f[1] = unpack_hi<T>(v.x); f[2] = unpack_lo<T>(v.y); f[3] = unpack_hi<T>(v.y);
  f[4] = unpack_lo<T>(v.z); f[5] = unpack_hi<T>(v.z); f[6] = unpack_lo<T>(v.w); f[7] = unpack_hi<T>(v.w);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl<N>(f, std::make_integer_sequence<int, N>{}); }

// silu(t) from u = -log2(e) * t (see the scale/shift table)
__device__ __forceinline__ float silu_from_scaled(float u) {
  constexpr float k = -1.4426950408889634f;
  return u * __builtin_amdgcn_rcpf(fmaf(__builtin_amdgcn_exp2f(u), k, k));
}

// One weight fragment (1 KiB, a lane's 16 bytes at lane16 = 16 * lane) at byte offset `off` of the packed weights.
// A buffer load takes the wave-uniform offset in a scalar register, so the address costs no vector-ALU work
// (a global load would add the 64-bit base per fragment), and offsets past the blob read zeros instead of faulting.
__device__ __forceinline__ u32x4 load_fragment(__amdgpu_buffer_rsrc_t rsrc, int lane16, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane16, off, 0);
}

// Inside a decoder run every layer's weights are new to the L2s, and a launch of one round has nothing to hide their latency under.
// So the launch before it carries a few workgroups more, which read them: each XCD (workgroup id % 8) those that its workgroups
// of the coming launch will ask for, by the mapping that all these kernels share (consecutive L on one XCD, channel tiles outermost).  They are dispatched
// last and run beside the others.
// us a frame, without / with, by the latent: 9x9 392.9 / 388.2, 17x23 539.3 / 535.6, 32x32 759.5 / 764.1, 45x60 1719 / 1597, 60x90 2662 / 2666, four 20x30
// 1480 / 1448, three 50x70 5059 / 4951.  Launches of any number of rounds carry them: left out in or in front of launches of more than 256, 512 or 1024
// workgroups, frames are within 0.4 % of these, slower as often as faster.
constexpr int kWarmAhead = 8;   // loads in flight per wavefront, a KiB each
__device__ __forceinline__ void warm_weights(const NextWeights& nw, int first_id, int waves, int wave, int lane) {
  const int x = blockIdx.x % 8, groups = (gridDim.x - first_id) / 8;
  const int per = nw.total / 8, rem = nw.total % 8;
  const int l0 = x * per + min(x, rem), count = per + (x < rem ? 1 : 0);
  if (count == 0) return;
  const int b0 = l0 / nw.per_tile * nw.tile_blocks, b1 = min(((l0 + count - 1) / nw.per_tile + 1) * nw.tile_blocks, nw.cout_blocks);
  const int blocks = b1 - b0, items = nw.rows * blocks, step = groups * waves;
  const char* w = reinterpret_cast<const char*>(nw.w) + lane * 16;
  for (int i0 = (blockIdx.x - first_id) / 8 * waves + wave; i0 < items; i0 += kWarmAhead * step) {
    u32x4 v[kWarmAhead];
#pragma unroll
    for (int k = 0; k < kWarmAhead; ++k) {
      const int i = min(i0 + k * step, items - 1);
      v[k] = *reinterpret_cast<const u32x4*>(w + ((size_t)(i / blocks) * nw.cout_blocks + b0 + i % blocks) * 1024);
    }
#pragma unroll
    for (int k = 0; k < kWarmAhead; ++k) asm volatile("" :: "v"(v[k]));
  }
}
// workgroups of `waves` wavefronts that a launch carries for it: two trips through the loads in flight, at most eight on an XCD
inline int warm_groups(const NextWeights& nw, int waves) {
  if (!nw.w) return 0;
  const long items = (long)nw.rows * nw.cout_blocks / std::max(1, std::min(8, (nw.cout_blocks + nw.tile_blocks - 1) / nw.tile_blocks));
  return 8 * (int)std::min(8L, (items + 2 * kWarmAhead * waves - 1) / (2 * kWarmAhead * waves));
}

// 16 bytes of every lane to a buffer, at a lane offset plus a wave-uniform one in a scalar register.  The store reads its data late: where
// the next instruction overwrites them it may store what that one wrote (seen on this chip, the last lanes of a row first).
// The compiler leaves a wait state between the two only where the scalar offset is a constant; here two stand in between, and
// uses of `v` that follow come after them.
__device__ __forceinline__ void store_vector(__amdgpu_buffer_rsrc_t rsrc, u32x4& v, int lane_offset, int base) {
  __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, lane_offset, base, 0);
  asm volatile("s_nop 1" : "+v"(v));
}

// pack2 by one instruction
template <typename T> __device__ __forceinline__ uint32_t pack_word(float f0, float f1) {
  if constexpr (std::is_same<T, f16_t>::value) return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{f0, f1}, f16x2_t));
  else return pack2<T>(f0, f1);
}

// Word (two channels) of a staged vector with the table entries ab = (a0, b0, a1, b1); ACT: 0 as it is, 1 scale/shift,
// 2 scale/shift + SiLU.  PIN: the last fp32 operation and the conversion stay apart.  The compiler otherwise folds them into
// one (v_fma_mixlo_f16, one rounding instead of two) at some places and not at others, and the bits of a value would
// depend on the instantiation that staged it.
template <typename T, int ACT, bool PIN = false> __device__ __forceinline__ uint32_t activate_word(uint32_t wv, const f32x4& ab) {
  if constexpr (ACT > 0) {
    float f0 = fmaf(unpack_lo<T>(wv), ab[0], ab[1]), f1 = fmaf(unpack_hi<T>(wv), ab[2], ab[3]);
    if constexpr (ACT == 2) { f0 = silu_from_scaled(f0); f1 = silu_from_scaled(f1); }
    if constexpr (PIN) {
      asm("" : "+v"(f0), "+v"(f1));
      return pack_word<T>(f0, f1);
    }
    wv = pack2<T>(f0, f1);
  }
  return wv;
}

// 1 / sqrt(m2 / n + eps) without the compiler's division and square root (some fifty dependent instructions a launch waits for) unless the variance
// leaves the range where the steps below are exact enough.  One ulp given v, two in all; by division and square root, which round twice, it is 1.5 and 2.3
// (four million draws each, eps 0, 1e-6 and 0.3, starting values an ulp off).
__device__ __forceinline__ float inverse_deviation(float m2, float n, float eps) {
  const float v = quotient(m2, n, __builtin_amdgcn_rcpf(n)) + eps;
  float r = __builtin_amdgcn_rsqf(v);
  r = fmaf(0.5f * r, fmaf(-(v * r), r, 1.0f), r);
  if (!(v > 1e-30f && v < 1e30f)) r = 1.0f / sqrtf(m2 / n + eps);   // (zero, infinite, NaN)
  return r;
}

// (mean, rstd) of G groups from the `count` triples of their rows, each merged by LANES consecutive lanes (all of them active), K
// loads in flight per lane and group: the mean first, then the differences to it and their squares, from the same registers.  (A chain
// of pairwise merges has a reciprocal each and stood in front of every layer's first chunk; one pass of sums about the
// first triple's mean cancels where that triple is an outlier: 1e-5 of the variance at 100 standard deviations.)  Triples
// past K * LANES are summed about the mean of those, at least half of the row, which costs a factor of two at most.
constexpr int kMaxTriples = 128;   // of a group that a prologue merges
template <int LANES, int K, int G>
__device__ __forceinline__ void merge_rows(const Moments* const (&row)[G], int count, int sub, float eps, float2 (&out)[G]) {
  float first[G];
  Moments t[G][K];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    first[g] = row[g][0].mean;
#pragma unroll
    for (int k = 0; k < K; ++k) t[g][k] = row[g][min(sub + LANES * k, count - 1)];
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    auto past = [&](int r0) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (r0 + LANES * k >= count) { t[g][k].n = 0.f; t[g][k].m2 = 0.f; }
    };
    float n = 0.f, s = 0.f, q = 0.f;
    auto add = [&](float shift) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const float d = t[g][k].n > 0.f ? t[g][k].mean - shift : 0.f, nd = t[g][k].n * d;   // an empty triple's mean has no meaning
        n += t[g][k].n; s += nd; q += fmaf(nd, d, t[g][k].m2);
      }
    };
    past(sub);
    add(first[g]);
    const float head = lanes_sum<LANES>(n);
    const float mean = first[g] + lanes_sum<LANES>(s) * __builtin_amdgcn_rcpf(head);
    n = 0.f; s = 0.f; q = 0.f;
    add(mean);
    if (K == 8 && K * LANES < kMaxTriples && count > K * LANES) {
      n = 0.f;
      for (int r0 = sub + K * LANES; r0 < count + sub; r0 += K * LANES) {
#pragma unroll
        for (int k = 0; k < K; ++k) t[g][k] = row[g][min(r0 + LANES * k, count - 1)];
        past(r0);
        add(mean);
      }
      n = head + lanes_sum<LANES>(n);
    } else {
      n = head;
    }
    s = lanes_sum<LANES>(s); q = lanes_sum<LANES>(q);
    const float d = s * __builtin_amdgcn_rcpf(n);     // (also what the roundings of `mean` left)
    q -= s * d;
    out[g] = make_float2(mean + d, inverse_deviation(q < 0.f ? 0.f : q, n, eps));   // (NaN stays NaN)
  }
}
// ... of all groups of a sample into s_stat, by NT threads: as many loads as the row needs (a triple that does not exist adds zeros,
// so the number changes no bits), and of two groups at a time where the threads do not reach round.
template <int LANES, int NT>
__device__ __forceinline__ void merge_sample(const Moments* rows, int groups, int count, int tid, float eps, float2* s_stat) {
  constexpr int STEP = NT / LANES;
  const int sub = tid % LANES;
  auto all = [&](auto k_c, auto g_c) __attribute__((always_inline)) {
    constexpr int K = decltype(k_c)::value, G = decltype(g_c)::value;
    for (int g0 = tid / LANES; g0 < groups; g0 += G * STEP) {
      const Moments* row[G];
      float2 st[G];
#pragma unroll
      for (int g = 0; g < G; ++g) row[g] = rows + (size_t)min(g0 + g * STEP, groups - 1) * count;
      merge_rows<LANES, K, G>(row, count, sub, eps, st);
#pragma unroll
      for (int g = 0; g < G; ++g)
        if (sub == 0 && g0 + g * STEP < groups) s_stat[g0 + g * STEP] = st[g];
    }
  };
  const std::integral_constant<int, 1> one{};
  const std::integral_constant<int, (STEP < 32 ? 2 : 1)> pair{};
  if (count <= LANES) all(one, pair);
  else if (count <= 2 * LANES) all(std::integral_constant<int, 2>{}, pair);
  else if (count <= 4 * LANES) all(std::integral_constant<int, 4>{}, pair);
  else all(std::integral_constant<int, 8>{}, one);
}

// Sums over lanes in the vector ALU.  row_rotate: the value N lanes further round the row of 16; quad_xor: of lane ^ N (1, 2);
// swap_sum: v of this lane plus that of lane ^ W (16, 32; the results of the swap are made opaque, as this compiler takes both
// for the first one where the operands are the same).
template <int N> __device__ __forceinline__ float row_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, true));
}
template <int N> __device__ __forceinline__ float quad_xor(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), N == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true));
}
template <int W> __device__ __forceinline__ float swap_sum(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  u32x2 r;
  if constexpr (W == 16) r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  else r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  unsigned a = r.x, b = r.y;
  asm volatile("" : "+v"(a), "+v"(b));
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

// value of the mirrored lane in eight, in sixteen lanes
__device__ __forceinline__ float mirror8(float v) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xf, 0xf, true)); }
__device__ __forceinline__ float mirror16(float v) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xf, 0xf, true)); }
// sum over WIDTH consecutive lanes (a power of two up to 16), in all of them
template <int WIDTH> __device__ __forceinline__ float lane_group_sum(float v) {
  if constexpr (WIDTH > 1) v += quad_xor<1>(v);
  if constexpr (WIDTH > 2) v += quad_xor<2>(v);
  if constexpr (WIDTH > 4) v += mirror8(v);
  if constexpr (WIDTH > 8) v += mirror16(v);
  return v;
}

// Moments of a group's channels (CPG consecutive lanes, a power of two up to 32) over the same pixels, in all of these lanes: the mean
// first, then the squares about it.
template <int CPG> __device__ __forceinline__ Moments merge_channels(Moments m) {
  auto sum = [&](float v) {
    v = lane_group_sum<(CPG < 16 ? CPG : 16)>(v);
    return CPG > 16 ? swap_sum<16>(v) : v;
  };
  const float inv = 1.f / CPG;                           // (a power of two: exact)
  const float mean = sum(m.mean) * inv, d = m.mean - mean;
  const float rest = sum(d) * inv;                       // what the roundings of the mean left
  const float m2 = sum(fmaf(m.n * d, d, m.m2)) - m.n * (float)CPG * rest * rest;
  return Moments{m.n * (float)CPG, mean + rest, m2 < 0.f ? 0.f : m2};   // (NaN stays NaN)
}
// f(integral_constant<int, cpg>): a form of its own for every size of a group.  (Where one form looked at the size between the lane moves, divided by it
// for the group and read a ragged block's values behind branches, the moments were 2130 of the 19 850 cycles of a workgroup of 512 channels at 17x23, now 1420.)
template <typename F> __device__ __forceinline__ void with_group_size(int cpg, F&& f) {
  if (cpg == 16) f(std::integral_constant<int, 16>{});
  else if (cpg == 8) f(std::integral_constant<int, 8>{});
  else if (cpg == 4) f(std::integral_constant<int, 4>{});
  else if (cpg == 2) f(std::integral_constant<int, 2>{});
  else if (cpg == 1) f(std::integral_constant<int, 1>{});
  else f(std::integral_constant<int, 32>{});
}

// Moments of one channel over a block of 4 x W pixels (rows x cols of them valid) in LDS, pixels PX and image rows ROW floats apart:
// sums about the block's first value, the rows in chains of their own, which are added in pairs (so that two lanes may take
// two rows each).
struct Sums { float s, q; };
__device__ __forceinline__ Sums operator+(Sums a, Sums b) { return Sums{a.s + b.s, a.q + b.q}; }
template <int W, int PX, bool FULL> __device__ __forceinline__ Sums row_sums(const float* src, float shift, int count) {
  float v[W];
#pragma unroll
  for (int x = 0; x < W; ++x) {
    v[x] = src[x * PX];
    if constexpr (!FULL) asm("" : "+v"(v[x]));   // (read whether it counts or not: the compiler would branch round every read)
  }
  Sums r{0.f, 0.f};
#pragma unroll
  for (int x = 0; x < W; ++x) {
    const float d = FULL || x < count ? v[x] - shift : 0.f;
    r.s += d; r.q = fmaf(d, d, r.q);
  }
  return r;
}
template <int W, int ROW, int PX> __device__ __forceinline__ Sums two_row_sums(const float* src, float shift, int rows, int cols) {
  if (rows >= 2 && cols == W) return row_sums<W, PX, true>(src, shift, W) + row_sums<W, PX, true>(src + ROW, shift, W);
  return row_sums<W, PX, false>(src, shift, rows > 0 ? cols : 0) + row_sums<W, PX, false>(src + ROW, shift, rows > 1 ? cols : 0);
}
__device__ __forceinline__ Moments block_moments(Sums t, float shift, int rows, int cols) {
  if (rows <= 0 || cols <= 0) return Moments{0.f, 0.f, 0.f};
  const float cnt = (float)(rows * cols), ds = quotient(t.s, cnt, __builtin_amdgcn_rcpf(cnt)), m2 = t.q - t.s * ds;
  return Moments{cnt, shift + ds, m2 < 0.f ? 0.f : m2};
}

// Row hand-over: the workgroup that finishes a (sample, tile row, channel tile) last merges that row's triples.  The
// triples were written with device-scope stores, every wavefront
// waits for its stores, the workgroup takes a ticket (a wrapping counter that returns to zero by itself), and only the
// last one reads, with device-scope loads, in a fixed order.  per_tile: triples of one group a workgroup leaves.
template <int NT>
__device__ __forceinline__ void hand_over_row(const MfmaParams& p, int n, int tile_y, int nt, int co0, int tn, int per_tile,
                                              int tid, int lane) {
  __shared__ unsigned s_last;
  wait_stores();
  __syncthreads();
  if (tid == 0) s_last = atomicInc(p.tickets + ((size_t)n * p.tiles_y + tile_y) * p.ntiles + nt, p.tiles_x - 1) == (unsigned)(p.tiles_x - 1);
  __syncthreads();
  if (!s_last) return;
  const int per_row = p.tiles_x * per_tile;                  // triples of one group in this tile row
  const int g0 = co0 / p.stats_cpg, gcount = min(tn, p.cout - co0) / p.stats_cpg;
  const int sub = tid & 7;
  for (int gi = tid >> 3; gi < gcount; gi += NT / 8) {
    const Moments* src = p.stats + ((size_t)n * p.stats_groups + g0 + gi) * p.stats_slots + (size_t)tile_y * per_row;
    Moments m{0.f, 0.f, 0.f};
    for (int e0 = sub; e0 < per_row; e0 += 64) {     // eight loads in flight per lane
      Moments t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int e = e0 + 8 * k;
        t[k] = load_device(src + min(e, per_row - 1));
        if (e >= per_row) t[k].n = 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) m = merge(m, t[k]);
    }
    m = merge_to_first(m, lane, 8);
    if (sub == 0) p.rows_out[((size_t)n * p.stats_groups + g0 + gi) * p.tiles_y + tile_y] = m;
  }
}

// The kernels address packed weights by 32-bit byte offsets, and a fragment past the last round by one of 0x7fff0000:
// larger layers are left to the general kernel.
inline bool packed_offsets_fit(int taps, int cout, int cin, int op_dtype) {
  return packed_elems(taps, cout, cin) * dtype_size(op_dtype) < 0x7fff0000u;
}

// Launch parameters of a th x tw tile (on an h_t x w_t grid) with tn output channels and slots_per_tile moment triples;
// the weights and the shortcut are the caller's.
inline MfmaParams conv_params(const ConvArgs& a, int th, int tw, int tn, int slots_per_tile, int h_t, int w_t) {
  MfmaParams p;
  p.x = a.x; p.mean = a.mean; p.rstd = a.rstd; p.gamma = a.gamma; p.beta = a.beta;
  p.w = nullptr; p.w_bytes = 0; p.bias = a.bias; p.res = a.res; p.y = a.y;
  p.silu = a.silu; p.groups = a.groups; p.norm = a.mean != nullptr || a.rows_in != nullptr;
  p.n = a.n; p.h = a.h; p.w_out = a.w; p.cin = a.cin; p.cout = a.cout;
  p.tiles_x = (w_t + tw - 1) / tw; p.tiles_y = (h_t + th - 1) / th; p.ntiles = (a.cout + tn - 1) / tn;
  p.total = p.tiles_x * p.tiles_y * p.ntiles * a.n;
  p.inv_tiles_n = reciprocal(p.tiles_x * p.tiles_y * a.n); p.inv_tiles = reciprocal(p.tiles_x * p.tiles_y); p.inv_tiles_x = reciprocal(p.tiles_x);
  p.cin_blocks = packed_cin_blocks(a.cin); p.cout_blocks = packed_cout_blocks(a.cout); p.y_nchw = a.y_nchw;
  p.stats = (Moments*)a.stats_ws; p.stats_groups = a.stats_groups; p.stats_cpg = a.stats_groups > 0 ? a.cout / a.stats_groups : 1;
  p.stats_slots = p.tiles_x * p.tiles_y * slots_per_tile;
  p.rows_out = (Moments*)a.rows_out; p.tickets = (unsigned*)a.tickets;
  p.rows_in = (const Moments*)a.rows_in; p.rows_in_count = a.rows_in_count; p.eps = a.eps;
  p.x2 = nullptr; p.w2 = nullptr; p.bias2 = nullptr; p.cin2 = 0; p.w2_bytes = 0;
  p.cpg_in = std::max(1, a.cin / a.groups); p.inv_cpg_in = reciprocal(p.cpg_in);
  p.next = a.next;
  return p;
}
// the statistics hand-over a launch is asked for is one its kernel can serve
inline int check_hand_over(const MfmaParams& p) {
  WMDEC_REQUIRE(!p.rows_out || (p.stats && p.tickets), WMDEC_ERR_INVALID_ARG, "convolution: row moments need the triple scratch and the ticket counters");
  WMDEC_REQUIRE(!p.rows_in || (p.rows_in_count >= 1 && p.rows_in_count <= kMaxTriples), WMDEC_ERR_UNSUPPORTED, "convolution: at most %d triples per group can be merged in the prologue", kMaxTriples);
  return WMDEC_OK;
}

}  // namespace wmdec
