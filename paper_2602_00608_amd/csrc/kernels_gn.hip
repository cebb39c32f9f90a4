// GroupNorm statistics: a streaming read of an NHWC tensor producing, per
// (sample, group), the mean and 1/sqrt(biased variance + eps).
//
// The pixels of a sample are cut into slabs; a workgroup reads its slab with
// 16-byte vector loads (every thread keeps a fixed set of channels), accumulates
// shifted sums in fp32 (so that E[d^2]-E[d]^2 never cancels) and produces one
// (count, mean, M2) triple per group.  Triples are merged with the pairwise
// update of Chan et al., or many at a time about their common mean, in a fixed
// order, so the result does not depend on scheduling.  Channel counts that fit the vector layout take gn_stats_columns (small
// images) or gn_stats_vec; everything else takes gn_partial_any.  Where several workgroups share a sample, gn_finalize merges their triples, as
// it does the moments a convolution emitted from its epilogue.
#include <mutex>
#include <type_traits>

#include "conv_moments.hpp"

namespace wmdec {
namespace {

struct alignas(16) f32x4s { float x, y, z, w; };

template <typename T> struct Vec16;  // 16-byte vector of T
template <> struct alignas(16) Vec16<float> { static constexpr int N = 4; float v[4]; };
template <> struct alignas(16) Vec16<bf16_t> { static constexpr int N = 8; bf16_t v[8]; };
template <> struct alignas(16) Vec16<f16_t> { static constexpr int N = 8; f16_t v[8]; };

// Fast path: c % V == 0, vp = c / V divides 1024, channels per group a power of two <= 64.
// grid = (chunks, n), 1024 threads.  ws: [n][groups][chunks] Moments.  A workgroup
// streams its slab (8 loads of 16 bytes in flight per thread, the ragged end as one masked batch), sums
// x - shift and its square per thread (shift = the thread's first pixel, so that an outlier costs only the sums of
// the thread that starts with it), merges the (mean, M2) of a channel's threads in a fixed order through LDS, the
// channels of a group in its lanes, and writes one triple per group, which gn_finalize merges (mean / rstd at once where a slab is the sample).  A launch of its own
// for that takes 2.3 us; with the merge in the sample's last workgroup (triples written through to memory, a ticket, triples read back: three
// memory round trips behind each other) all shapes took longer.  us, that way / this way: f16 512 channels 60x90 11.1 / 9.0, 120x180 15.5 / 11.0, 256 channels 240x360 18.6 / 14.0,
// 128 channels 480x720 23.1 / 19.9, four of them 71.5 / 65.6; f32 512 channels 60x90 11.6 / 8.1, 120x180 17.3 / 12.5, 128 channels 480x720 39.8 / 37.6.
constexpr int kVecThreads = 1024;
constexpr int kVecMaxChunks = 256;
constexpr int kVecMaxGroups = 256;    // (more take the general pass; no level of a decoder has them)

// MIX: of f16, conversion and shift are one instruction (v_fma_mix_f32; the compiler makes it if it does not see that the factor is 1).
template <typename T, int V, bool MASKED, int U = 8, bool MIX = false>
__device__ __forceinline__ void gn_accumulate(const char* slab, unsigned off, unsigned end, unsigned sweep, const float* shift,
                                              float* s, float* q) {
  float one = 1.f;
  if constexpr (MIX && std::is_same<T, f16_t>::value) asm("" : "+v"(one));
  Vec16<T> v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned at = off + u * sweep;
    v[u] = *reinterpret_cast<const Vec16<T>*>(slab + (MASKED && at >= end ? off : at));   // always a pixel of this slab: no branch around the load
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool live = !MASKED || off + u * sweep < end;
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const float d = live ? fmaf(to_float(v[u].v[j]), one, -shift[j]) : 0.f;
      s[j] += d;
      q[j] = fmaf(d, d, q[j]);
    }
  }
}

// Merge of the triples at(0), ..., at(COUNT-1), or of `count` of them if COUNT is 0: the mean first, then the differences to it and their squares.
template <int COUNT, typename At> __device__ __forceinline__ Moments merge_all(At&& at, int count = COUNT) {
  const float first = at(0).mean;
  Moments m{0.f, 0.f, 0.f};
  float s = 0.f;
#pragma unroll 8
  for (int k = 0; k < (COUNT ? COUNT : count); ++k) { const Moments t = at(k); m.n += t.n; s = fmaf(t.n, t.mean - first, s); }
  if (m.n == 0.f) return m;
  const float inv = __builtin_amdgcn_rcpf(m.n);   // 1 ulp: the second pass corrects the mean
  m.mean = fmaf(s, inv, first);
  s = 0.f;
#pragma unroll 8
  for (int k = 0; k < (COUNT ? COUNT : count); ++k) {
    const Moments t = at(k);
    const float d = t.mean - m.mean, nd = t.n * d;
    s += nd; m.m2 += fmaf(nd, d, t.m2);
  }
  m.mean = fmaf(s, inv, m.mean);
  return m;
}

// Eight wavefronts per SIMD, two workgroups per compute unit, where 64 registers hold the eight loads and the sums: at one,
// eight f16 samples of 256 channels at 68x92 took 2.7 us more.  bf16, which converts by shifts and masks, would spill.
template <typename T> constexpr int vec_waves() { return std::is_same<T, bf16_t>::value ? 4 : 8; }

template <typename T>
__global__ __launch_bounds__(kVecThreads, vec_waves<T>()) void gn_stats_vec(const T* __restrict__ x, int pixels, int c, int groups,
                                                            int chunk_pixels, Moments* ws, float eps,
                                                            float* __restrict__ mean, float* __restrict__ rstd) {
  constexpr int V = Vec16<T>::N;
  constexpr int U = 8;
  __shared__ float2 s_e[kVecThreads * V];   // (mean, M2) per (pixel lane, channel)
  __shared__ Moments s_p[kVecThreads];      // triples per (part of the pixel lanes, channel)
  const int tid = threadIdx.x;
  const int vp = c / V;           // vectors per pixel
  const int cv = tid % vp;        // this thread's channel vector
  const int ppi = kVecThreads / vp;   // pixels per sweep of the workgroup
  const int chunk = blockIdx.x, n = blockIdx.y, chunks = gridDim.x;
  const int p0 = chunk * chunk_pixels;
  const int p1 = min(p0 + chunk_pixels, pixels);
  // A sweep is 16 KiB of consecutive memory, a thread's vectors are 16 KiB apart.  Byte offsets into the slab have 32 bits
  // (a slab is the 256th part of a sample, or a few sweeps).
  const char* slab = reinterpret_cast<const char*>(x + ((size_t)n * pixels + p0) * c);
  const unsigned end = (unsigned)(p1 - p0) * vp * 16, sweep = kVecThreads * 16;

  unsigned off = tid * 16;   // pixel tid / vp, channel vector tid % vp
  float shift[V], s[V], q[V];
  {
    const Vec16<T> v = *reinterpret_cast<const Vec16<T>*>(slab + (off < end ? off : cv * 16));
#pragma unroll
    for (int j = 0; j < V; ++j) { shift[j] = to_float(v.v[j]); s[j] = 0.f; q[j] = 0.f; }
  }
  for (; off + (U - 1) * sweep < end; off += U * sweep) gn_accumulate<T, V, false>(slab, off, end, sweep, shift, s, q);
  if (off < end) gn_accumulate<T, V, true>(slab, off, end, sweep, shift, s, q);

  const int sweeps = (p1 - p0) / ppi, rest = (p1 - p0) % ppi;
  auto lane_pixels = [&](int lane) { return (float)(sweeps + (lane < rest ? 1 : 0)); };   // pixels of a pixel lane
  {
    const float cnt = lane_pixels(tid / vp), inv = cnt > 0.f ? __builtin_amdgcn_rcpf(cnt) : 0.f;   // 1 ulp of a difference to the shift
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const float ds = s[j] * inv, m2 = q[j] - s[j] * ds;
      s_e[(tid / vp) * c + cv * V + j] = float2{shift[j] + ds, m2 < 0.f ? 0.f : m2};   // (NaN stays NaN)
    }
  }
  __syncthreads();
  // all threads take V of a channel's ppi entries each (c is a power of two <= 1024 here), then one per channel the parts:
  // with a thread per channel alone the walk over 64 entries at 64 channels was a quarter of a small tensor's time
  const int parts = kVecThreads / c;
  s_p[tid] = merge_all<V>([&](int k) {
    const int r = tid / c + k * parts;
    const float2 e = s_e[r * c + tid % c];
    return Moments{lane_pixels(r), e.x, e.y};
  });
  __syncthreads();
  const int cpg = c / groups;
  for (int ch = tid; ch < c; ch += kVecThreads) {
    Moments m = merge_all<0>([&](int r) { return s_p[r * c + ch]; }, parts);
    m = merge_to_first(m, tid & 63, cpg);   // cpg consecutive lanes = one group
    if ((ch & (cpg - 1)) == 0) {
      if (chunks == 1) {   // a slab is the sample: nothing to hand over
        mean[n * groups + ch / cpg] = m.mean;
        rstd[n * groups + ch / cpg] = 1.0f / sqrtf(m.m2 / m.n + eps);
      } else ws[((size_t)n * groups + ch / cpg) * chunks + chunk] = m;
    }
  }
}

// (mean, rstd) of the triples of LANES lanes, as the prologues of the convolutions merge theirs: the mean first, as a difference to `first`, then the squares about it.
template <int LANES> __device__ __forceinline__ float2 merge_lanes(const Moments& t, float first, float eps) {
  const float n = lanes_sum<LANES>(t.n), inv = __builtin_amdgcn_rcpf(n);
  float d = t.n > 0.f ? t.mean - first : 0.f;   // an empty triple's mean has no meaning
  const float mid = lanes_sum<LANES>(t.n * d) * inv;
  d = t.n > 0.f ? d - mid : 0.f;
  const float s = lanes_sum<LANES>(t.n * d), rest = s * inv, q = lanes_sum<LANES>(fmaf(t.n * d, d, t.n > 0.f ? t.m2 : 0.f)) - s * rest;
  return make_float2(first + (mid + rest), inverse_deviation(q < 0.f ? 0.f : q, n, eps));   // (NaN stays NaN)
}

// Columns: a workgroup takes 64 bytes of every pixel of a sample, whole groups, and needs nothing from the others.  A thread sums the channels of
// its vector shifted by its first pixel, the lanes of a wavefront are merged as in the convolutions' epilogues, where they lie far from zero by their means' differences to one lane's (a lane has a few
// pixels: at 54x24, f16 of 37 +- 0.01, rstd was wrong by 2e-5, now 8e-8; us, before / now, f32 64 channels at 32x32 3.25 / 3.27, f16 512 at 17x23 4.50 / 4.53), the 16 wavefronts' triples of a
// group by 16 lanes.  Few compute units stream it, each bound by latency and conversions (four vectors in flight a thread: eight or sixteen are slower, as are 32 bytes
// a pixel), so it is for images of few pixels, where the launch that merges the triples of gn_stats_vec takes longer.
constexpr int kColThreads = 1024, kColVecs = 4;
template <typename T>
__global__ __launch_bounds__(kColThreads) void gn_stats_columns(const T* __restrict__ x, int pixels, int c, int groups, float eps, float* __restrict__ mean, float* __restrict__ rstd) {
  constexpr int V = Vec16<T>::N, VECS = kColVecs, U = 4, CH = VECS * V, WAVES = kColThreads / 64, ROWS = kColThreads / VECS;
  __shared__ RelMoments s_w[CH][WAVES];   // moments per (group, wavefront)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // workgroup id -> (sample, column); the ids of one XCD (id % 8) are neighbours: the columns of a 128-byte line come out of one L2
  const unsigned cols = c / CH, total = gridDim.x, per = total / 8, rem = total % 8, xcd = blockIdx.x % 8;
  const unsigned at = xcd * per + min(xcd, rem) + blockIdx.x / 8, n = at / cols, col = at % cols;
  const unsigned pitch = (unsigned)c * sizeof(T), sweep = ROWS * pitch, end = (unsigned)pixels * pitch;   // (a sample is below 2^31 bytes)
  const char* slab = reinterpret_cast<const char*>(x + (size_t)n * pixels * c) + col * (VECS * 16);
  const int row = tid / VECS, own = row < pixels ? (pixels - row + ROWS - 1) / ROWS : 0;
  unsigned off = (unsigned)row * pitch + (tid % VECS) * 16;
  LaneMoments<V> st[1];
  st[0].n = (float)own;
  {
    const Vec16<T> v = *reinterpret_cast<const Vec16<T>*>(slab + (off < end ? off : (tid % VECS) * 16));
#pragma unroll
    for (int j = 0; j < V; ++j) { st[0].shift[j] = to_float(v.v[j]); st[0].s[j] = 0.f; st[0].q[j] = 0.f; }
  }
  for (; off + (U - 1) * sweep < end; off += U * sweep) gn_accumulate<T, V, false, U, true>(slab, off, end, sweep, st[0].shift, st[0].s, st[0].q);
  if (off < end) gn_accumulate<T, V, true, U, true>(slab, off, end, sweep, st[0].shift, st[0].s, st[0].q);
  const int cpg = c / groups;
  RelMoments* const dst[1] = {&s_w[0][wave]};
  emit_vectors<VECS, V, true>(st, lane, 0, dst, cpg, WAVES, false);
  __syncthreads();
  const int own_groups = CH / cpg;
  if (tid < own_groups * WAVES) {   // (whole rows of 16 lanes)
    const int own_group = tid / WAVES, sub = tid % WAVES;
    const RelMoments lead = s_w[own_group][0];
    RelMoments w = s_w[own_group][sub];
    w.mean += w.about - lead.about;
    const float2 out = merge_lanes<WAVES>(Moments{w.n, w.mean, w.m2}, lead.mean, eps);
    if (sub == 0) {
      const int g = n * groups + col * own_groups + own_group;
      mean[g] = lead.about + out.x; rstd[g] = out.y;
    }
  }
}

// General path (any c, groups): grid = (chunks, groups, n); one workgroup walks
// the (pixel, channel-in-group) pairs of its slab.
template <typename T>
__global__ __launch_bounds__(256) void gn_partial_any(const T* __restrict__ x, int pixels, int c, int groups,
                                                      int chunk_pixels, Moments* __restrict__ ws) {
  __shared__ Moments s_m[256];
  const int tid = threadIdx.x;
  const int chunk = blockIdx.x, g = blockIdx.y, n = blockIdx.z, chunks = gridDim.x;
  const int cpg = c / groups;
  const int p0 = chunk * chunk_pixels, p1 = min(p0 + chunk_pixels, pixels);
  const long total = (long)(p1 - p0) * cpg;
  const T* base = x + ((size_t)n * pixels + p0) * c + (size_t)g * cpg;
  float shift = 0.f, s = 0.f, q = 0.f, cnt = 0.f;
  for (long i = tid; i < total; i += 256) {
    const float v = to_float(base[(size_t)(i / cpg) * c + (i % cpg)]);
    if (cnt == 0.f) shift = v;
    const float d = v - shift;
    s += d; q = fmaf(d, d, q); cnt += 1.f;
  }
  Moments m{0.f, 0.f, 0.f};
  if (cnt > 0.f) { m.n = cnt; const float ds = s / cnt; m.mean = shift + ds; m.m2 = fmaxf(q - s * ds, 0.f); }
  s_m[tid] = m;
  __syncthreads();
  for (int step = 128; step > 0; step >>= 1) {
    if (tid < step) s_m[tid] = merge(s_m[tid], s_m[tid + step]);
    __syncthreads();
  }
  if (tid == 0) ws[((size_t)n * groups + g) * chunks + chunk] = s_m[0];
}

// grid = n*groups workgroups of as many wavefronts as hold the row's triples, kFinLoads in a lane (up to 16; of rows of more than 4096 every lane takes
// more, reading them twice: sums about the mean of the first 4096 alone would cancel as many times over as the row is longer).  A wavefront
// takes the mean of its triples first, then the differences to it and their squares from the same registers; up to 256 triples that is the
// result, otherwise 16 lanes merge the wavefronts' triples the same way.  Bound by the launch, one trip to memory and the chain behind it: with
// pairwise merges, a reciprocal in each, and always 16 wavefronts, us of calls with one merge, before / now: ResBlock 256 -> 256 channels at 120x180 76.4 / 74.7,
// 128 -> 128 at 480x720 209.8 / 207.3, 256 -> 128 at 61x47 (two) 28.9 / 28.1.
constexpr int kFinThreads = 1024, kFinLoads = 4;
__device__ __forceinline__ float wave_sum(float v) { return swap_sum<32>(swap_sum<16>(lane_group_sum<16>(v))); }
__global__ __launch_bounds__(kFinThreads) void gn_finalize(const Moments* __restrict__ ws, int chunks, float eps,
                                                           float* __restrict__ mean, float* __restrict__ rstd) {
  constexpr int WAVES = kFinThreads / 64;
  constexpr float kUnit = 0x1p-20f;   // pixels are counted in it where they weigh a mean: the weighted sum of large means stays in range
  __shared__ Moments s_w[WAVES];
  const int ng = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
  const Moments* row = ws + (size_t)ng * chunks;
  // (an infinite mean stays one: what would be subtracted from it is left out)
  auto finite = [](float v) { return fabsf(v) < __builtin_inff() ? v : 0.f; };
  auto step = [&](const Moments& t, float about, float& weight, float& sum, float& squares) {   // an empty triple's mean has no meaning
    const float w = t.n * kUnit, d = t.n > 0.f ? t.mean - about : 0.f;
    weight += w; sum = fmaf(w, d, sum); squares += fmaf(t.n * d, d, t.n > 0.f ? t.m2 : 0.f);
  };
  Moments t[kFinLoads];
  auto fetch = [&](int i0) {
#pragma unroll
    for (int k = 0; k < kFinLoads; ++k) t[k] = row[min(i0 + k * nt, chunks - 1)];
#pragma unroll
    for (int k = 0; k < kFinLoads; ++k)
      if (i0 + k * nt >= chunks) t[k].n = 0.f;
  };
  float first = row[0].mean, w = 0.f, s = 0.f, q = 0.f;
  auto rest = [&](float about) {   // of a longer row, behind the triples at hand
    for (int i0 = tid + kFinLoads * nt; i0 - tid < chunks; i0 += kFinLoads * nt) {
      fetch(i0);
#pragma unroll
      for (int k = 0; k < kFinLoads; ++k) step(t[k], about, w, s, q);
    }
  };
  fetch(tid);
  first = finite(first);
#pragma unroll
  for (int k = 0; k < kFinLoads; ++k) step(t[k], first, w, s, q);
  if (chunks > kFinLoads * nt) {
    rest(first);
    fetch(tid);
  }
  w = wave_sum(w);
  const float mid = first + wave_sum(s) * (w > 0.f ? __builtin_amdgcn_rcpf(w) : 0.f), about = finite(mid);   // 1 ulp: what the roundings leave follows
  w = 0.f; s = 0.f; q = 0.f;
#pragma unroll
  for (int k = 0; k < kFinLoads; ++k) step(t[k], about, w, s, q);
  rest(about);
  auto close = [&](float all_w, float all_s, float all_q) -> Moments {
    const float ds = all_s * (all_w > 0.f ? __builtin_amdgcn_rcpf(all_w) : 0.f), m2 = all_q - all_s * (1.f / kUnit) * ds;
    return Moments{all_w * (1.f / kUnit), about + ds, m2 < 0.f ? 0.f : m2};   // (NaN stays NaN)
  };
  auto write = [&](const Moments& m) { mean[ng] = m.mean; rstd[ng] = inverse_deviation(m.m2, m.n, eps); };
  const Moments own = close(wave_sum(w), wave_sum(s), wave_sum(q));
  if (nt == 64) {
    if (tid == 0) write(own);
    return;
  }
  if ((tid & 63) == 0) s_w[tid >> 6] = own;
  __syncthreads();
  if (tid >= WAVES) return;
  static_assert(WAVES == 16, "one row of 16 lanes");
  Moments m = s_w[min(tid, nt / 64 - 1)];
  if (tid >= nt / 64) m.n = 0.f;
  const float head = finite(s_w[0].mean);
  w = 0.f; s = 0.f; q = 0.f;
  step(m, head, w, s, q);
  w = lane_group_sum<16>(w);
  const float at = head + lane_group_sum<16>(s) * __builtin_amdgcn_rcpf(w);
  s = 0.f; q = 0.f;
  float again = 0.f;
  step(m, finite(at), again, s, q);
  s = lane_group_sum<16>(s); q = lane_group_sum<16>(q);
  const float ds = s * __builtin_amdgcn_rcpf(w), m2 = q - s * (1.f / kUnit) * ds;
  if (tid == 0) write(Moments{w * (1.f / kUnit), finite(at) + ds, m2 < 0.f ? 0.f : m2});
}

int pick_chunks(int pixels, int c, int V, bool vec) {
  // vector path: <= 256 workgroups of 1024 threads per sample (one per compute unit, 128 KiB of loads in flight),
  // every one sweeping its slab at least 4 times; general path: <= 2048 slabs of >= 1024 pixels.
  // Never a function of the batch size: a sample's result must not depend on its neighbours.
  const int ppi = vec ? kVecThreads / (c / V) : 1;
  const int min_chunk = vec ? 4 * ppi : 1024;
  // A tensor of at most 16 sweeps (256 KiB a sample) stays with one workgroup: streaming it alone takes less than a launch that merges.
  if (vec && pixels <= 16 * ppi) return 1;
  int chunks = (pixels + min_chunk - 1) / min_chunk;
  const int cap = vec ? kVecMaxChunks : 2048;
  if (chunks > cap) chunks = cap;
  if (chunks < 1) chunks = 1;
  return chunks;
}

// Images of up to so many pixels take gn_stats_columns.  us, gn_stats_vec with its merge / columns, inputs from beyond the L2s: f16 256 channels two 61x47 8.7 / 8.0, 128 channels 68x68
// 8.7 / 8.6; past the line 60x90 of 512 9.0 / 12.7, 80x100 9.4 / 14.3; far below it 512 channels 17x23 take 4.9 in columns, 32x32 5.0, 45x60 8.7, f32 64 channels 32x32 4.3,
// where a merging launch alone is 2.3.  Groups of one 16-bit channel, eight chains of lane moves a lane, stay with gn_stats_vec where one workgroup streams the sample and no merge follows:
// 64 channels at 6x6 4.9 / 6.2, 32x32 5.8 / 6.9, 32 channels at 64x64 8.2 / 8.9; beyond, 64 at 48x48 10.6 / 8.3.  (Not a function of the batch: a sample's result must not depend on its
// neighbours.)
constexpr int kColPixels = 4096;

struct Plan { bool vec; int chunks; int chunk_pixels; bool columns; };

Plan make_plan(int x_dtype, int n, int h, int w, int c, int groups) {
  (void)n;
  const int V = x_dtype == WMDEC_F32 ? 4 : 8;
  const int pixels = h * w;
  const int cpg = c / groups;
  Plan p;
  const bool divisible = (c % V == 0) && (kVecThreads % (c / V) == 0) && c <= kVecThreads;
  p.vec = divisible && (cpg & (cpg - 1)) == 0 && cpg <= 64 && groups <= kVecMaxGroups;   // groups are runs of 2^k lanes in the channel reduction
  p.chunks = pick_chunks(pixels, c, V, p.vec);
  p.chunk_pixels = (pixels + p.chunks - 1) / p.chunks;
  if (p.vec) {
    const int ppi = kVecThreads / (c / V);
    p.chunk_pixels = ((p.chunk_pixels + ppi - 1) / ppi) * ppi;
  }
  p.chunks = (pixels + p.chunk_pixels - 1) / p.chunk_pixels;
  p.columns = p.vec && pixels <= kColPixels && c % (kColVecs * V) == 0 && cpg <= kColVecs * V && !(V == 8 && cpg == 1 && p.chunks == 1);
  return p;
}

}  // namespace

int launch_gn_finalize(const void* ws, int n_groups, int slots, float eps, float* mean, float* rstd, hipStream_t s) {
  const int waves = min(kFinThreads / 64, (slots + 64 * kFinLoads - 1) / (64 * kFinLoads));
  hipLaunchKernelGGL(gn_finalize, dim3((unsigned)n_groups), dim3((unsigned)(64 * waves)), 0, s, (const Moments*)ws, slots, eps, mean, rstd);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

// head of a caller's workspace, four bytes a sample: nothing is kept there any more, its size is what callers have passed
size_t gn_stats_ticket_bytes(int n) { return ((size_t)n * sizeof(unsigned) + 255) / 256 * 256; }

size_t gn_stats_moments_bytes(int n, int groups) {
  // upper bound over shapes and dtypes: 2048 chunks per (sample, group)
  return (size_t)n * groups * 2048 * sizeof(Moments);
}

int gn_stats_num_launches(int x_dtype, int h, int w, int c, int groups) {
  const Plan p = make_plan(x_dtype, 1, h, w, c, groups);
  return p.columns || (p.vec && p.chunks == 1) ? 1 : 2;
}

const char* gn_stats_label(int x_dtype, int h, int w, int c, int groups) {
  const Plan p = make_plan(x_dtype, 1, h, w, c, groups);
  return p.columns ? "gn_stats_columns" : p.vec ? "gn_stats_vec" : "gn_partial_any";
}

static int launch_general(const void* x, int x_dtype, int n, int pixels, int c, int groups, int slabs, int slab_pixels, float eps,
                          float* mean, float* rstd, Moments* wsm, hipStream_t s) {
  dim3 grid((unsigned)slabs, (unsigned)groups, (unsigned)n);
  switch (x_dtype) {
    case WMDEC_F32: hipLaunchKernelGGL(gn_partial_any<float>, grid, dim3(256), 0, s, (const float*)x, pixels, c, groups, slab_pixels, wsm); break;
    case WMDEC_BF16: hipLaunchKernelGGL(gn_partial_any<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)x, pixels, c, groups, slab_pixels, wsm); break;
    default: hipLaunchKernelGGL(gn_partial_any<f16_t>, grid, dim3(256), 0, s, (const f16_t*)x, pixels, c, groups, slab_pixels, wsm); break;
  }
  WMDEC_HIP(hipGetLastError());
  return launch_gn_finalize(wsm, n * groups, slabs, eps, mean, rstd, s);
}

int launch_gn_stats(const void* x, int x_dtype, int n, int h, int w, int c, int groups, float eps,
                    float* mean, float* rstd, void* moments, size_t moments_bytes, hipStream_t s) {
  const Plan p = make_plan(x_dtype, n, h, w, c, groups);
  WMDEC_REQUIRE(moments && moments_bytes >= (size_t)n * groups * p.chunks * sizeof(Moments), WMDEC_ERR_WORKSPACE,
                "gn_stats: workspace of %zu bytes is too small", moments_bytes);
  Moments* wsm = (Moments*)moments;
  const int pixels = h * w;
  if (p.columns) {
    auto launch = [&](auto t) {
      using T = decltype(t);
      hipLaunchKernelGGL(gn_stats_columns<T>, dim3((unsigned)(c / (kColVecs * Vec16<T>::N) * n)), dim3(kColThreads), 0, s, (const T*)x, pixels, c, groups, eps, mean, rstd);
    };
    if (x_dtype == WMDEC_F32) launch(float{});
    else if (x_dtype == WMDEC_BF16) launch(bf16_t{});
    else launch(f16_t{});
    WMDEC_HIP(hipGetLastError());
    return WMDEC_OK;
  }
  if (p.vec) {
    dim3 grid((unsigned)p.chunks, (unsigned)n);
    switch (x_dtype) {
      case WMDEC_F32: hipLaunchKernelGGL(gn_stats_vec<float>, grid, dim3(kVecThreads), 0, s, (const float*)x, pixels, c, groups, p.chunk_pixels, wsm, eps, mean, rstd); break;
      case WMDEC_BF16: hipLaunchKernelGGL(gn_stats_vec<bf16_t>, grid, dim3(kVecThreads), 0, s, (const bf16_t*)x, pixels, c, groups, p.chunk_pixels, wsm, eps, mean, rstd); break;
      default: hipLaunchKernelGGL(gn_stats_vec<f16_t>, grid, dim3(kVecThreads), 0, s, (const f16_t*)x, pixels, c, groups, p.chunk_pixels, wsm, eps, mean, rstd); break;
    }
    WMDEC_HIP(hipGetLastError());
    if (p.chunks > 1) return launch_gn_finalize(wsm, n * groups, p.chunks, eps, mean, rstd, s);
    return WMDEC_OK;
  }
  return launch_general(x, x_dtype, n, pixels, c, groups, p.chunks, p.chunk_pixels, eps, mean, rstd, wsm, s);
}

// The general path in at most max_slabs slabs, for callers whose workspace holds that many triples per (sample, group).
int launch_gn_stats_small_ws(const void* x, int x_dtype, int n, int h, int w, int c, int groups, float eps, float* mean,
                             float* rstd, void* moments, int max_slabs, hipStream_t s) {
  const int pixels = h * w;
  const int slabs = max(1, min(max_slabs, (pixels + 63) / 64));
  const int slab_pixels = (pixels + slabs - 1) / slabs;
  return launch_general(x, x_dtype, n, pixels, c, groups, (pixels + slab_pixels - 1) / slab_pixels, slab_pixels, eps, mean, rstd, (Moments*)moments, s);
}

// ---- the variant for callers that cannot allocate: the workspace is a file-scope device array
constexpr size_t kStaticTicketBytes = 256;                 // a head of four bytes a sample, as in a caller's workspace: the interface takes at most 64
constexpr size_t kStaticMomentsBytes = (size_t)1 << 20;    // 87381 moment triples
static __device__ __align__(256) unsigned char scratch[kStaticTicketBytes + kStaticMomentsBytes];

size_t gn_stats_static_capacity_bytes() { return kStaticMomentsBytes; }

int launch_gn_stats_static(const void* x, int x_dtype, int n, int h, int w, int c, int groups, float eps,
                           float* mean, float* rstd, hipStream_t s) {
  const Plan p = make_plan(x_dtype, n, h, w, c, groups);
  const size_t need = (size_t)n * groups * p.chunks * sizeof(Moments);
  WMDEC_REQUIRE((size_t)n * sizeof(unsigned) <= kStaticTicketBytes && need <= kStaticMomentsBytes, WMDEC_ERR_WORKSPACE,
                "gn_stats_noalloc: %d samples x %d groups x %d slabs need %zu bytes of built-in scratch, the limit is %zu "
                "(and 64 samples); use wmdec_gn_stats with a workspace", n, groups, p.chunks, need, kStaticMomentsBytes);
  // every device holds its own copy of the array at its own address: resolve it once per device, with that device current
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static unsigned char* dev_scratch[kMaxDevices] = {};
  int dev = -1;
  WMDEC_HIP(hipGetDevice(&dev));
  WMDEC_REQUIRE(dev >= 0 && dev < kMaxDevices, WMDEC_ERR_UNSUPPORTED, "gn_stats_noalloc: device index %d not supported", dev);
  unsigned char* ptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!dev_scratch[dev]) {
      void* sym = nullptr;
      WMDEC_HIP(hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)));
      dev_scratch[dev] = (unsigned char*)sym;
    }
    ptr = dev_scratch[dev];
  }
  // (the array keeps what the last call left; the moment slots are all written before they are read)
  return launch_gn_stats(x, x_dtype, n, h, w, c, groups, eps, mean, rstd, ptr + kStaticTicketBytes, kStaticMomentsBytes, s);
}

}  // namespace wmdec
