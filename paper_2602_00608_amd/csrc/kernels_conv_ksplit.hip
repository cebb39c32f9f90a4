// 3x3 convolution for small images and for fp32: the contraction is split over the wavefronts of a workgroup.
//
// Same GEMM view, staging and epilogue semantics as kernels_conv_mfma.hip (GroupNorm scale/shift and SiLU applied once
// per staged element, zeros outside the image, bias / residual / folded 1x1 shortcut, moments of the stored output), for
// layers that leave most compute units empty when every workgroup takes 128 pixels x 128 channels: there a wavefront is
// alone on its SIMD and walks the whole contraction (4608 products deep at 512 channels) by itself, so the launch takes
// the latency of one such walk however small the image is.  Here a workgroup takes a small tile (32 or 64 pixels x 32 to
// 128 channels) with eight wavefronts (two or four for the 32-channel tiles), WN of them side by side in the channels and WK in the contraction: a round stages
// 16 * WK input channels, wavefront wk multiplies its own 16 of them with all nine taps, and the WK partial sums
// of an output are added in a fixed order through LDS at the end.  What bounds it is the activation on the load path
// (a staged element serves only the tile's channels) and the fixed parts of a launch, not the matrix pipe.
//
// The operands of the MFMAs are exchanged against the other kernel (A = weights, B = pixels): a lane then holds four
// consecutive channels of one pixel, so that the partial sums move through LDS as 16-byte vectors.
//
// fp32 runs on the 32x32x2 fp32 MFMAs (operands and sums in fp32): the eight channels that a lane holds of a fragment
// are eight MFMAs, each with one channel of either half of the 16.
#include <stdio.h>

#include <mutex>

#include "conv_device.hpp"

namespace wmdec {
namespace {

// LDS layout of a staged round: pixel stride 32 * WK + 16 bytes (16-bit types; 64 * WK + 16 for fp32), an odd multiple
// of 16 bytes, so that the 16 lanes the LDS serves per cycle fall on distinct banks; the row stride is congruent to
// TW pixel strides mod 256, so that lanes i and i + 16 of an M tile are a multiple of 256 bytes apart also
// where the tile crosses a row of the patch (any other distance costs a second pass).
template <typename T> constexpr int pixel_bytes(int wk) { return 16 * wk * (int)sizeof(T) + 16; }
template <typename T> constexpr int row_bytes(int tw, int wk) { return tw * pixel_bytes<T>(wk) + (2 * pixel_bytes<T>(wk) + 255) / 256 * 256; }
template <typename T> constexpr int stage_bytes(int th, int tw, int wk) { return (th + 2) * row_bytes<T>(tw, wk) + pixel_bytes<T>(wk); }
// floats of a pixel's row in the reduction: + 4 spreads the pixels over the banks
constexpr int reduce_row(int tn) { return tn + 4; }

// fp32: the shift is subtracted first, so that |mean| >> std does not cancel
__device__ __forceinline__ float activate_f32(float v, float mu, float2 ab, bool silu) {
  const float t = fmaf(v - mu, ab.x, ab.y);
  return silu ? silu_f(t) : t;
}

// One fragment: 32 rows x 16 channels, 8 channels of a row per lane.
template <typename T> struct Frag { u32x4 v[sizeof(T) / 2]; };

template <typename T> __device__ __forceinline__ f32x16 mma_frag(const Frag<T>& a, const Frag<T>& b, f32x16 c) {
  if constexpr (sizeof(T) == 2) {
    return Mma<T>::m32(a.v[0], b.v[0], c);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const f32x4 av = __builtin_bit_cast(f32x4, a.v[j / 4]), bv = __builtin_bit_cast(f32x4, b.v[j / 4]);
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j % 4], bv[j % 4], c, 0, 0, 0);
    }
    return c;
  }
}

// OCC: wavefronts per SIMD the register budget is sized for.  AHEAD: rounds the weight fragments travel ahead of their MFMAs (1 or 2; a round is nine fragments per channel tile).
template <typename T, int TH, int TW, int NI, int WN, int WK, int AHEAD, int OCC, int ACT>
__global__ __launch_bounds__(64 * WN * WK, OCC) void conv_ksplit_kernel(MfmaParams p, int y_f32) {
  constexpr int NW = WN * WK, NT = 64 * NW;
  constexpr int M = TH * TW, MI = M / 32, TN = WN * NI * 32;
  constexpr int ES = (int)sizeof(T), EPV = 16 / ES;          // element size, elements of a 16-byte vector
  constexpr int KC = 16 * WK, VPP = KC / EPV;                // channels of a round, vectors of a pixel in a round
  constexpr int HW_ = TW + 2, HH_ = TH + 2, HP = HW_ * HH_;
  constexpr int NV = (HP * VPP + NT - 1) / NT;
  constexpr int PSB = pixel_bytes<T>(WK), ROWB = row_bytes<T>(TW, WK), BUFB = stage_bytes<T>(TH, TW, WK);
  constexpr int SPARE = HH_ * ROWB;
  constexpr int FB = 512 * ES, FV = ES / 2;                  // bytes of a weight fragment, 16-byte vectors of it per lane
  constexpr int STEPS = 9, WORDS = NV * 4;
  static_assert(M % 32 == 0 && NT % VPP == 0 && (AHEAD == 1 || AHEAD == 2), "tile shape");

  extern __shared__ __align__(16) unsigned char smem[];
  float2* s_ab = reinterpret_cast<float2*>(smem + 2 * BUFB);       // [cin] (scale, shift)
  float* s_mu = reinterpret_cast<float*>(s_ab + p.cin);            // [cin] mean per channel (fp32 only), read as 16-byte vectors
  float2* s_stat = reinterpret_cast<float2*>(s_mu + (ES == 4 ? p.cin : 0));   // [groups] (mean, rstd): any number, so it comes last

  fetch_arguments<sizeof(MfmaParams) + sizeof(int)>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WN, wk = wave / WN;
  const int lm = lane & 31, lk = lane >> 5;

  const WorkTile wt = workgroup_tile(p);
  if (__builtin_expect(carries_weights(p), 0)) { warm_weights(p.next, p.total, NW, wave, lane); return; }
  const int nt = wt.nt, n = wt.n;
  const int ty0 = wt.y * TH, tx0 = wt.x * TW;
  const int co0 = nt * TN;
  const int rounds = p.cin / KC;

  // ---- weight fragments: round r, tap t of this wavefront is fragment (t, r * WK + wk); past the last round the lane
  // offset points behind the blob, which reads zeros without touching memory
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, p.w_bytes, 0x00020000);
  const int kk_stride = p.cout_blocks * FB, tap_stride = p.cin_blocks * kk_stride;
  const int wcol = ((co0 >> 5) + wn * NI) * FB + wk * kk_stride;
  const int lane_off = lane * 8 * ES;
  Frag<T> bq[AHEAD][STEPS][NI];
  auto load_weights = [&](Frag<T>& f, int r, int tap, int ni) {
    const int off = wcol + min(r, rounds - 1) * WK * kk_stride + tap * tap_stride + ni * FB;
    const int lo = r < rounds ? lane_off : 0x7fff0000;
#pragma unroll
    for (int k = 0; k < FV; ++k) f.v[k] = load_fragment(wrsrc, lo + 16 * k, off);
  };

  // The first rounds' weights, behind the moments and the input, which are needed first: loads return in order.
  auto first_weights = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < AHEAD; ++r)
#pragma unroll
      for (int t = 0; t < STEPS; ++t)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) load_weights(bq[r][t][ni], r, t, ni);
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- staging: a thread owns NV (pixel, channel vector) pairs of the halo patch; the channel vector is the same for all
  const int cvec = tid % VPP;
  int src_pix[NV], dst_off[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int hp = (tid + i * NT) / VPP;
    const int hy = hp / HW_, hx = hp % HW_;
    const int gy = ty0 + hy - 1, gx = tx0 + hx - 1;
    const bool in_patch = hp < HP, inside = in_patch & ((unsigned)gy < (unsigned)p.h) & ((unsigned)gx < (unsigned)p.w_out);   // (no branches)
    src_pix[i] = inside ? gy * p.w_out + gx : 0;
    // a vector outside the image is loaded from pixel 0 and stored to the spare slot; its real slot is zeroed here, once
    const int at = hy * ROWB + hx * PSB;
    dst_off[i] = (inside ? at : SPARE) + cvec * 16;
    if (in_patch & !inside) {
      *reinterpret_cast<u32x4*>(smem + at + cvec * 16) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(smem + BUFB + at + cvec * 16) = u32x4{0u, 0u, 0u, 0u};
    }
  }
  u32x4 raw[2][NV];   // two rounds in flight: round r lives in raw[r & 1]
  auto issue = [&](u32x4 (&dst)[NV], const void* x, int cin, int r) {
    const char* base = reinterpret_cast<const char*>(x) + ((size_t)n * p.h * p.w_out * cin + (size_t)r * KC) * ES;
#pragma unroll
    for (int i = 0; i < NV; ++i) dst[i] = *reinterpret_cast<const u32x4*>(base + (unsigned)((src_pix[i] * cin + cvec * EPV) * ES));
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // byte offset of this lane's pixel in each of its M tiles (tap (0,0)), in this wavefront's 16 channels
  int p_off[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    const int px = mi * 32 + lm;
    p_off[mi] = (px / TW) * ROWB + (px % TW) * PSB + wk * 16 * ES + lk * 8 * ES;
  }
  auto load_pixels = [&](Frag<T>& f, const unsigned char* buf, int mi, int tap_off) {
#pragma unroll
    for (int k = 0; k < FV; ++k) f.v[k] = *reinterpret_cast<const u32x4*>(buf + p_off[mi] + tap_off + 16 * k);
  };

  // ---- folded 1x1 shortcut: W2 * x2 over the tile's own pixels (centre tap), taken as stored, into the same accumulators
  if (p.x2) {
    const int rounds2 = p.cin2 / KC;
    const __amdgpu_buffer_rsrc_t wrsrc2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w2), 0, p.w2_bytes, 0x00020000);
    Frag<T> b2[2][NI];
    auto load2 = [&](Frag<T> (&f)[NI], int r) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int k = 0; k < FV; ++k) f[ni].v[k] = load_fragment(wrsrc2, lane_off + 16 * k, wcol + min(r, rounds2 - 1) * WK * kk_stride + ni * FB);
    };
    load2(b2[0], 0); load2(b2[1], 1);
    issue(raw[0], p.x2, p.cin2, 0);
    issue(raw[1], p.x2, p.cin2, min(1, rounds2 - 1));
    auto round2 = [&](auto par_c, int r) {
      constexpr int P = decltype(par_c)::value;
      unsigned char* buf = smem + P * BUFB;
#pragma unroll
      for (int i = 0; i < NV; ++i) *reinterpret_cast<u32x4*>(buf + dst_off[i]) = raw[P][i];
      if (r + 2 < rounds2) issue(raw[P], p.x2, p.cin2, r + 2);
      __syncthreads();   // (the other buffer is rewritten only behind the next barrier)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        Frag<T> af;
        load_pixels(af, buf, mi, ROWB + PSB);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = mma_frag<T>(b2[P][ni], af, acc[mi][ni]);
      }
      load2(b2[P], r + 2);
    };
    for (int r = 0; r < rounds2; r += 2) {
      round2(std::integral_constant<int, 0>{}, r);
      if (r + 1 < rounds2) round2(std::integral_constant<int, 1>{}, r + 1);
    }
  }

  issue(raw[0], p.x, p.cin, 0);
  issue(raw[1], p.x, p.cin, min(1, rounds - 1));

  // ---- mean and rstd of the groups
  constexpr int PRE = 2;                             // table entries of a thread whose gamma and beta are requested together with the moments
  float gpre[PRE] = {}, bpre[PRE] = {};
  int group[PRE] = {};
  if constexpr (ACT > 0) {
    constexpr int TPG = 16;                          // lanes that merge the triples of a group
#pragma unroll
    for (int j = 0; j < PRE; ++j) {
      const int c = min(tid + j * NT, p.cin - 1);
      gpre[j] = p.gamma[c]; bpre[j] = p.beta[c];
      group[j] = quotient_of(c, p.cpg_in, p.inv_cpg_in);
    }
    if (p.rows_in) {
      merge_sample<TPG, NT>(p.rows_in + (size_t)n * p.groups * p.rows_in_count, p.groups, p.rows_in_count, tid, p.eps, s_stat);   // (at most 128 triples per group)
    } else {
      for (int g = tid; g < p.groups; g += NT) s_stat[g] = make_float2(p.mean[n * p.groups + g], p.rstd[n * p.groups + g]);
    }
  }
  first_weights();
  // ---- scale/shift table.  16-bit types: (a, b) = k * (gamma * rstd, beta - mean * gamma * rstd), k = -log2(e) with
  // SiLU (see silu_from_scaled).  fp32: (gamma * rstd, beta), the mean stays apart.
  if constexpr (ACT > 0) {
    __syncthreads();
    const float k = (ES == 2 && ACT == 2) ? -1.4426950408889634f : 1.0f;
    auto entry = [&](int c, int g, float ga, float be) {
      const float2 st = s_stat[g];
      const float a = ga * st.y;
      s_ab[c] = ES == 2 ? make_float2(k * a, k * (be - st.x * a)) : make_float2(a, be);
      if constexpr (ES == 4) s_mu[c] = st.x;
    };
#pragma unroll
    for (int j = 0; j < PRE; ++j)
      if (tid + j * NT < p.cin) entry(tid + j * NT, group[j], gpre[j], bpre[j]);
    for (int c = tid + PRE * NT; c < p.cin; c += NT) entry(c, quotient_of(c, p.cpg_in, p.inv_cpg_in), p.gamma[c], p.beta[c]);
  }
  __syncthreads();

  // word w (0..3) of a staged vector of the round that starts at channel c0
  struct Table { f32x4 e[4]; f32x4 mu; };
  auto read_table = [&](int c0) -> Table {
    Table t{};
    if constexpr (ACT > 0) {
      const f32x4* tab = reinterpret_cast<const f32x4*>(s_ab + c0 + cvec * EPV);
#pragma unroll
      for (int k = 0; k < EPV / 2; ++k) t.e[k] = tab[k];
      if constexpr (ES == 4) t.mu = *reinterpret_cast<const f32x4*>(s_mu + c0 + cvec * EPV);
    }
    return t;
  };
  auto activate = [&](uint32_t wv, const Table& t, int w) -> uint32_t {
    if constexpr (ES == 2) return activate_word<T, ACT, true>(wv, t.e[w]);
    else if constexpr (ACT == 0) return wv;
    else return __builtin_bit_cast(uint32_t, activate_f32(__builtin_bit_cast(float, wv), t.mu[w], make_float2(t.e[w / 2][(w % 2) * 2], t.e[w / 2][(w % 2) * 2 + 1]), ACT == 2));
  };

  {
    const Table t = read_table(0);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      u32x4 v;
#pragma unroll
      for (int w = 0; w < 4; ++w) v[w] = activate(raw[0][i][w], t, w);
      *reinterpret_cast<u32x4*>(smem + dst_off[i]) = v;
    }
    if (rounds > 2) issue(raw[0], p.x, p.cin, 2);
  }
  __syncthreads();

  // ---- one round: nine k-steps on the staged buffer, the activation of the next round sliced in between, weight
  // fragments refreshed in place AHEAD rounds ahead.  MORE: a further round follows.
  auto round = [&](auto par_c, auto more_c, int r) {
    constexpr int P = decltype(par_c)::value;
    constexpr bool MORE = decltype(more_c)::value;
    const unsigned char* buf = smem + P * BUFB;
    unsigned char* nbuf = smem + (1 - P) * BUFB;
    constexpr int W = P % AHEAD;
    Table tab{};
    if constexpr (MORE) tab = read_table((r + 1) * KC);
    Frag<T> af[2][MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) load_pixels(af[0][mi], buf, mi, 0);
    static_for<STEPS>([&](auto s_c) {
      constexpr int s = decltype(s_c)::value;
      if constexpr (s + 1 < STEPS) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) load_pixels(af[(s + 1) & 1][mi], buf, mi, ((s + 1) / 3) * ROWB + ((s + 1) % 3) * PSB);
      }
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = mma_frag<T>(bq[W][s][ni], af[s & 1][mi], acc[mi][ni]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) load_weights(bq[W][s][ni], r + AHEAD, s, ni);
      if constexpr (MORE) {
        constexpr int w0 = s * WORDS / STEPS, w1 = (s + 1) * WORDS / STEPS;
        static_for<w1 - w0>([&](auto k_c) {
          constexpr int wi = w0 + decltype(k_c)::value, i = wi / 4, w = wi % 4;
          raw[1 - P][i][w] = activate(raw[1 - P][i][w], tab, w);
          if constexpr (w == 3) *reinterpret_cast<u32x4*>(nbuf + dst_off[i]) = raw[1 - P][i];
        });
      }
      __builtin_amdgcn_sched_barrier(0);   // keeps the refreshed fragments' loads here instead of at their next use
    });
    if constexpr (MORE) {
      if (r + 3 < rounds) issue(raw[1 - P], p.x, p.cin, r + 3);
    }
    __syncthreads();
  };
  {
    const std::integral_constant<int, 0> even{};
    const std::integral_constant<int, 1> odd{};
    int r = 0;
    for (; r + 2 < rounds; r += 2) { round(even, std::true_type{}, r); round(odd, std::true_type{}, r + 1); }
    if (r + 1 < rounds) { round(even, std::true_type{}, r); round(odd, std::false_type{}, r + 1); }
    else round(even, std::false_type{}, r);
  }

  // ---- the WK partial sums of every output, added in wavefront order
  constexpr int RR = reduce_row(TN);
  float* red = reinterpret_cast<float*>(smem);                         // [WK][M][RR]
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(red + (size_t)(wk * M + mi * 32 + lm) * RR + (wn * NI + ni) * 32 + 8 * q + 4 * lk) =
            f32x4{acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2], acc[mi][ni][4 * q + 3]};
  constexpr int C4 = TN / 4, NJ = M * C4 / NT;                         // four-channel vectors of a pixel, per thread
  static_assert(NT % C4 == 0 && C4 <= 64 && NJ * NT == M * C4, "a thread keeps its four channels, all threads as many");
  const int c4 = tid % C4, co = co0 + c4 * 4;
  const T* rin = p.res ? reinterpret_cast<const T*>(p.res) + (size_t)n * p.h * p.w_out * p.cout : nullptr;
  int out_off[NJ];      // element offset of this thread's vectors in the sample (-1: outside the image)
  uint32_t rv[NJ][ES];  // residual vectors, requested before the partial sums are complete (clamped addresses)
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int px = tid / C4 + j * (NT / C4);
    const int oy = ty0 + px / TW, ox = tx0 + px % TW;
    out_off[j] = oy < p.h && ox < p.w_out ? (oy * p.w_out + ox) * p.cout + co : -1;
#pragma unroll
    for (int e = 0; e < ES; ++e) rv[j][e] = 0u;
    if (rin) {
      const T* src = rin + max(out_off[j], 0);
      if constexpr (ES == 4) {
        const u32x4 t = *reinterpret_cast<const u32x4*>(src);
#pragma unroll
        for (int e = 0; e < 4; ++e) rv[j][e] = t[e];
      } else {
        const u32x2 t = *reinterpret_cast<const u32x2*>(src);
        rv[j][0] = t.x; rv[j][1] = t.y;
      }
    }
  }
  f32x4 bv = f32x4{0.f, 0.f, 0.f, 0.f};
  if (p.bias) bv = f32x4{p.bias[co], p.bias[co + 1], p.bias[co + 2], p.bias[co + 3]};
  if (p.bias2) bv += f32x4{p.bias2[co], p.bias2[co + 1], p.bias2[co + 2], p.bias2[co + 3]};
  __syncthreads();
  const size_t sample = (size_t)n * p.h * p.w_out * p.cout;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int px = tid / C4 + j * (NT / C4);
    float* own = red + (size_t)px * RR + c4 * 4;
    f32x4 v = *reinterpret_cast<const f32x4*>(own);
#pragma unroll
    for (int k = 1; k < WK; ++k) v += *reinterpret_cast<const f32x4*>(red + (size_t)(k * M + px) * RR + c4 * 4);
    v += bv;
    if constexpr (ES == 4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += __builtin_bit_cast(float, rv[j][e]);
    } else {
      v += f32x4{unpack_lo<T>(rv[j][0]), unpack_hi<T>(rv[j][0]), unpack_lo<T>(rv[j][1]), unpack_hi<T>(rv[j][1])};
    }
    if (ES == 4 || y_f32) {
      if (out_off[j] >= 0) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.y) + sample + out_off[j]) = v;
    } else if constexpr (ES == 2) {
      const u32x2 t = u32x2{pack2<T>(v[0], v[1]), pack2<T>(v[2], v[3])};
      if (out_off[j] >= 0) *reinterpret_cast<u32x2*>(reinterpret_cast<T*>(p.y) + sample + out_off[j]) = t;
      v = f32x4{unpack_lo<T>(t.x), unpack_hi<T>(t.x), unpack_lo<T>(t.y), unpack_hi<T>(t.y)};   // moments of what is stored
    }
    if (p.stats) *reinterpret_cast<f32x4*>(own) = v;
  }
  // ---- moments of the stored values, one triple per (group, 4x8 block of pixels) whatever the tile, in an order that
  // depends on neither the tile nor the batch: a lane takes one channel of two rows of the block, the lane 32 further the
  // other two, and the channels of a group are consecutive lanes.  (One lane walking all 32 pixels held the launch up for
  // 0.8 us more at 17x23.)
  if (p.stats) {
    __syncthreads();
    constexpr int BX = TW / 8;
    static_assert(TH == 4 && TW % 8 == 0 && TN % 32 == 0, "blocks of 4 x 8 pixels");
    const int half = lane >> 5, blocks_x = (p.w_out + 7) / 8;
    with_group_size(p.stats_cpg, [&](auto cpg_c) __attribute__((always_inline)) {
      constexpr int CPG = decltype(cpg_c)::value;
      for (int i = wave; i < BX * (TN / 32); i += NW) {   // (uniform: a wavefront takes 32 channels of a block)
        const int b = i / (TN / 32), c = i % (TN / 32) * 32, x0 = tx0 + 8 * b;
        const int rows = min(4, p.h - ty0), cols = min(8, p.w_out - x0);
        if (cols <= 0) continue;
        Moments* dst = p.stats + (size_t)(n * p.stats_groups + (co0 + c) / CPG) * p.stats_slots + (ty0 / 4) * blocks_x + x0 / 8;
        const float* src = red + (size_t)(8 * b) * RR + c + lm;
        const Sums own = two_row_sums<8, TW * RR, RR>(src + 2 * half * TW * RR, src[0], rows - 2 * half, cols);
        const Moments m = merge_channels<CPG>(block_moments(Sums{swap_sum<32>(own.s), swap_sum<32>(own.q)}, src[0], rows, cols));
        if (half == 0 && lm % CPG == 0) dst[lm / CPG * p.stats_slots] = m;
      }
    });
  }
}

// triples per (sample, group): one per 4x8 block of pixels
int ksplit_slots(const ConvArgs& a) { return ((a.h + 3) / 4) * ((a.w + 7) / 8); }

template <typename T, int TH, int TW, int NI, int WN, int WK, int AHEAD, int OCC, int ACT>
int launch_act(const ConvArgs& a, hipStream_t s) {
  constexpr int TN = WN * NI * 32, NT = 64 * WN * WK, KC = 16 * WK;
  MfmaParams p = conv_params(a, TH, TW, TN, 1, a.h, a.w);
  p.stats_slots = ksplit_slots(a);
  const int rc = check_hand_over(p);
  if (rc != WMDEC_OK) return rc;
  p.w = a.wt; p.w_bytes = (int)(packed_elems(9, a.cout, a.cin) * sizeof(T));
  WMDEC_REQUIRE(a.cin % KC == 0 && a.cout % TN == 0 && !a.rows_out, WMDEC_ERR_UNSUPPORTED, "conv_ksplit: channels do not fit the tile");
  if (a.x2) {
    WMDEC_REQUIRE(a.w2 && a.cin2 > 0 && a.cin2 % KC == 0, WMDEC_ERR_UNSUPPORTED, "conv_ksplit: shortcut channels do not fit the tile");
    p.x2 = a.x2; p.w2 = a.w2; p.bias2 = a.bias2; p.cin2 = a.cin2;
    p.w2_bytes = (int)(packed_elems(1, a.cout, a.cin2) * sizeof(T));
  }
  size_t smem = (size_t)2 * stage_bytes<T>(TH, TW, WK) + (size_t)(a.cin + a.groups) * sizeof(float2) + (sizeof(T) == 4 ? (size_t)a.cin * sizeof(float) : 0);
  const size_t red = (size_t)WK * TH * TW * reduce_row(TN) * sizeof(float);
  if (smem < red) smem = red;
  constexpr int kMaxLds = 160 * 1024;
  WMDEC_REQUIRE(smem <= kMaxLds, WMDEC_ERR_UNSUPPORTED, "conv_ksplit: %zu bytes of LDS needed", smem);
  void (*kern)(MfmaParams, int) = conv_ksplit_kernel<T, TH, TW, NI, WN, WK, AHEAD, OCC, ACT>;
  static std::once_flag attr_once;
  hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds); });
  WMDEC_HIP(attr_err);
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.total + warm_groups(p.next, WN * WK))), dim3(NT), smem, s, p, a.y_dtype == WMDEC_F32 ? 1 : 0);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

template <typename T, int TH, int TW, int NI, int WN, int WK, int AHEAD, int OCC>
int launch_tile(const ConvArgs& a, hipStream_t s) {
  if (!a.mean && !a.rows_in) return launch_act<T, TH, TW, NI, WN, WK, AHEAD, OCC, 0>(a, s);
  return a.silu ? launch_act<T, TH, TW, NI, WN, WK, AHEAD, OCC, 2>(a, s) : launch_act<T, TH, TW, NI, WN, WK, AHEAD, OCC, 1>(a, s);
}

// Tiles of the 16-bit launches (4 rows high, WK = 4 everywhere: the order in which an output's products are added, and
// with it a frame's bits, depends neither on the tile nor on the batch, so the tile may follow the workgroups of the whole
// launch).  The smallest tile whose workgroups fit one round of the compute units wins; measured on 512 -> 512 layers, us,
// in the order K32x32, K32x64, K64x64, K64x128: 17x23 8.6 / 8.5 / 12.2 / 16.3; 32x32 12.9 / 11.5 / 12.3 / 16.4; 34x46 21.0 / 16.8 / 14.5 / 16.5; two samples of it 34.1 / 32.8 / 28.2 / 21.3.
enum KsplitTile { K32x32 = 0, K32x64, K64x64, K64x128 };
KsplitTile pick_ksplit_tile(const ConvArgs& a) {
  const long b8 = (long)((a.h + 3) / 4) * ((a.w + 7) / 8) * a.n, b16 = (long)((a.h + 3) / 4) * ((a.w + 15) / 16) * a.n;
  if (b8 * (a.cout / 32) <= 256) return K32x32;
  if (b8 * (a.cout / 64) <= 256) return K32x64;
  if (b16 * (a.cout / 64) <= 256 || a.cout % 128 != 0) return K64x64;
  return K64x128;
}

template <typename T> int launch_16bit(const ConvArgs& a, hipStream_t s) {
  switch (pick_ksplit_tile(a)) {
    case K32x32: return launch_tile<T, 4, 8, 1, 1, 4, 2, 2>(a, s);
    case K32x64: return launch_tile<T, 4, 8, 1, 2, 4, 1, 4>(a, s);
    case K64x64: return launch_tile<T, 4, 16, 1, 2, 4, 2, 2>(a, s);
    default: return launch_tile<T, 4, 16, 2, 2, 4, 1, 2>(a, s);
  }
}

// Batches past one round of the largest tile above take the 128 x 128 form that reproduces this kernel's sums and moments
// (launch_conv_quarters): a weight fragment then feeds four MFMAs instead of two.  Its tiles are eight rows high, so
// images that leave much of them empty stay here (ratio of the two tile counts below 5 / 3).  ResBlocks in us, this kernel /
// that form: 512 channels 17x23 6 samples 56.5 / 77.8, 8 samples 83.6 / 79.6; 32x32 4: 62.1 / 77.5, 6: 93.2 / 85.1, 16: 195.6 /
// 169.0; 34x46 2: 58.3 / 78.9, 3: 90.8 / 82.8, 8: 182.3 / 157.2; 256 channels 46x60 2: 41.8 / 54.7, 3: 64.1 / 55.9, 16: 185.2 /
// 142.8.  (The ordinary 128 x 128 tile, whose order of summation is another, takes 4 to 8 % less than that form: it fits
// three workgroups on a compute unit, the second set of accumulators two.)
bool batched_form(const ConvArgs& a) {
  if (!is_16bit(a.op_dtype) || a.cout % 128 != 0 || a.x2) return false;
  const long cols = (a.w + 15) / 16, b4 = (a.h + 3) / 4 * cols, b8 = (a.h + 7) / 8 * cols;
  return b4 * (a.cout / 128) * a.n > 256 && 5 * b8 <= 3 * b4;
}

}  // namespace

// 16-bit types: images of at most 2^20 output elements a sample (2048 pixels of 512 channels), where the 128 x 128 tiles
// leave at least three quarters of the compute units empty.  Measured against what takes larger layers (64 x 128 tiles), us at
// one sample: 17x23 of 512 channels 8.3 against 17.3; 32x32 11.5 / 17.4; 34x46 13.6 / 17.5; past the line 68x92 of 256 channels
// 12.0 / 11.3, 64x64 of 512 22.0 / 22.3.  The
// line may not depend on the batch: the order of summation does.  What the batch decides is the tile, see batched_form
// and pick_ksplit_tile.
// fp32: every size; 64 -> 64 channels at 32x32 take 10 us where the vector-ALU kernel takes 97.
bool conv_ksplit_supported(const ConvArgs& a) {
  if (a.ksize != 3 || a.upsample || a.x_nchw || a.y_nchw || a.x_dtype != a.op_dtype || a.rows_out || a.wide_tiles) return false;
  if (a.res && a.res_dtype != a.op_dtype) return false;
  if (a.y_dtype != a.op_dtype && a.y_dtype != WMDEC_F32) return false;
  if (a.cin > 2048 || a.cin2 > 2048 || a.groups > 2048) return false;   // scale/shift table in LDS
  if (!packed_offsets_fit(9, a.cout, a.cin, a.op_dtype) || !packed_offsets_fit(1, a.cout, a.cin2, a.op_dtype)) return false;
  if ((long)a.h * a.w * a.cin >= (1L << 29) || (long)a.h * a.w * a.cout >= (1L << 29) || (long)a.h * a.w * a.cin2 >= (1L << 29)) return false;
  if (a.op_dtype == WMDEC_F32) return a.cin % 32 == 0 && a.cin2 % (a.cin % 64 == 0 ? 64 : 32) == 0 && a.cout % 32 == 0 && !a.stats_ws;
  return is_16bit(a.op_dtype) && a.cin % 64 == 0 && a.cin2 % 64 == 0 && a.cout % 64 == 0 && (long)a.h * a.w * a.cout <= (1L << 20);
}

void conv_ksplit_grid(const ConvArgs& a, NextWeights* next) {
  static const struct { int th, tw, blocks; } shapes[] = {{4, 8, 1}, {4, 8, 2}, {4, 16, 2}, {4, 16, 4}, {8, 16, 4}};   // as KsplitTile, and the batched form
  const auto& t = shapes[batched_form(a) ? 4 : a.op_dtype == WMDEC_F32 ? 0 : (int)pick_ksplit_tile(a)];
  next->per_tile = ((a.h + t.th - 1) / t.th) * ((a.w + t.tw - 1) / t.tw) * a.n;
  next->tile_blocks = t.blocks;
  next->total = next->per_tile * (a.cout / (32 * t.blocks));
}

int conv_ksplit_stats_slots(const ConvArgs& a) {
  if (a.op_dtype == WMDEC_F32 || a.stats_groups <= 0 || a.cout % a.stats_groups != 0) return 0;
  const int cpg = a.cout / a.stats_groups;
  return (cpg & (cpg - 1)) != 0 || cpg > 32 ? 0 : ksplit_slots(a);   // the channels of a group are lanes of one wavefront
}

const char* conv_ksplit_label(const ConvArgs& a) {
  static thread_local char buf[128];
  static const char* const tile[] = {"4, 8, 1, 1, 4, 2, 2", "4, 8, 1, 2, 4, 1, 4", "4, 16, 1, 2, 4, 2, 2", "4, 16, 2, 2, 4, 1, 2"};
  const int act = a.mean == nullptr && a.rows_in == nullptr && !a.groups_norm ? 0 : (a.silu ? 2 : 1);
  const char* const ty = a.op_dtype == WMDEC_BF16 ? "wmdec::bf16_t" : "wmdec::f16_t";
  if (batched_form(a)) snprintf(buf, sizeof(buf), "conv_mfma_kernel<%s, %s, 8, 16, 1, 4, 1, 3, 32, %d, 2, 9>", ty, a.y_dtype == WMDEC_F32 ? "float" : ty, act);
  else if (a.op_dtype == WMDEC_F32) snprintf(buf, sizeof(buf), "conv_ksplit_kernel<float, 4, 8, 1, 1, %d, 1, 1, %d>", a.cin % 64 == 0 ? 4 : 2, act);
  else snprintf(buf, sizeof(buf), "conv_ksplit_kernel<%s, %s, %d>", ty, tile[pick_ksplit_tile(a)], act);
  return buf;
}

int launch_conv_ksplit(const ConvArgs& a, hipStream_t s) {
  if (batched_form(a)) return launch_conv_quarters(a, s);
  if (a.op_dtype == WMDEC_F32) return a.cin % 64 == 0 ? launch_tile<float, 4, 8, 1, 1, 4, 1, 1>(a, s) : launch_tile<float, 4, 8, 1, 1, 2, 1, 1>(a, s);
  return a.op_dtype == WMDEC_BF16 ? launch_16bit<bf16_t>(a, s) : launch_16bit<f16_t>(a, s);
}

}  // namespace wmdec
