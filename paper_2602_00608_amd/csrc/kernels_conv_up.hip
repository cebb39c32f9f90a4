// Nearest-2x upsampling followed by a 3x3 convolution, on the low-resolution grid, with nine products per input pixel.
//
// Output pixel (2i + py, 2j + px) sums the nine taps W[ky][kx] over input pixels (i + r(py,ky), j + r(px,kx)), where
// r(0,.) = -1, 0, 0 and r(1,.) = 0, 0, 1: its four phases use 36 products per input pixel, of which only nine differ
// (tap times input pixel).  With u[ky][kx] taken at input pixel (i - [ky = 0], j - [kx = 0]), every phase is a sum over
//   A = u11,  B = u10 + u12,  C = u01 + u21,  D = u00 + u02 + u20 + u22
// at grid position (i, j) or its neighbours:
//   phase (0,0) = A + B + C + D                       phase (0,1) = A + C + (B + D)[j+1]
//   phase (1,0) = A + B + (C + D)[i+1]                phase (1,1) = A + B[j+1] + C[i+1] + D[i+1][j+1]
// so four accumulators take all nine products: 9 instead of the 16 of four 2x2 convolutions with pre-summed weights (and
// of the 36 of the plain form), no weight is rounded after a sum, and it serves both 16-bit types from the
// ordinary 3x3 pack.  A workgroup takes an 8 x 16 grid and writes the 7 x 15 input pixels whose neighbours lie
// inside it (1.22x of the products), 32 channels per wavefront column; grid columns are lanes of a 16-lane row, so that
// j+1 is a lane shift and i+1 a row swap, and the phases are formed in registers.
#include <stdio.h>

#include "conv_device.hpp"

namespace wmdec {
namespace {

constexpr int GH = 8, GW = 16, TH = GH - 1, TW = GW - 1;   // grid of a workgroup, input pixels it finishes
constexpr int PH_ = GH + 1, PW = GW + 1, KC = 32;          // staged patch (from pixel (-1,-1) of the tile), channels of a chunk
// LDS layout as in kernels_conv_mfma.hip: pixel stride 80 bytes (conflict-free 16-byte reads), row stride a multiple of 256
constexpr int PSB = KC * 2 + 16, ROWB = (PW * PSB + 255) / 256 * 256, BUFB = PH_ * ROWB + PSB, SPARE = PH_ * ROWB;

// The four pixel shifts of a k-step with the taps that read them, (1,1): 11 12 21 22, (0,1): 01 02, (0,0): 00, (1,0): 10 20,
// and the accumulator of each tap.
constexpr int kShift[4] = {ROWB + PSB, PSB, 0, ROWB};
constexpr int kFirst[5] = {0, 4, 6, 7, 9};
constexpr int kTap[9] = {4, 5, 7, 8, 1, 2, 0, 3, 6};
constexpr int kAcc[9] = {0, 1, 2, 3, 2, 3, 3, 1, 3};

// v[lane + 1] within a row of 16 lanes (the last lane of a row takes 0: it finishes no pixel)
__device__ __forceinline__ float next_column(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x101, 0xf, 0xf, true));
}
// the value one grid row down: an M tile holds rows 2m (lanes 0-15 of each half) and 2m + 1 (lanes 16-31)
__device__ __forceinline__ float next_row(float cur, float below, bool odd) {
  const u32x2 r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, cur), __builtin_bit_cast(unsigned, below), false, false);
  unsigned a = r.x, b = r.y;   // a: rows (cur 0, below 0), b: rows (cur 1, below 1)
  asm volatile("" : "+v"(a), "+v"(b));
  return __builtin_bit_cast(float, odd ? a : b);
}

// sum over the 32 lanes of this lane's half of the wavefront, in the half's first lane
__device__ __forceinline__ float half_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x101, 0xf, 0xf, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x102, 0xf, 0xf, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x104, 0xf, 0xf, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x108, 0xf, 0xf, true));
  return v + __shfl_xor(v, 16);
}

// Four wavefronts: WM rows share the grid's four M tiles, WN columns of 32 channels.  Where that leaves wavefronts over, KS
// groups of them take a part of the input channels each, with patches of their own, and every wavefront finishes a KS-th of
// its row's M tiles after the partial sums were exchanged through LDS.
// FINE: moments of groups of one or two channels (sums per channel instead of per quad).
template <typename T, int WM, int WN, bool FINE>
__global__ __launch_bounds__(256, 2) void conv_up_kernel(MfmaParams p, int y_f32) {
  constexpr int NT = 256, KS = 4 / (WM * WN), NTK = NT / KS, MI = 4 / WM, TN = 32 * WN;
  constexpr int ME = MI / KS, WR = WM * KS;   // the epilogue's M tiles per wavefront, and its wavefront rows
  constexpr int VPP = KC / 8, NV = (PH_ * PW * VPP + NTK - 1) / NTK;
  static_assert(KS == 1 || (KS == 2 && MI == 2), "the exchange below hands over one of two M tiles");
  extern __shared__ __align__(16) unsigned char smem_all[];   // [KS][2][BUFB]

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave % WN, wm = wave / WN % WM, wk = wave / (WN * WM);
  const int tid = threadIdx.x - wk * NTK;   // within the group
  unsigned char* smem = smem_all + wk * 2 * BUFB;
  const int lm = lane & 31, lk = lane >> 5;
  int L;   // consecutive ids of one XCD (id % 8) are neighbours
  {
    const int i = blockIdx.x, per = p.total / 8, rem = p.total % 8;
    const int x = i % 8, j = i / 8;
    L = x * per + (x < rem ? x : rem) + j;
  }
  const int tiles = p.tiles_x * p.tiles_y;
  const int nt = L / (tiles * p.n), n = (L / tiles) % p.n, tile = L % tiles;
  const int ty0 = (tile / p.tiles_x) * TH, tx0 = (tile % p.tiles_x) * TW;
  const int h_in = p.h >> 1, w_in = p.w_out >> 1;
  const int co_w = nt * TN + wn * 32;

  // weight fragments: tap t of k-step s is fragment (t, s); in place, one k-step (nine fragments) ahead
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, p.w_bytes, 0x00020000);
  const int kk_stride = p.cout_blocks * 1024, tap_stride = p.cin_blocks * kk_stride, wcol = (co_w >> 5) * 1024;
  const int chunks = p.cin / KC / KS, c0 = wk * chunks;   // chunks of the group, and its first
  const int lane16 = lane * 16, ksteps = 2 * (c0 + chunks);
  u32x4 bq[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) bq[t] = load_fragment(wrsrc, lane16, wcol + 2 * c0 * kk_stride + kTap[t] * tap_stride);

  const int cvec = tid % VPP;
  const char* xin = reinterpret_cast<const char*>(p.x) + (size_t)n * h_in * w_in * p.cin * 2;
  int src_off[NV], dst_off[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int hp = (tid + i * NTK) / VPP, hy = hp / PW, hx = hp % PW;
    const int gy = ty0 + hy - 1, gx = tx0 + hx - 1;
    const bool in_patch = hp < PH_ * PW, inside = in_patch && gy >= 0 && gy < h_in && gx >= 0 && gx < w_in;
    // outside the image: loaded from pixel 0, stored to the spare slot; the real slot is zeroed once
    src_off[i] = ((inside ? gy * w_in + gx : 0) * p.cin + cvec * 8) * 2;
    dst_off[i] = (inside ? hy * ROWB + hx * PSB : SPARE) + cvec * 16;
    if (in_patch && !inside) {
      *reinterpret_cast<u32x4*>(smem + hy * ROWB + hx * PSB + cvec * 16) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(smem + BUFB + hy * ROWB + hx * PSB + cvec * 16) = u32x4{0u, 0u, 0u, 0u};
    }
  }
  u32x4 raw[NV];
  auto issue = [&](int c) {
    const int cb = (c0 + min(c, chunks - 1)) * KC * 2;   // past the last chunk: a harmless reload
#pragma unroll
    for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const u32x4*>(xin + (unsigned)(src_off[i] + cb));
  };
  auto store = [&](unsigned char* buf) {
#pragma unroll
    for (int i = 0; i < NV; ++i) *reinterpret_cast<u32x4*>(buf + dst_off[i]) = raw[i];
  };

  f32x16 acc[4][MI];   // A, B, C, D; every phase holds A once, so A starts from the bias
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float bias = p.bias && wk == 0 ? p.bias[co_w + 8 * (r / 4) + 4 * lk + r % 4] : 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) acc[a][mi][r] = a == 0 ? bias : 0.f;
  }
  int p_off[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) p_off[mi] = (2 * (wm * MI + mi) + lm / GW) * ROWB + (lm % GW) * PSB + lk * 16;

  issue(0);
  store(smem);
  issue(1);
  __syncthreads();
  for (int c = 0; c < chunks; ++c) {
    const unsigned char* buf = smem + (c & 1) * BUFB;
    unsigned char* nbuf = smem + ((c + 1) & 1) * BUFB;
    // pixel fragments are read two shifts ahead: the shortest shift is a single tap, less than the LDS latency
    u32x4 af[3][MI];
    auto read_shift = [&](u32x4 (&f)[MI], int g) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) f[mi] = *reinterpret_cast<const u32x4*>(buf + p_off[mi] + kShift[g % 4] + (g / 4) * 32);
    };
    read_shift(af[0], 0);
    read_shift(af[1], 1);
    static_for<8>([&](auto g_c) {
      constexpr int g = decltype(g_c)::value, kk = g / 4, s = g % 4;   // shift s of k-step kk
      if constexpr (g + 2 < 8) read_shift(af[(g + 2) % 3], g + 2);
      const int next = wcol + min(2 * (c0 + c) + kk + 1, ksteps - 1) * kk_stride;
      static_for<kFirst[s + 1] - kFirst[s]>([&](auto t_c) {
        constexpr int t = kFirst[s] + decltype(t_c)::value;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) acc[kAcc[t]][mi] = Mma<T>::m32(bq[t], af[g % 3][mi], acc[kAcc[t]][mi]);
        bq[t] = load_fragment(wrsrc, lane16, next + kTap[t] * tap_stride);
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (g == 3) {   // half way: the next chunk to LDS, the one after it on its way
        store(nbuf);
        issue(c + 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    __syncthreads();
  }

  // ---- the partial sums: a wavefront gives the M tile that the other group's wavefront of its row finishes
  f32x16 sum[4][ME];
  if constexpr (KS > 1) {
    float* half = reinterpret_cast<float*>(smem_all);   // [4 wavefronts][2][16][64]: two accumulators at a time
    const int other = wave ^ (WN * WM);
#pragma unroll
    for (int a0 = 0; a0 < 4; a0 += 2) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) half[((wave * 2 + a) * 16 + r) * 64 + lane] = wk ? acc[a0 + a][0][r] : acc[a0 + a][1][r];
      __syncthreads();
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[a0 + a][0][r] = (wk ? acc[a0 + a][1][r] : acc[a0 + a][0][r]) + half[((other * 2 + a) * 16 + r) * 64 + lane];
      __syncthreads();
    }
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int mi = 0; mi < ME; ++mi) sum[a][mi] = acc[a][mi];
  }
  const int wr = wm * KS + wk;   // wavefront row of the epilogue, M tiles wr * ME + (0 .. ME - 1)

  // ---- the four phases of every finished pixel, in registers.  Element r of a lane: channel co_w + 8 (r / 4) + 4 lk + r % 4
  // of grid position (2 m + lm / 16, lm % 16).  Wavefront row wr needs the first grid row of the M tile below its last,
  // which another wavefront holds when WR > 1: C and D of it travel through LDS.
  float* ex = reinterpret_cast<float*>(smem_all);   // [WR][WN][2][16][64]
  if constexpr (WR > 1) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) ex[(((wr * WN + wn) * 2 + a) * 16 + r) * 64 + lane] = sum[2 + a][0][r];
    __syncthreads();
  }
  const int wb = (min(wr + 1, WR - 1) * WN + wn) * 2;   // the wavefront below; the last row's copy of itself reaches no output
  const bool odd_row = (lm & 16) != 0;
  const size_t sample = (size_t)n * p.h * p.w_out * p.cout;
  const int cpg = p.stats_cpg;
  // output bytes of the sample are addressed by 32-bit offsets (< 2^31, checked on the host); a lane without a pixel
  // gets an offset of 2^31, behind any sample, where a store is dropped (a row further is still below 2^32)
  const int es = y_f32 ? 4 : 2;
  const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(p.y) + sample * es, 0, p.h * p.w_out * p.cout * es, 0x00020000);
  unsigned y_off[ME];
  int live_px = 0, first_px = 0;   // pixels this wavefront finishes, and those of its first M tile (of which it has some if any)
  bool live[ME];
#pragma unroll
  for (int mi = 0; mi < ME; ++mi) {
    const int gy = 2 * (wr * ME + mi) + lm / GW, gx = lm % GW;
    const int iy = ty0 + gy, ix = tx0 + gx;
    live[mi] = gy < TH && gx < TW && iy < h_in && ix < w_in;
    y_off[mi] = live[mi] ? ((2 * iy * p.w_out + 2 * ix) * p.cout + co_w + (y_f32 ? 4 : 8) * lk) * es : 0x80000000u;
    live_px += __builtin_popcountll(__ballot(live[mi])) / 2;   // (both halves of the wavefront hold every pixel)
    if (mi == 0) first_px = live_px;
  }
  Moments mq[4];
#pragma unroll
  for (int qp = 0; qp < 2; ++qp) {              // eight channels of the lane at a time: quads 2 qp and 2 qp + 1
    // moments of the stored values: plain sums of a quad, shifted by the mean of the first M tile's first phase over the
    // quad (over both halves where a group spans them): an eighth of the values or more, so that no single one of them,
    // however far off, can cancel the sums
    constexpr int NS = FINE ? 8 : 2, CH = 8 / NS;
    float sh[NS], ss[NS], sq[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) { sh[k] = 0.f; ss[k] = 0.f; sq[k] = 0.f; }
#pragma unroll
    for (int mi = 0; mi < ME; ++mi) {
      float out[4][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = 8 * qp + e;
        const float a = sum[0][mi][r], b = sum[1][mi][r], c = sum[2][mi][r], d = sum[3][mi][r];
        float cb = 0.f, db = 0.f;
        if (mi + 1 < ME) { cb = sum[2][mi + 1 < ME ? mi + 1 : mi][r]; db = sum[3][mi + 1 < ME ? mi + 1 : mi][r]; }
        else if constexpr (WR > 1) { cb = ex[((wb + 0) * 16 + r) * 64 + lane]; db = ex[((wb + 1) * 16 + r) * 64 + lane]; }
        const float c1 = next_row(c, cb, odd_row), d1 = next_row(d, db, odd_row);
        out[0][e] = (a + b) + (c + d);
        out[1][e] = (a + c) + next_column(b + d);
        out[2][e] = (a + b) + (c1 + d1);
        out[3][e] = (a + next_column(b)) + (c1 + next_column(d1));
      }
#pragma unroll
      for (int ph = 0; ph < 4; ++ph) {
        const int so = (((ph >> 1) * p.w_out + (ph & 1)) * p.cout + 16 * qp) * es;   // wave-uniform
        if (y_f32) {
#pragma unroll
          for (int q = 0; q < 2; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{out[ph][4 * q], out[ph][4 * q + 1], out[ph][4 * q + 2], out[ph][4 * q + 3]}), yrsrc, y_off[mi] + so + 32 * q, 0, 0);
        } else {
          uint32_t w[2][2];
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const int e = 4 * q + 2 * k;
              w[q][k] = pack2<T>(out[ph][e], out[ph][e + 1]);
              out[ph][e] = unpack_lo<T>(w[q][k]); out[ph][e + 1] = unpack_hi<T>(w[q][k]);
            }
          // the halves of the wavefront exchange quads, so that a lane stores eight consecutive channels
          u32x4 v;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const u32x2 t = __builtin_amdgcn_permlane32_swap(w[0][k], w[1][k], false, false);
            unsigned lo = t.x, hi = t.y;
            asm volatile("" : "+v"(lo), "+v"(hi));
            v[k] = lo; v[2 + k] = hi;
          }
          __builtin_amdgcn_raw_buffer_store_b128(v, yrsrc, y_off[mi] + so, 0, 0);
        }
      }
      if (p.stats) {
        if (mi == 0) {
          const float inv = first_px > 0 ? 1.0f / (float)(CH * first_px) : 0.f;
#pragma unroll
          for (int k = 0; k < NS; ++k) {
            float v = 0.f;
#pragma unroll
            for (int e = 0; e < CH; ++e) v += out[0][CH * k + e];
            const int sum = __builtin_bit_cast(int, half_sum(live[0] ? v : 0.f));
            const float v0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(sum, 0)), v1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(sum, 32));
            sh[k] = (cpg >= 8 ? 0.5f * v0 + 0.5f * v1 : lk ? v1 : v0) * inv;
          }
        }
        if (live[mi]) {
#pragma unroll
          for (int ph = 0; ph < 4; ++ph)
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float dv = out[ph][e] - sh[e / CH]; ss[e / CH] += dv; sq[e / CH] = fmaf(dv, dv, sq[e / CH]); }
        }
      }
    }
    if (p.stats) {   // over the lanes of one half of the wavefront, and both halves where a group spans them
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        float s = half_sum(ss[k]), t = half_sum(sq[k]), cnt = 4.f * CH * (float)live_px;
        if (!FINE && cpg >= 8) { s += __shfl_xor(s, 32); t += __shfl_xor(t, 32); cnt *= 2.f; }
        const float ds = live_px > 0 ? s / cnt : 0.f;   // (without a finished pixel all zeros: nothing outside the image enters)
        const float m2 = t - s * ds;
        const Moments m{cnt, sh[k] + ds, m2 < 0.f ? 0.f : m2};
        if constexpr (FINE) mq[k % 4] = m;
        else mq[2 * qp + k] = m;
        if (FINE && k % 4 == 3 && lm == 0) {   // one quad's channels: four groups of one or two of two
          Moments* dst = p.stats + ((size_t)n * p.stats_groups + (co_w + 8 * (2 * qp + k / 4) + 4 * lk) / cpg) * p.stats_slots + tile * WR + wr;
          if (cpg == 2) { mq[0] = merge(mq[0], mq[1]); mq[1] = merge(mq[2], mq[3]); }
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (g < 2 || cpg == 1) store_device(dst + (size_t)g * p.stats_slots, mq[g]);
        }
      }
    }
  }
  if (!FINE && p.stats) {   // quads of a group; WR wavefront rows leave a slot each
    if (cpg >= 16) { mq[0] = merge(mq[0], mq[1]); mq[2] = merge(mq[2], mq[3]); }
    if (cpg >= 32) mq[0] = merge(mq[0], mq[2]);
    if (lm == 0 && (lk == 0 || cpg == 4)) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if ((8 * q) % cpg == 0 || cpg == 4)
          store_device(p.stats + ((size_t)n * p.stats_groups + (co_w + 8 * q + 4 * lk) / cpg) * p.stats_slots + tile * WR + wr, mq[q]);
    }
  }
  if (p.rows_out) hand_over_row<NT>(p, n, tile / p.tiles_x, nt, nt * TN, TN, WR, threadIdx.x, lane);
}

// 64 channels a workgroup, two wavefronts on either half of the grid, two workgroups per compute unit: their epilogues
// overlap each other's sweeps.  Measured, us: 512 channels at 120x180 143 (four wavefront columns of 128 channels 164 to
// 170, one wavefront row 170, four 246); a wavefront row per M tile re-reads every weight fragment four times.
constexpr int kWM = 2, kWN = 2, kTN = 32 * kWN;

// ... or 32 channels, with the contraction split in two: one round of half as many channels then leaves compute units idle, and
// a lone workgroup is bound by the weights that its wavefronts take through the vector L1 (64 B/clk), 1.2 MB at 512
// channels, of which half the channels need half.  A function of the sample's shape: the sums do not depend on the batch.
// 512 channels, us: 17x23 20.7 -> 17.4, 32x32 22.0 -> 19.3; frames of these sizes 1.008x and 1.006x.  Past 128 workgroups the halves
// would share a compute unit again.
bool split_channels(const ConvArgs& a) {
  const long wgs = (long)((a.h / 2 + TH - 1) / TH) * ((a.w / 2 + TW - 1) / TW) * (a.cout / kTN);
  return a.cin % (2 * KC) == 0 && wgs <= 128;
}
int tile_channels(const ConvArgs& a) { return split_channels(a) ? 32 : kTN; }
int slots_per_tile(const ConvArgs& a) { return split_channels(a) ? 4 : kWM; }

bool fine_moments(const ConvArgs& a) { return a.stats_groups > 0 && a.cout / a.stats_groups < 4; }

template <typename T>
int launch_up(const ConvArgs& a, hipStream_t s) {
  const bool split = split_channels(a);
  MfmaParams p = conv_params(a, TH, TW, tile_channels(a), slots_per_tile(a), a.h / 2, a.w / 2);
  const int rc = check_hand_over(p);
  if (rc != WMDEC_OK) return rc;
  p.w = a.wt;
  p.w_bytes = (int)(packed_elems(9, a.cout, a.cin) * sizeof(T));
  constexpr size_t kExchange = (size_t)kWM * kWN * 2 * 16 * 64 * sizeof(float);   // rows handed between wavefront rows
  constexpr size_t kSmem = 2 * BUFB > kExchange ? 2 * BUFB : kExchange;
  constexpr size_t kSplitSmem = 4 * BUFB;   // patches of two groups
  static_assert(kSplitSmem >= kExchange && kExchange == (size_t)4 * 2 * 16 * 64 * sizeof(float), "rows and partial sums fit the patches");
  void (*kern)(MfmaParams, int) = split ? (fine_moments(a) ? conv_up_kernel<T, kWM, 1, true> : conv_up_kernel<T, kWM, 1, false>)
                                        : (fine_moments(a) ? conv_up_kernel<T, kWM, kWN, true> : conv_up_kernel<T, kWM, kWN, false>);
  hipLaunchKernelGGL(kern, dim3((unsigned)p.total), dim3(256), split ? kSplitSmem : kSmem, s, p, a.y_dtype == WMDEC_F32 ? 1 : 0);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

}  // namespace

bool conv_up_supported(const ConvArgs& a) {
  if (a.ksize != 3 || !a.upsample || !is_16bit(a.op_dtype) || a.x_dtype != a.op_dtype || a.x_nchw || a.y_nchw) return false;
  if (a.mean || a.groups_norm || a.rows_in || a.res || a.x2 || a.cin2 || (a.y_dtype != a.op_dtype && a.y_dtype != WMDEC_F32)) return false;
  if (a.cin % KC != 0 || a.cout % kTN != 0 || a.h % 2 != 0 || a.w % 2 != 0 || !packed_offsets_fit(9, a.cout, a.cin, a.op_dtype)) return false;
  if (a.stats_ws && conv_up_stats_slots(a) == 0) return false;
  // 32-bit byte offsets per sample
  return (long)(a.h / 2) * (a.w / 2) * a.cin < (1L << 29) && (long)a.h * a.w * a.cout * (long)dtype_size(a.y_dtype) < (1L << 31);
}

int conv_up_stats_slots(const ConvArgs& a) {
  if (a.stats_groups <= 0 || a.cout % a.stats_groups != 0) return 0;
  const int cpg = a.cout / a.stats_groups;
  if ((cpg & (cpg - 1)) != 0 || cpg > 32) return 0;   // a group must sit inside one wavefront's 32 channels
  return ((a.h / 2 + TH - 1) / TH) * ((a.w / 2 + TW - 1) / TW) * slots_per_tile(a);
}

void conv_up_row_extents(const ConvArgs& a, int* tile_rows, int* channel_tiles, int* tiles_per_row) {
  *tile_rows = (a.h / 2 + TH - 1) / TH;
  *channel_tiles = a.cout / tile_channels(a);
  *tiles_per_row = (a.w / 2 + TW - 1) / TW;
}

const char* conv_up_label(const ConvArgs& a) {
  static thread_local char buf[64];
  snprintf(buf, sizeof(buf), "conv_up_kernel<%s, %d, %d, %s>", a.op_dtype == WMDEC_BF16 ? "wmdec::bf16_t" : "wmdec::f16_t", kWM,
           split_channels(a) ? 1 : kWN, fine_moments(a) ? "true" : "false");
  return buf;
}

int launch_conv_up(const ConvArgs& a, hipStream_t s) { return a.op_dtype == WMDEC_BF16 ? launch_up<bf16_t>(a, s) : launch_up<f16_t>(a, s); }

}  // namespace wmdec
