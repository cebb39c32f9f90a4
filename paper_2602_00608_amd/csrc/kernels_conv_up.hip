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
// inside it (1.22x of the products).  On 16x16x32 MFMAs a wavefront holds all eight grid rows of 16 channels (A = weights, B = pixels): a
// weight fragment feeds eight MFMAs, i+1 is the lane's next row of accumulators and j+1 a lane shift within a
// row of 16 lanes, so that the phases are formed in registers.
#include <stdio.h>

#include "conv_device.hpp"

namespace wmdec {
namespace {

constexpr int GH = 8, GW = 16, TH = GH - 1, TW = GW - 1;   // grid of a workgroup, input pixels it finishes
constexpr int PH_ = GH + 1, PW = GW + 1, KC = 32;          // staged patch (from pixel (-1,-1) of the tile), channels of a chunk
// LDS layout as in kernels_conv_rows.hip: 96 bytes from pixel to pixel
constexpr int PSB = KC * 2 + 32, ROWB = PW * PSB, BUFB = PH_ * ROWB + PSB, SPARE = PH_ * ROWB;

// Steps of a chunk: the taps, those of the left column first; the accumulator of each.
constexpr int kTap[9] = {0, 3, 6, 1, 2, 4, 5, 7, 8};
constexpr int kAcc[9] = {3, 1, 3, 2, 3, 0, 1, 2, 3};

// v[lane + 1] within a row of 16 lanes (the last lane of a row takes 0: it finishes no pixel)
__device__ __forceinline__ float next_column(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x101, 0xf, 0xf, true));
}
// sum over the 16 lanes of a row, in all of them
__device__ __forceinline__ float row_sum(float v) {
  v += row_rotate<1>(v);
  v += row_rotate<2>(v);
  v += row_rotate<4>(v);
  return v + row_rotate<8>(v);
}

// Four wavefronts of 16 channels (H = 2 of them make the 32 of a packed fragment, WN such pairs).  Where WN = 1 leaves wavefronts over, KS
// groups of them take a part of the input channels each, with patches of their own, and every group finishes a KS-th of
// the rows after the partial sums were exchanged through LDS.
// FINE: moments of groups of one or two channels (sums per channel instead of per quad).
template <typename T, int H, int WN, bool FINE>
__global__ __launch_bounds__(256, 2) void conv_up_kernel(MfmaParams p, int y_f32) {
  static_assert(H == 2 && (WN == 1 || WN == 2), "pairs of wavefronts");
  constexpr int NT = 256, KS = 4 / (H * WN), NTK = NT / KS, TN = 32 * WN, WAVES = H * WN;
  constexpr int ER = GH / KS;                // grid rows whose pixels a wavefront finishes (the last group: one less)
  constexpr int VPP = KC / 8, NV = (PH_ * PW * VPP + NTK - 1) / NTK;
  fetch_arguments<sizeof(MfmaParams) + sizeof(int)>();
  extern __shared__ __align__(16) unsigned char smem_all[];   // [KS][2][BUFB]

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave % WAVES, wk = wave / WAVES;
  const int tid = threadIdx.x - wk * NTK;   // within the group
  unsigned char* smem = smem_all + wk * 2 * BUFB;
  const int px = lane & 15, oct = lane >> 4;
  const WorkTile wt = workgroup_tile(p);
  if (__builtin_expect(carries_weights(p), 0)) { warm_weights(p.next, p.total, 4, wave, lane); return; }
  const int nt = wt.nt, n = wt.n, tile = wt.tile;
  const int ty0 = wt.y * TH, tx0 = wt.x * TW;
  const int h_in = p.h >> 1, w_in = p.w_out >> 1;
  const int co_w = nt * TN + wn * 16;

  // weights: tap t of a chunk, 16 channels x 32 input channels, is half of two packed fragments; a ring in place, a chunk ahead
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, p.w_bytes, 0x00020000);
  const int kk_stride = p.cout_blocks * 1024, tap_stride = p.cin_blocks * kk_stride;
  const int chunks = p.cin / KC / KS, c0 = wk * chunks;   // chunks of the group, and its first
  const int wcol = (co_w >> 5) * 1024 + (co_w & 16) * 16;
  const int lane_w = (oct >> 1) * kk_stride + (px + 32 * (oct & 1)) * 16;
  u32x4 bq[9];

  const int cvec = tid % VPP;
  const char* xin = reinterpret_cast<const char*>(p.x) + (size_t)n * h_in * w_in * p.cin * 2;
  int src_off[NV], dst_off[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int hp = (tid + i * NTK) / VPP, hy = hp / PW, hx = hp % PW;
    const int gy = ty0 + hy - 1, gx = tx0 + hx - 1;
    const bool in_patch = hp < PH_ * PW, inside = in_patch & ((unsigned)gy < (unsigned)h_in) & ((unsigned)gx < (unsigned)w_in);   // (no branches)
    // outside the image: loaded from pixel 0, stored to the spare slot; the real slot is zeroed once
    src_off[i] = ((inside ? gy * w_in + gx : 0) * p.cin + cvec * 8) * 2;
    const int at = hy * ROWB + hx * PSB;
    dst_off[i] = (inside ? at : SPARE) + cvec * 16;
    if (in_patch & !inside) {
      *reinterpret_cast<u32x4*>(smem + at + cvec * 16) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(smem + BUFB + at + cvec * 16) = u32x4{0u, 0u, 0u, 0u};
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

  issue(0);
  // (behind the first input, which is needed first: loads return in order)
#pragma unroll
  for (int t = 0; t < 9; ++t) bq[t] = load_fragment(wrsrc, lane_w, wcol + 2 * c0 * kk_stride + kTap[t] * tap_stride);

  f32x4 acc[4][GH];   // A, B, C, D of every grid row: channels co_w + 4 oct + 0..3 of column px; every phase holds A once, so A starts from the bias
  {
    f32x4 bias = f32x4{0.f, 0.f, 0.f, 0.f};
    if (p.bias && wk == 0) bias = f32x4{p.bias[co_w + 4 * oct], p.bias[co_w + 4 * oct + 1], p.bias[co_w + 4 * oct + 2], p.bias[co_w + 4 * oct + 3]};
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int r = 0; r < GH; ++r) acc[a][r] = a == 0 ? bias : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int p_off = px * PSB + oct * 16;

  store(smem);
  issue(1);
  __syncthreads();
  for (int c = 0; c < chunks; ++c) {
    const unsigned char* buf = smem + (c & 1) * BUFB + p_off;
    unsigned char* nbuf = smem + ((c + 1) & 1) * BUFB;
    // Pixel fragments: patch row f of the left column is number f, of the other number 9 + f, in a ring of nine places; one is
    // refreshed behind the last MFMA that reads it, at least eight MFMAs before its next use.
    u32x4 af[PH_];
    auto read = [&](auto q_c) {
      constexpr int q = decltype(q_c)::value;
      af[q % PH_] = *reinterpret_cast<const u32x4*>(buf + q % PH_ * ROWB + q / PH_ * PSB);
    };
    static_for<PH_>(read);
    const int next = wcol + 2 * (c0 + min(c + 1, chunks - 1)) * kk_stride;
    static_for<9>([&](auto t_c) {
      constexpr int t = decltype(t_c)::value, down = kTap[t] >= 3;   // tap rows 1 and 2 read one row further down
      static_for<GH>([&](auto r_c) {
        constexpr int r = decltype(r_c)::value, f = r + down;
        acc[kAcc[t]][r] = Mma<T>::m16(bq[t], af[f], acc[kAcc[t]][r]);
        // the left column's row f was read for the last time: row 0 by its first tap, the others by its third
        if constexpr (t == 0 && r == 0) read(std::integral_constant<int, PH_>{});
        if constexpr (t == 2) read(std::integral_constant<int, PH_ + f>{});
        __builtin_amdgcn_sched_barrier(0);
      });
      bq[t] = load_fragment(wrsrc, lane_w, next + kTap[t] * tap_stride);
      if constexpr (t == 4) {   // half way: the next chunk to LDS, the one after it on its way
        store(nbuf);
        issue(c + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
  }

  // ---- the partial sums: a wavefront gives the rows that the other group's wavefront of its channels finishes, of C and D also the
  // row below the last of them
  const int row0 = wk * ER;            // first grid row that this wavefront finishes
  if constexpr (KS > 1) {
    static_assert(KS <= 2 && (size_t)4 * 2 * 5 * 64 * 16 <= (size_t)KS * 2 * BUFB, "two accumulators of five rows fit the patches");
    f32x4* half = reinterpret_cast<f32x4*>(smem_all);   // [4 wavefronts][2][5][64]: two accumulators at a time
    const int other = wave ^ WAVES;
#pragma unroll
    for (int a0 = 0; a0 < 4; a0 += 2) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < ER + 1; ++r)   // group 1 gives rows 0 .. 4, group 0 rows 4 .. 7
          if (r < ER || wk) half[((wave * 2 + a) * 5 + r) * 64 + lane] = wk ? acc[a0 + a][r] : acc[a0 + a][min(r + ER, GH - 1)];
      __syncthreads();
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        f32x4 own[ER + 1];
#pragma unroll
        for (int r = 0; r < ER + 1; ++r) own[r] = wk ? acc[a0 + a][min(r + ER, GH - 1)] : acc[a0 + a][r];
#pragma unroll
        for (int r = 0; r < ER + 1; ++r)   // from here on the wavefront's rows are 0 .. ER
          acc[a0 + a][r] = r < ER || !wk ? own[r] + half[((other * 2 + a) * 5 + r) * 64 + lane] : f32x4{0.f, 0.f, 0.f, 0.f};
      }
      __syncthreads();
    }
  }

  // ---- the four phases of every finished pixel, in registers
  const size_t sample = (size_t)n * p.h * p.w_out * p.cout;
  const int cpg = p.stats_cpg;
  // output bytes of the sample are addressed by 32-bit offsets (< 2^31, checked on the host); a lane without a pixel
  // gets an offset of 2^31, behind any sample, where a store is dropped (a row further is still below 2^32)
  const int es = y_f32 ? 4 : 2;
  const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(p.y) + sample * es, 0, p.h * p.w_out * p.cout * es, 0x00020000);
  // 16 bits: a lane stores eight channels of the left or (odd octets) the right of two neighbouring pixels; fp32: four of either
  const unsigned lane_y = y_f32 ? (unsigned)(2 * px * p.cout + 4 * oct) * 4u : (unsigned)((2 * px + (oct & 1)) * p.cout + (oct >> 1) * 8) * 2u;
  const int rows = min(ER - (KS == 1 || wk == KS - 1 ? 1 : 0), h_in - ty0 - row0), cols = min(TW, w_in - tx0);   // finished by this wavefront (rows may be < 1)
  const bool col_live = px < cols;
  auto live = [&](int r) -> bool { return r < rows && col_live; };
  auto phases = [&](int r, int e, float (&out)[4]) {
    const float a = acc[0][r][e], b = acc[1][r][e], c = acc[2][r][e], d = acc[3][r][e], c1 = acc[2][r + 1][e], d1 = acc[3][r + 1][e];
    out[0] = (a + b) + (c + d);
    out[1] = (a + c) + next_column(b + d);
    out[2] = (a + b) + (c1 + d1);
    out[3] = (a + next_column(b)) + (c1 + next_column(d1));
  };
  // Moments of the stored values: plain sums of a quad (FINE: of a channel), shifted by the mean of the first phase over every other row
  // (over a whole group where one spans quads of this wavefront): an eighth of the values or more, so that no single
  // one of them, however far off, can cancel the sums
  constexpr int NS = FINE ? 4 : 1, CH = 4 / NS;
  float sh[NS], ss[NS], sq[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    sh[k] = 0.f; ss[k] = 0.f; sq[k] = 0.f;
    if (p.stats && rows > 0) {
      float v = 0.f;
#pragma unroll
      for (int r = 0; r < ER; r += 2)
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          const int x = CH * k + e;
          v += live(r) ? (acc[0][r][x] + acc[1][r][x]) + (acc[2][r][x] + acc[3][r][x]) : 0.f;
        }
      v = row_sum(v) * (1.0f / (float)(CH * cols * ((rows + 1) / 2)));
      if (!FINE && cpg >= 8) v = 0.5f * swap_sum<16>(v);
      if (!FINE && cpg >= 16) v = 0.5f * swap_sum<32>(v);
      sh[k] = v;
    }
  }
#pragma unroll
  for (int r = 0; r < (KS == 1 ? GH - 1 : ER); ++r) {
    float out[4][4];   // [channel][phase]
#pragma unroll
    for (int e = 0; e < 4; ++e) phases(r, e, out[e]);
#pragma unroll
    for (int py = 0; py < 2; ++py) {
      const unsigned so = (((unsigned)(2 * (ty0 + row0 + r) + py) * p.w_out + 2 * tx0) * p.cout + co_w) * es;   // wave-uniform
      const unsigned at = live(r) ? lane_y + so : 0x80000000u;
      if (y_f32) {
#pragma unroll
        for (int qx = 0; qx < 2; ++qx)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{out[0][2 * py + qx], out[1][2 * py + qx], out[2][2 * py + qx], out[3][2 * py + qx]}), yrsrc,
                                                 at + (unsigned)(qx * p.cout * 4), 0, 0);
      } else {
        uint32_t w[2][2];
#pragma unroll
        for (int qx = 0; qx < 2; ++qx)
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            w[qx][k] = pack2<T>(out[2 * k][2 * py + qx], out[2 * k + 1][2 * py + qx]);
            out[2 * k][2 * py + qx] = unpack_lo<T>(w[qx][k]); out[2 * k + 1][2 * py + qx] = unpack_hi<T>(w[qx][k]);
          }
        // octets 2 k and 2 k + 1 exchange their quads of the two pixels, so that a lane stores eight consecutive channels of one
        u32x4 v;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const u32x2 t = __builtin_amdgcn_permlane16_swap(w[0][k], w[1][k], false, false);
          unsigned lo = t.x, hi = t.y;
          asm volatile("" : "+v"(lo), "+v"(hi));
          v[k] = lo; v[2 + k] = hi;
        }
        __builtin_amdgcn_raw_buffer_store_b128(v, yrsrc, at, 0, 0);
      }
    }
    if (p.stats && live(r)) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int ph = 0; ph < 4; ++ph) { const float dv = out[e][ph] - sh[e / CH]; ss[e / CH] += dv; sq[e / CH] = fmaf(dv, dv, sq[e / CH]); }
    }
  }
  if (p.stats) {   // over the lanes of a row, and the octets of a group; a group of 32 channels has a triple of either wavefront
    const int per_tile = KS * (cpg > 16 ? 2 : 1), slot = tile * per_tile + wk * (per_tile / KS) + (cpg > 16 ? wn % 2 : 0);
    Moments mq[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      float s = row_sum(ss[k]), t = row_sum(sq[k]), cnt = rows > 0 ? 4.f * CH * (float)(rows * cols) : 0.f;
      if (!FINE && cpg >= 8) { s = swap_sum<16>(s); t = swap_sum<16>(t); cnt *= 2.f; }
      if (!FINE && cpg >= 16) { s = swap_sum<32>(s); t = swap_sum<32>(t); cnt *= 2.f; }
      const float ds = cnt > 0.f ? s / cnt : 0.f;   // (without a finished pixel all zeros: nothing outside the image enters)
      const float m2 = t - s * ds;
      mq[k] = Moments{cnt, sh[k] + ds, m2 < 0.f ? 0.f : m2};
    }
    Moments* dst = p.stats + (size_t)n * p.stats_groups * p.stats_slots + slot;
    if constexpr (FINE) {
      if (cpg == 2) { mq[0] = merge(mq[0], mq[1]); mq[1] = merge(mq[2], mq[3]); }
      if (px == 0) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (g < 2 || cpg == 1) store_device(dst + (size_t)((co_w + 4 * oct) / cpg + g) * p.stats_slots, mq[g]);
      }
    } else if (px == 0 && (oct * 4) % min(cpg, 16) == 0) {
      store_device(dst + (size_t)((co_w + 4 * oct) / cpg) * p.stats_slots, mq[0]);
    }
  }
  if (p.rows_out) hand_over_row<NT>(p, n, wt.y, nt, nt * TN, TN, KS * (cpg > 16 ? 2 : 1), threadIdx.x, lane);
}

// 64 channels a workgroup, 16 a wavefront, two workgroups per compute unit: their epilogues
// overlap each other's sweeps.
constexpr int kH = 2, kWN = 2, kTN = 32 * kWN;

// ... or 32 channels, with the contraction split in two: one round of half as many channels then leaves compute units idle, and
// a lone workgroup is bound by the weights that its wavefronts take through the vector L1 (64 B/clk), 1.2 MB at 512
// channels, of which half the channels need half.  A function of the sample's shape: the sums do not depend on the batch.
// us, whole / split, by the number of whole workgroups: 512 channels 48 16.2 / 11.9, 120 16.4 / 12.6, 128 16.9 / 13.6, 160 17.3 / 19.1, 240 20.7 / 22.9;
// 256 channels 60 10.7 / 9.0, 120 11.1 / 9.8, 144 11.4 / 12.9; 128 channels 96 8.3 / 7.8.  Past 128 workgroups the halves share a compute unit again.
bool split_channels(const ConvArgs& a) {
  const long wgs = (long)((a.h / 2 + TH - 1) / TH) * ((a.w / 2 + TW - 1) / TW) * (a.cout / kTN);
  return a.cin % (2 * KC) == 0 && wgs <= 128;
}
int tile_channels(const ConvArgs& a) { return split_channels(a) ? 32 : kTN; }
// triples a workgroup leaves per group: one of every part of its rows, and of either wavefront of a group of 32 channels
int slots_per_tile(const ConvArgs& a) { return (split_channels(a) ? 2 : 1) * (a.stats_groups > 0 && a.cout / a.stats_groups > 16 ? 2 : 1); }

bool fine_moments(const ConvArgs& a) { return a.stats_groups > 0 && a.cout / a.stats_groups < 4; }

template <typename T>
int launch_up(const ConvArgs& a, hipStream_t s) {
  const bool split = split_channels(a);
  MfmaParams p = conv_params(a, TH, TW, tile_channels(a), slots_per_tile(a), a.h / 2, a.w / 2);
  const int rc = check_hand_over(p);
  if (rc != WMDEC_OK) return rc;
  p.w = a.wt;
  p.w_bytes = (int)(packed_elems(9, a.cout, a.cin) * sizeof(T));
  constexpr size_t kSmem = 2 * BUFB, kSplitSmem = 4 * BUFB;   // patches of one group, of two
  void (*kern)(MfmaParams, int) = split ? (fine_moments(a) ? conv_up_kernel<T, kH, 1, true> : conv_up_kernel<T, kH, 1, false>)
                                        : (fine_moments(a) ? conv_up_kernel<T, kH, kWN, true> : conv_up_kernel<T, kH, kWN, false>);
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.total + warm_groups(p.next, 4))), dim3(256), split ? kSplitSmem : kSmem, s, p, a.y_dtype == WMDEC_F32 ? 1 : 0);
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
  if ((cpg & (cpg - 1)) != 0 || cpg > 32) return 0;   // a group must sit inside a pair of wavefronts
  return ((a.h / 2 + TH - 1) / TH) * ((a.w / 2 + TW - 1) / TW) * slots_per_tile(a);
}

void conv_up_row_extents(const ConvArgs& a, int* tile_rows, int* channel_tiles, int* tiles_per_row) {
  *tile_rows = (a.h / 2 + TH - 1) / TH;
  *channel_tiles = a.cout / tile_channels(a);
  *tiles_per_row = (a.w / 2 + TW - 1) / TW;
}

void conv_up_grid(const ConvArgs& a, NextWeights* next) {
  next->per_tile = ((a.h / 2 + TH - 1) / TH) * ((a.w / 2 + TW - 1) / TW) * a.n;
  next->tile_blocks = tile_channels(a) / 32;
  next->total = next->per_tile * (a.cout / tile_channels(a));
}

const char* conv_up_label(const ConvArgs& a) {
  static thread_local char buf[64];
  snprintf(buf, sizeof(buf), "conv_up_kernel<%s, %d, %d, %s>", a.op_dtype == WMDEC_BF16 ? "wmdec::bf16_t" : "wmdec::f16_t", kH,
           split_channels(a) ? 1 : kWN, fine_moments(a) ? "true" : "false");
  return buf;
}

int launch_conv_up(const ConvArgs& a, hipStream_t s) { return a.op_dtype == WMDEC_BF16 ? launch_up<bf16_t>(a, s) : launch_up<f16_t>(a, s); }

}  // namespace wmdec
