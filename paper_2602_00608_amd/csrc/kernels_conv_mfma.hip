// Implicit-GEMM convolution on the gfx950 matrix cores: 1x1 layers, 3x3 layers with 64 output channels or few, the batched form of
// kernels_conv_ksplit.hip; and the choice of tile for all, also for the 3x3 layers of kernels_conv_rows.hip.
//
// GEMM view: M = output pixels, N = output channels, K = taps * C_in.
// One workgroup (4 wavefronts) owns a TH x TW patch of output pixels and TN
// output channels.  Per chunk of KC input channels it stages the patch plus its
// one-pixel halo into LDS -- GroupNorm scale/shift and SiLU are applied there,
// once per element, and positions outside the image are zeros -- and then sweeps
// the nine taps over that tile: the A operand of every MFMA is a 16-byte LDS read
// at a tap-dependent constant offset, the B operand (weights) is loaded straight
// from the L2-resident packed weights, where every 32(co) x 16(ci) fragment is
// 1 KiB in lane order, so a wavefront's load is one contiguous KiB.
// Accumulators stay in registers for the whole K loop; bias, residual, the single
// rounding to the storage type and the GroupNorm moments of the output happen in
// the epilogue.
// The staged tile is double-buffered: the raw vectors of chunk c+2 are loaded
// right after the sweep of chunk c, and chunk c+1 is activated and stored into
// the other buffer in compile-time slots inside the sweep of chunk c, with one
// workgroup barrier per chunk.  Two or three workgroups fit on a compute unit, so
// the prologue and epilogue of one overlap the sweeps of the others.
#include <stdio.h>

#include <mutex>

#include "conv_moments.hpp"

namespace wmdec {
namespace {

// Wavefront-private epilogue patches of 32 padded rows: a second one, for the next M tile's values, where there is a next M tile
// and the workgroups that the registers allow still fit the LDS with it (four of 36.9 KB with one channel tile a wavefront, two of
// 69.6 KB with two of them and eight accumulator tiles).  A third and fourth workgroup are worth more than the patch: one / two
// patches, us, 3x3 64 -> 64 at 240x360 14.1 / 15.6, at 480x720 48.0 / 51.3; 1x1 512 -> 1536 at 60x90 21.6 / 23.7, 256 -> 64 at 240x360
// 13.3 / 15.7.
constexpr int epilogue_patches(int mi, int ni) { return mi > 1 && (ni == 1 || mi * ni > 4) ? 2 : 1; }
constexpr int patch_floats(int mi, int ni) { return epilogue_patches(mi, ni) * 32 * (ni * 32 + 4); }

struct EpilogueParams {
  __amdgpu_buffer_rsrc_t res, y;           // the sample's residual and output, with its size: accesses outside are dropped
  void* planar;                            // the sample's output where it is planar
  int h, w, cout;
  bool nchw;
  Moments* stats; int cpg, stats_stride, pair_stride;
  bool handed_over;
};

// Epilogue of one wavefront: its MI x NI accumulator tiles (32 pixels x 32 channels each, a lane holding one channel column)
// go through wavefront-private LDS patches, one 32-pixel M tile at a time (the next one's values on their way to the other patch,
// where there are two), and come back as rows of 8 consecutive channels per lane, so that residual and output move as 16-byte vectors and every
// pixel's channel run is written contiguously.  LDS operations of one wavefront execute in order: no barrier.
// The bias (of the lane's channel columns) is added to the finished sums, on their way to LDS: accumulators that start from it
// round every partial sum at its exponent, an error of 4e-7 of the result against 3e-8 where the bias is many times the sum.
// Residual and output are accessed through buffers with a lane offset that is the same for all vectors, or past the end for
// pixels outside the image, and the vector's position in a scalar register: no address arithmetic, no masks.
// Moments: one triple per group for all M tiles.  kQuarters (NI = 1):
// one for each M tile of 4 x 8 pixels, from the values written back to the patches of a pair: a lane walks one channel
// of either tile, as the kernel that it reproduces does.
template <typename T, typename TO, int MI, int NI, int MTW, int MTH, int MT_PER_ROW, bool RES, int MODE>
__device__ __forceinline__ void epilogue_store(const f32x16 (&acc)[MI][NI], const float (&bias)[NI], float* wave_lds, int lane, int mt0,
                                               int ty0, int tx0, int co_w, const EpilogueParams& p) {
  constexpr int RW = NI * 32 + 4;       // padded row of a patch, floats
  constexpr bool PAIRS = MODE == kQuarters;
  constexpr int PATCHES = epilogue_patches(MI, NI);
  const int lm = lane & 31, lk = lane >> 5;
  auto put = [&](float* patch, int mi) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) patch[(8 * (r / 4) + 4 * lk + (r % 4)) * RW + ni * 32 + lm] = acc[mi][ni][r] + bias[ni];
  };
  if (p.nchw) {
    // planar output with few channels (the frame): a lane owns one pixel of the M tile and walks the
    // channels, so that 32 lanes write 32 consecutive pixels of one plane
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int mt = mt0 + mi;
      const int oy = ty0 + (mt / MT_PER_ROW) * MTH + lm / MTW, ox = tx0 + (mt % MT_PER_ROW) * MTW + lm % MTW;
      put(wave_lds, mi);
      if (oy < p.h && ox < p.w) {
        for (int c = lk; c < NI * 32 && co_w + c < p.cout; c += 2)
          reinterpret_cast<TO*>(p.planar)[((size_t)(co_w + c) * p.h + oy) * p.w + ox] = from_float<TO>(wave_lds[lm * RW + c]);
      }
    }
    return;
  }
  constexpr int VPL = 2 * NI;           // 8-channel vectors per lane per M tile (32 pixels x NI*4 vectors / 64 lanes)
  constexpr int STEP = 64 / (NI * 4);   // pixels between two of them
  static_assert(STEP % MTW == 0 || MTW % STEP == 0, "a vector's row and column are the lane's plus a constant");
  const int cvec = lane % (NI * 4);     // which 8-channel vector of the row this lane reads back
  const int prow = lane / (NI * 4);     // first pixel it reads; the others are prow + j * STEP
  const int lane_row = prow / MTW, lane_col = prow % MTW;
  // elements: the lane's part, and that of vector j of M tile mi
  const unsigned lane_off = (unsigned)((lane_row * p.w + lane_col) * p.cout + cvec * 8);
  auto row_of = [&](int mi, int j) { return ty0 + (mt0 + mi) / MT_PER_ROW * MTH + j * STEP / MTW; };
  auto col_of = [&](int mi, int j) { return tx0 + (mt0 + mi) % MT_PER_ROW * MTW + j * STEP % MTW; };
  auto inside = [&](int mi, int j) -> bool { return row_of(mi, j) + lane_row < p.h && col_of(mi, j) + lane_col < p.w; };
  auto base_of = [&](int mi, int j) -> int { return vector_base(row_of(mi, j), col_of(mi, j), p.h, p.w, p.cout, co_w); };
  // residual vectors are requested ahead so that their latency hides behind the LDS round trips of the tiles before
  constexpr int RD = NI == 1 && MI <= 4 ? MI : 2;
  u32x4 rv[RD][VPL];
  auto request = [&](int mi) {
#pragma unroll
    for (int j = 0; j < VPL; ++j)
      rv[mi % RD][j] = __builtin_amdgcn_raw_buffer_load_b128(p.res, (int)((inside(mi, j) ? lane_off : kOutside) * sizeof(T)), base_of(mi, j) * (int)sizeof(T), 0);
  };
  if constexpr (RES) {
#pragma unroll
    for (int mi = 0; mi < RD && mi < MI; ++mi) request(mi);
  }
  LaneMoments<8> st = {};
  put(wave_lds, 0);
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    float* lds = wave_lds + mi % PATCHES * 32 * RW;
    const bool ahead = PATCHES == 2 && mi + 1 < MI && !(PAIRS && mi % 2 == 1);   // (a pair's patches are read once more at its end)
    if (ahead) put(wave_lds + (mi + 1) % PATCHES * 32 * RW, mi + 1);
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
      const int pi = prow + j * STEP;
      const bool ok = inside(mi, j);
      const f32x4 lo = *reinterpret_cast<const f32x4*>(lds + pi * RW + cvec * 8);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(lds + pi * RW + cvec * 8 + 4);
      float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      if constexpr (RES) {
        float rf[8];
        unpack8<T>(rv[mi % RD][j], rf);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += rf[e];
      }
      // the stored vector; the moments are those of the values as stored (after the rounding to the storage
      // type), which is what the consumer of the tensor normalises
      u32x4 packed;
      if constexpr (sizeof(TO) == 2) packed = u32x4{pack2<T>(v[0], v[1]), pack2<T>(v[2], v[3]), pack2<T>(v[4], v[5]), pack2<T>(v[6], v[7])};
      const int at = (int)((ok ? lane_off : kOutside) * sizeof(TO)), base = base_of(mi, j) * (int)sizeof(TO);
      if constexpr (sizeof(TO) == 4) {
        u32x4 a = __builtin_bit_cast(u32x4, f32x4{v[0], v[1], v[2], v[3]}), b = __builtin_bit_cast(u32x4, f32x4{v[4], v[5], v[6], v[7]});
        store_vector(p.y, a, at, base);
        store_vector(p.y, b, at + 16, base);
      } else {
        store_vector(p.y, packed, at, base);
      }
      if (p.stats) {
        float sv[8];
        if constexpr (sizeof(TO) == 2) {
          unpack8<T>(packed, sv);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) sv[e] = v[e];
        }
        if constexpr (PAIRS) {
          if (ok) {
            *reinterpret_cast<f32x4*>(lds + pi * RW + cvec * 8) = f32x4{sv[0], sv[1], sv[2], sv[3]};
            *reinterpret_cast<f32x4*>(lds + pi * RW + cvec * 8 + 4) = f32x4{sv[4], sv[5], sv[6], sv[7]};
          }
        } else {
          if (mi == 0 && j == 0) {   // (outside the image only if all vectors of the lane are)
            st.n = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) { st.shift[e] = sv[e]; st.s[e] = 0.f; st.q[e] = 0.f; }
          }
          if (ok) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float dv = sv[e] - st.shift[e]; st.s[e] += dv; st.q[e] = fmaf(dv, dv, st.q[e]); }
            st.n += 1.f;
          }
        }
      }
    }
    if constexpr (RES) {
      if (mi + RD < MI) request(mi + RD);
    }
    if constexpr (PAIRS) {
      static_assert(NI == 1 && PATCHES == 2 && MI % 2 == 0 && MTW == 8 && MTH == 4 && MT_PER_ROW == 2, "a pair is four rows of 16 pixels");
      if (mi % 2 == 1 && p.stats) {   // lanes 0-31: a channel of the pair's first tile, lanes 32-63: of the second
        Moments* dst = p.stats + (mi / 2) * p.pair_stride;
        const int y0 = ty0 + (mt0 + mi - 1 + lk) / MT_PER_ROW * MTH, x0 = tx0 + (mt0 + mi - 1 + lk) % MT_PER_ROW * MTW;
        const float* src = wave_lds + lk * 32 * RW + lm;
        const int rows = min(MTH, p.h - y0), cols = min(MTW, p.w - x0);
        Moments m = block_moments(two_row_sums<MTW, MTW * RW, RW>(src, src[0], rows, cols) +
                                  two_row_sums<MTW, MTW * RW, RW>(src + 2 * MTW * RW, src[0], rows - 2, cols), src[0], rows, cols);
        with_group_size(p.cpg, [&](auto cpg_c) __attribute__((always_inline)) { m = merge_channels<decltype(cpg_c)::value>(m); });
        if ((lm & (p.cpg - 1)) == 0 && m.n > 0.f) dst[(size_t)((co_w + lm) / p.cpg) * p.stats_stride + lk] = m;
      }
    } else if (mi + 1 == MI) {
      if (p.stats) emit_vectors<NI * 4, 8>({st}, lane, co_w, {p.stats}, p.cpg, p.stats_stride, p.handed_over);
    }
    if (mi + 1 < MI && !ahead) put(wave_lds + (mi + 1) % PATCHES * 32 * RW, mi + 1);
  }
}

// Ring length of the weight-fragment prefetch: it must divide the k-steps of a chunk so that the ring
// position is the same at every chunk start (18 with 3x3 taps; 4 or 2 with one).  The fragments come from the L2, whose latency is
// several k-steps.
constexpr int prefetch_ring(int steps) { return steps % 6 == 0 ? 6 : steps % 4 == 0 ? 4 : 2; }

struct NoFlush { __device__ void operator()(int) const {} };

// MFMA work of one staged chunk: STEPS = taps * KC/16 k-steps, each MI x NI 32x32x16 MFMAs.
// Weight fragments are fetched D-1 steps ahead (bq is a ring that persists across chunks: on
// entry it holds steps 0..D-2 of this chunk, on exit steps 0..D-2 of the chunk at `bnext`).
// The A fragment of an M tile is refreshed in place for the next step right after the MFMAs
// that consumed it, which gives the LDS read the rest of the step to land.  The scheduling
// barriers pin that order: without them the compiler sinks every load to just before its use
// and each k-step pays a full memory latency.
// VALU_PER_MFMA: -1 pins the order as written (slot hook after the MFMAs of an M tile); >= 0 asks the scheduler to
// interleave that many vector-ALU instructions behind every MFMA of a k-step.
// KMAJOR: all taps of the chunk's first 16 channels come before those of its second 16 (otherwise both 16 tap by tap), the
// weights of the two lie at bcur / bcur1, and flush(0 / 1) runs behind each.
// AD: how many k-steps ahead the A fragments are read (1 or 2).  One step is MI - 1 MFMAs of slack, about the LDS
// latency: enough where other wavefronts of the SIMD fill the gaps, too little for a wavefront that is alone on it.
template <typename T, int MI, int NI, int KS, int KC, int ROW, int PS, int D, bool SLICED, int VALU_PER_MFMA, typename Slice, int AD = 1, bool KMAJOR = false, typename Flush = NoFlush>
__device__ __forceinline__ void mfma_chunk(const T* buf, const int (&a_off)[MI], __amdgpu_buffer_rsrc_t wrsrc, int bcur, int bnext,
                                           int tap_stride, int kk_stride, int lane16, u32x4 (&bq)[D][NI],
                                           f32x16 (&acc)[MI][NI], Slice&& slice, int bcur1 = 0, int bnext1 = 0, Flush&& flush = NoFlush()) {
  constexpr int KK = KC / 16, TAPS = KS * KS, STEPS = TAPS * KK;
  static_assert(!KMAJOR || KK == 2, "two groups of 16 channels");
  // element offset of a k-step's pixels in the staged tile
  auto a_at = [](int s) constexpr {
    const int tap = KMAJOR ? s % TAPS : s / KK, kk = KMAJOR ? s / TAPS : s % KK;
    return (tap / KS) * ROW + (tap % KS) * PS + kk * 16;
  };
  static_assert(AD == 1 || AD == 2, "A fragments one or two k-steps ahead");
  u32x4 af[AD][MI];   // af[s % AD]: fragments of k-step s
#pragma unroll
  for (int a = 0; a < AD && a < STEPS; ++a) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) af[a][mi] = *reinterpret_cast<const u32x4*>(buf + a_off[mi] + a_at(a));
  }
  // one k-step; the slot hook runs after the MFMAs of every M tile so that its vector-ALU work issues
  // while those MFMAs occupy the matrix pipe
  auto step = [&](auto s_c) {
    constexpr int s = decltype(s_c)::value;
    {
      constexpr int sp = s + D - 1;
      constexpr int spp = sp < STEPS ? sp : sp - STEPS;
      int at;
      if constexpr (KMAJOR) at = (sp < STEPS ? (spp / TAPS ? bcur1 : bcur) : (spp / TAPS ? bnext1 : bnext)) + (spp % TAPS) * tap_stride;
      else at = (sp < STEPS ? bcur : bnext) + (spp / KK) * tap_stride + (spp % KK) * kk_stride;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) bq[sp % D][ni] = load_fragment(wrsrc, lane16, at + ni * 1024);
    }
    __builtin_amdgcn_sched_barrier(0);
    auto tile = [&](auto mi_c) {
      constexpr int mi = decltype(mi_c)::value;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = Mma<T>::m32(af[s % AD][mi], bq[s % D][ni], acc[mi][ni]);
      if constexpr (s + AD < STEPS) {
        constexpr int at = a_at(s + AD);
        af[s % AD][mi] = *reinterpret_cast<const u32x4*>(buf + a_off[mi] + at);
      }
      if constexpr (SLICED) slice(std::integral_constant<int, s * MI + mi>{});
      if constexpr (VALU_PER_MFMA < 0) __builtin_amdgcn_sched_barrier(0);
    };
    static_for<MI>(tile);
    if constexpr (VALU_PER_MFMA >= 0) {
      // The whole k-step is one scheduling region; spell out the issue order inside it: after every MFMA the A
      // refresh that belongs to it (one LDS read per NI MFMAs) and an equal share of the step's activation work,
      // so that each MFMA's 32 cycles in the matrix pipe cover vector-ALU work instead of the next MFMA's wait.
      static_for<MI * NI>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // one MFMA
        if constexpr (j % NI == NI - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
        if constexpr (VALU_PER_MFMA > 0) __builtin_amdgcn_sched_group_barrier(0x402, VALU_PER_MFMA, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (KMAJOR && s % TAPS == TAPS - 1) {
      flush(s / TAPS);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_for<STEPS>(step);
}

// ACT: what happens to an input element on its way into LDS: 0 nothing, 1 scale/shift, 2 scale/shift + SiLU
constexpr int wave_m_tiles(int th, int tw, int wm) { return th * tw / 32 / wm; }
// Workgroups per compute unit the register budget is sized for: three for the small accumulator tiles, except the
// 2x2-wavefront 128x128 shape, which is only picked for layers with at most two workgroups per compute unit and
// uses the registers for a longer prefetch instead.
constexpr int resident_workgroups(int acc_tiles, int wm, int wn) {
  return acc_tiles <= 4 && !(wm == 2 && wn == 2) ? 3 : 2;
}

// LDS layout of a staged tile (elements of the 16-bit type): pixel (hy, hx) of the halo patch sits at hy * ROW + hx * PS.
// PS = KC + 8: the 16-byte pad makes the 16 lanes that the LDS serves per cycle (consecutive pixels of a row, 16 bytes
// each) fall on 64 distinct banks.  A 32-pixel M tile that spans two patch rows (16-pixel-wide patches) has lanes i and
// i + 16 one row apart; the LDS only runs at full rate when such lane pairs are a multiple of 256 bytes apart (measured:
// any other row stride costs a second pass per read), so for those patches the row stride is rounded up to 256 bytes.
// One pixel slot behind the patch is spare: vectors that lie outside the image (or past the patch) are stored there,
// where no MFMA reads them.
// Where an M tile is 8 pixels wide and spans four rows, i and i + 16 are two rows apart and i and i + 8 one: the stride of a
// row is then 128 modulo 256, that of eight pixels.
constexpr int tile_row_elems(int tw, int pad, int kc, int mtw) {
  const int raw = (tw + 2 * pad) * (kc + 8);
  return mtw == 8 ? (raw * 2 + 127) / 256 * 128 + 64 : tw < 32 ? (raw * 2 + 255) / 256 * 128 : raw;
}
constexpr int tile_buf_elems(int th, int tw, int pad, int kc, int mtw) { return (th + 2 * pad) * tile_row_elems(tw, pad, kc, mtw) + (kc + 8); }

// RING: 0 = weight-fragment ring sized by prefetch_ring; otherwise its length in k-steps (a divisor of the k-steps of
// a chunk).
constexpr int m_tile_width(int tw, int mode) { return mode == kQuarters ? 8 : tw < 32 ? tw : 32; }
template <typename T, typename TO, int TH, int TW, int WM, int WN, int NI, int KS, int KC, int ACT, int MODE = kPlain, int RING = 0>
__global__ __launch_bounds__(64 * WM * WN, RING > 6 ? 2 : resident_workgroups(wave_m_tiles(TH, TW, WM) * NI, WM, WN))
void conv_mfma_kernel(MfmaParams p) {
  static_assert(WM * WN == 4 || WM * WN == 8, "four or eight wavefronts");
  constexpr int NT = 64 * WM * WN;               // threads of the workgroup
  constexpr int MI = wave_m_tiles(TH, TW, WM);   // 32-pixel M tiles per wavefront
  constexpr int PAD = KS / 2;
  constexpr int HW_ = TW + 2 * PAD, HH_ = TH + 2 * PAD, HP = HW_ * HH_;
  constexpr int PS = KC + 8;                     // LDS pixel stride in elements (+16 B: conflict-free 16-byte reads)
  constexpr bool QUARTERS = MODE == kQuarters;
  constexpr int MTW = m_tile_width(TW, MODE), MTH = 32 / MTW, MT_PER_ROW = TW / MTW;
  constexpr int TN = WN * NI * 32;
  constexpr int VPP = KC / 8;                    // 16-byte vectors per pixel per chunk
  constexpr int NV = (HP * VPP + NT - 1) / NT;   // vectors a thread stages per chunk
  constexpr int ROW = tile_row_elems(TW, PAD, KC, MTW);       // LDS row stride of the staged tile, elements
  constexpr int BUF = tile_buf_elems(TH, TW, PAD, KC, MTW);   // elements of one staged tile: the halo patch plus the spare slot
  constexpr int SPARE = HH_ * ROW;                       // element offset of the spare pixel slot
  constexpr int STEPS = KS * KS * (KC / 16), SLOTS = STEPS * MI;
  constexpr bool SLICED = KS == 3;               // activation of the next chunk is sliced into the MFMA sweep
  static_assert(NT % VPP == 0, "a thread keeps one channel octet");
  static_assert((RING > 6 ? 2 : resident_workgroups(MI * NI, WM, WN)) * WM * WN * patch_floats(MI, NI) * sizeof(float) <= 160 * 1024,
                "the workgroups that the registers are budgeted for fit the LDS of a compute unit");

  fetch_arguments<sizeof(MfmaParams)>();
  extern __shared__ __align__(16) unsigned char smem[];
  T* s_a = reinterpret_cast<T*>(smem);                                          // [2][BUF]
  float2* s_ab = reinterpret_cast<float2*>(smem + ((2 * BUF * 2 + 15) & ~15));  // [cin] (scale, shift)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform: keeps the per-wave addresses scalar
  const int wm = wave / WN, wn = wave % WN;
  const int lm = lane & 31, lk = lane >> 5;

  const WorkTile wt = workgroup_tile(p);
  if (__builtin_expect(carries_weights(p), 0)) { warm_weights(p.next, p.total, WM * WN, wave, lane); return; }
  const int nt = wt.nt, n = wt.n, tile = wt.tile;
  const int ty0 = wt.y * TH, tx0 = wt.x * TW;
  const int co0 = nt * TN;

  // the bias of the lane's channel columns, for the epilogue: requested here, as a load there would be waited for, unless the
  // main loop has no register left to hold it
  constexpr bool BIAS_EARLY = !QUARTERS;
  float bias[NI];
  auto load_bias = [&]() {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const int co = min(co0 + (wn * NI + ni) * 32 + lm, p.cout - 1);   // (the frame has fewer channels than the tile)
      bias[ni] = p.bias ? p.bias[co] : 0.f;
      if (p.bias2) bias[ni] += p.bias2[co];
    }
  };
  if constexpr (BIAS_EARLY) load_bias();

  // LDS element offset of this lane's pixel in each of its M tiles (tap (0,0), k offset of the lane half)
  int a_off[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    const int mt = wm * MI + mi;
    const int ty = (mt / MT_PER_ROW) * MTH + lm / MTW;
    const int tx = (mt % MT_PER_ROW) * MTW + lm % MTW;
    a_off[mi] = ty * ROW + tx * PS + 8 * lk;
  }
  constexpr int KK = KC / 16;
  constexpr int D = RING > 0 ? RING : prefetch_ring(KS * KS * KK);   // weight fragments are fetched D-1 k-steps ahead
  static_assert((KS * KS * KK) % D == 0, "the ring position must be the same at every chunk start");
  const int tap_stride = p.cin_blocks * p.cout_blocks * 1024, kk_stride = p.cout_blocks * 1024;   // bytes
  // byte offset of this wavefront's fragment column (wave-uniform; the lane's 16 bytes are added by the load)
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, p.w_bytes, 0x00020000);
  const int wcol = ((co0 >> 5) + wn * NI) * 1024;
  const int lane16 = lane * 16;
  // QUARTERS: partial sum k takes the groups of 16 channels k, k + 4, k + 8, ...; the two groups of a chunk are kept for the current chunk and
  // the two after it, and advance by running counters (a division per use cost 10 % of a launch of one round)
  const int quarter = p.cin / 64;
  int run_j = 0, run_k = 0;
  auto next_group = [&]() {
    const int g = run_j * 4 + run_k;
    const bool wrap = ++run_j == quarter;
    run_j = wrap ? 0 : run_j;
    run_k += wrap ? 1 : 0;
    return g;
  };
  struct Groups { int a, b; };
  Groups grp[3] = {};     // of chunks c, c + 1, c + 2; past the last chunk: those of the last, a harmless reload
  if constexpr (QUARTERS) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (i < 2 || p.cin > 2 * KC) { grp[i].a = next_group(); grp[i].b = next_group(); }
      else grp[i] = grp[i - 1];
    }
  }
  auto weights_at = [&](int chunk, int ahead, int kk) {   // chunk = c + ahead
    if constexpr (QUARTERS) return __builtin_amdgcn_readfirstlane(wcol + (kk ? grp[ahead].b : grp[ahead].a) * kk_stride);   // (said to be uniform: else a loop around every load)
    else return wcol + (chunk * KK + kk) * kk_stride;
  };
  u32x4 bq[D][NI];
  f32x16 acc[MI][NI];
#pragma unroll
  for (int sp = 0; sp < D - 1; ++sp) {
    const int tap = QUARTERS ? sp % (KS * KS) : sp / KK, kk = QUARTERS ? sp / (KS * KS) : sp % KK;
    const int at = weights_at(0, 0, kk) + tap * tap_stride;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) bq[sp][ni] = load_fragment(wrsrc, lane16, at + ni * 1024);
  }

  // ---- staging: a thread owns NV (pixel, channel-octet) vectors of the halo tile; the octet is the same for all
  const int cvec = tid % VPP;
  const char* xin = reinterpret_cast<const char*>(p.x) + (size_t)n * p.h * p.w_out * p.cin * sizeof(T);   // uniform base
  // Zero padding without per-element work: a vector outside the image is loaded from pixel 0 (a load under a lane
  // mask would make the compiler wait for it at the end of the branch), activated like any other, and stored to
  // the spare pixel slot behind the patch; its real slot is zeroed once, here, in both buffers.  A 1x1 convolution
  // has no halo: what its out-of-image pixels hold only reaches outputs that are never stored.
  int src_off[NV];          // byte offset of the vector's pixel in x
  int dst_off[NV];          // element offset of its slot in a staged tile
  int src_pix[NV];          // index of its source pixel in the sample (0 outside the image); only the shortcut phase reads it
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int v = tid + i * NT;
    const int hp = v / VPP;
    const int hy = hp / HW_, hx = hp % HW_;
    const int gy = ty0 + hy - PAD, gx = tx0 + hx - PAD;
    const bool in_patch = v < HP * VPP, inside = in_patch & ((unsigned)gy < (unsigned)p.h) & ((unsigned)gx < (unsigned)p.w_out);   // (no branches)
    src_pix[i] = inside ? gy * p.w_out + gx : 0;
    src_off[i] = src_pix[i] * p.cin * (int)sizeof(T);
    const bool keep = KS == 1 ? in_patch : inside;
    dst_off[i] = (keep ? hy * ROW + hx * PS : SPARE) + cvec * 8;
    if (KS != 1 && in_patch && !inside) {
      *reinterpret_cast<u32x4*>(s_a + hy * ROW + hx * PS + cvec * 8) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(s_a + BUF + hy * ROW + hx * PS + cvec * 8) = u32x4{0u, 0u, 0u, 0u};
    }
  }
  // One register set of raw vectors.  The loads of chunk k+1 are issued right after the MFMA sweep of chunk
  // k-1 (vector-memory loads return in order, so weight-fragment loads issued behind them cannot be consumed
  // before they have landed: the workgroup barrier and the first third of the next sweep cover that), and the
  // vectors are activated and stored into the other LDS buffer in the last two thirds of the sweep of chunk k,
  // a few elements after every M tile's MFMAs, so that this vector-ALU work overlaps the matrix pipe instead of
  // forming a phase of its own.
  u32x4 raw[NV];
  // first channel of this thread's octet in chunk c + ahead; past the last chunk: that of the last, a harmless reload
  auto channel = [&](int chunk, int ahead) -> int {
    if constexpr (QUARTERS) return (cvec / 2 ? grp[ahead].b : grp[ahead].a) * 16 + cvec % 2 * 8;
    else return min(chunk, p.cin / KC - 1) * KC + cvec * 8;
  };
  auto issue = [&](int chunk, int ahead) {
    const int cb = channel(chunk, ahead) * (int)sizeof(T);
#pragma unroll
    for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const u32x4*>(xin + (unsigned)(src_off[i] + cb));
  };
  // word (two channels) of a staged vector: scale/shift (+ SiLU) with the table entries ab = (a0, b0, a1, b1)
  auto activate_with = [&](uint32_t wv, const f32x4& ab) -> uint32_t { return wmdec::activate_word<T, ACT, MODE != kPlain>(wv, ab); };
  // table entries of word `part` of the octet that starts at channel c0
  auto table_entry = [&](int part, int c0) -> f32x4 {
    if constexpr (ACT > 0) return *reinterpret_cast<const f32x4*>(s_ab + c0 + 2 * part);
    else return f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto activate_word = [&](uint32_t wv, int i, int part, int c0) -> uint32_t {
    (void)i;
    return activate_with(wv, table_entry(part, c0));
  };
  auto store_vec = [&](int i, T* buf) { *reinterpret_cast<u32x4*>(buf + dst_off[i]) = raw[i]; };
  auto activate_all = [&](int c0, T* buf) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      raw[i] = u32x4{activate_word(raw[i].x, i, 0, c0), activate_word(raw[i].y, i, 1, c0),
                     activate_word(raw[i].z, i, 2, c0), activate_word(raw[i].w, i, 3, c0)};
      store_vec(i, buf);
    }
  };
  const int nchunks = p.cin / KC;
  // vector-ALU instructions of the activation per MFMA of an active k-step (8 per element with SiLU, 3 without),
  // one less than the average so that the tail of a word does not delay the next k-step (against the order as written: 1 to 2 %)
  constexpr int SPREAD_AVG = (NV * 8 * (ACT == 2 ? 8 : 3) + (SLOTS - SLOTS / 3) * NI - 1) / ((SLOTS - SLOTS / 3) * NI);
  constexpr int SPREAD = ACT == 0 ? -1 : (SPREAD_AVG > 1 ? SPREAD_AVG - 1 : 1);
  f32x4 abv[2];   // table entries of the part being activated and of the next one (sliced activation)

  float zero = 0.f;
  asm volatile("" : "+v"(zero));   // (seen as a constant, it costs the fullest of these kernels 190 spilled registers)
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = zero;
  // ---- shortcut phase (3x3 kernels with a second input): acc = W2 * x2 over the tile's own pixels, a 1x1
  // contraction over cin2 channels taken as stored (no normalisation).  Chunks of KC channels go through the same
  // two LDS buffers with the tile's halo layout (only the centre tap is read), loads two chunks ahead; the main
  // loop below then adds the 3x3 contraction to the same accumulators, so the shortcut tensor never exists in
  // memory and the epilogue adds both biases.
  if constexpr (KS == 3 && !QUARTERS) {
    if (p.x2) {
      const char* xin2 = reinterpret_cast<const char*>(p.x2) + (size_t)n * p.h * p.w_out * p.cin2 * sizeof(T);
      const int nch2 = p.cin2 / KC;
      auto issue2 = [&](int chunk) {
        const int cb = min(chunk, nch2 - 1) * KC * (int)sizeof(T);
#pragma unroll
        for (int i = 0; i < NV; ++i)
          raw[i] = *reinterpret_cast<const u32x4*>(xin2 + (unsigned)((src_pix[i] * p.cin2 + cvec * 8) * (int)sizeof(T) + cb));
      };
      auto store_all = [&](T* buf) {
#pragma unroll
        for (int i = 0; i < NV; ++i) store_vec(i, buf);
      };
      int a_ctr[MI];   // centre tap of the halo patch
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) a_ctr[mi] = a_off[mi] + PAD * ROW + PAD * PS;
      constexpr int D2 = 2;
      const __amdgpu_buffer_rsrc_t wrsrc2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w2), 0, p.w2_bytes, 0x00020000);
      const int wcol2 = ((co0 >> 5) + wn * NI) * 1024;
      u32x4 bq2[D2][NI];
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) bq2[0][ni] = load_fragment(wrsrc2, lane16, wcol2 + ni * 1024);
      issue2(0);
      store_all(s_a);
      issue2(1);
      __syncthreads();
      auto none = [](auto) {};
      for (int c = 0; c < nch2; ++c) {
        const int bcur = wcol2 + c * KK * kk_stride;
        const int bnext = c + 1 < nch2 ? bcur + KK * kk_stride : bcur;
        mfma_chunk<T, MI, NI, 1, KC, ROW, PS, D2, false, -1>(s_a + (c & 1) * BUF, a_ctr, wrsrc2, bcur, bnext, 0, kk_stride, lane16, bq2, acc, none);
        if (c + 1 < nch2) store_all(s_a + ((c + 1) & 1) * BUF);
        issue2(c + 2);
        __syncthreads();
      }
    }
  }

  issue(0, 0);
  // (built behind the first chunk's loads, so that its own global loads overlap them)
  // per-channel scale/shift table: a = gamma*rstd, b = beta - mean*a.  With SiLU the table holds -log2(e) * (a, b):
  // the staged value is u = -log2(e) * t, from which silu(t) = t / (1 + 2^u) = u / (-log2(e) - log2(e) * 2^u) takes
  // one exp2, one fma, one reciprocal and one multiply
  if constexpr (ACT > 0) {
    const float k = ACT == 2 ? -1.4426950408889634f : 1.0f;
    auto entry = [&](int c, float2 st, float ga, float be) {
      const float a = ga * st.y;
      s_ab[c] = make_float2(k * a, k * (be - st.x * a));
    };
    if (p.rows_in) {
      // mean / rstd of every group from the row triples its producer left: eight lanes per group take the rows
      // round-robin (16 in the form that has to reproduce a kernel with 16); (mean, rstd) parked behind the table
      float2* s_stat = s_ab + p.cin;
      // kQuarters: gamma / beta of this thread's first two table
      // entries are requested together with the triples, one memory round trip less in front of the first chunk
      // (elsewhere other workgroups cover that latency and the registers are better left to the main loop).
      constexpr int PRE = RING > 6 ? 2 : 0;
      float gpre[2] = {0.f, 0.f}, bpre[2] = {0.f, 0.f};
      int group[2] = {0, 0};
#pragma unroll
      for (int j = 0; j < PRE; ++j) {
        const int c = min(tid + j * NT, p.cin - 1);
        gpre[j] = p.gamma[c]; bpre[j] = p.beta[c];
        group[j] = quotient_of(c, p.cpg_in, p.inv_cpg_in);
      }
      constexpr int LANES = QUARTERS ? 16 : 8;
      merge_sample<LANES, NT>(p.rows_in + (size_t)n * p.groups * p.rows_in_count, p.groups, p.rows_in_count, tid, p.eps, s_stat);
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PRE; ++j)
        if (tid + j * NT < p.cin) entry(tid + j * NT, s_stat[group[j]], gpre[j], bpre[j]);
      for (int c = tid + PRE * NT; c < p.cin; c += NT) entry(c, s_stat[quotient_of(c, p.cpg_in, p.inv_cpg_in)], p.gamma[c], p.beta[c]);
    } else {
      for (int c = tid; c < p.cin; c += NT) {
        const int g = n * p.groups + quotient_of(c, p.cpg_in, p.inv_cpg_in);
        entry(c, make_float2(p.mean[g], p.rstd[g]), p.gamma[c], p.beta[c]);
      }
    }
  }
  __syncthreads();            // scale/shift table complete
  activate_all(channel(0, 0), s_a);
  issue(1, 1);
  f32x16 total[QUARTERS ? MI : 1][NI];   // the partial sums so far
#pragma unroll
  for (int i = 0; i < (QUARTERS ? MI : 1); ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) total[i][j][r] = 0.f;
  int left = quarter;   // groups of 16 channels until the running partial sum is complete
  auto flush = [&](int) {
    if constexpr (QUARTERS) {
      if (--left == 0) {
        left = quarter;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { total[i][j][r] += acc[i][j][r]; acc[i][j][r] = 0.f; }
      }
    }
  };
  __syncthreads();
  for (int c = 0; c < nchunks; ++c) {
    const bool more = c + 1 < nchunks;
    const int next = more ? c + 1 : c;
    const int bcur = weights_at(c, 0, 0), bnext = weights_at(next, 1, 0);
    const int bcur1 = QUARTERS ? weights_at(c, 0, 1) : 0, bnext1 = QUARTERS ? weights_at(next, 1, 1) : 0;
    const T* buf = s_a + (c & 1) * BUF;
    T* nbuf = s_a + ((c + 1) & 1) * BUF;
    const int c0n = channel(c + 1, 1);
    if constexpr (SLICED) {
      // Slots FIRST .. SLOTS-1 share the NV*4 words of the next chunk evenly.  All vectors of a thread hold the same
      // channel octet, so the words are taken part by part (word `part` of every vector, then the next part) and
      // the four table entries of the octet are read from LDS once each, one part ahead of their first use: a read
      // issued right where it is needed would expose the LDS latency in every slot.
      auto slice = [&](auto slot_c) {
        constexpr int slot = decltype(slot_c)::value;
        constexpr int FIRST = SLOTS / 3, SPAN = SLOTS - FIRST, NW = NV * 4;
        if constexpr (slot == FIRST - 1) abv[0] = table_entry(0, c0n);
        if constexpr (slot >= FIRST) {
          constexpr int w0 = (slot - FIRST) * NW / SPAN, w1 = (slot - FIRST + 1) * NW / SPAN;
          static_for<w1 - w0>([&](auto k_c) {
            constexpr int wi = w0 + decltype(k_c)::value;
            constexpr int part = wi / NV, i = wi % NV;
            if constexpr (i == 0 && part < 3) abv[(part + 1) & 1] = table_entry(part + 1, c0n);
            raw[i][part] = activate_with(raw[i][part], abv[part & 1]);
            if constexpr (part == 3) store_vec(i, nbuf);
          });
        }
      };
      // the last chunk activates a harmless reload into the buffer nobody reads: one instruction stream, no
      // control flow inside the pinned schedule
      mfma_chunk<T, MI, NI, KS, KC, ROW, PS, D, true, SPREAD, decltype(slice)&, (RING > 6 ? 2 : 1), QUARTERS>(buf, a_off, wrsrc, bcur, bnext, tap_stride, kk_stride, lane16, bq, acc, slice, bcur1, bnext1, flush);
    } else {
      auto none = [](auto) {};
      mfma_chunk<T, MI, NI, KS, KC, ROW, PS, D, false, -1, decltype(none)&, (RING > 6 ? 2 : 1)>(buf, a_off, wrsrc, bcur, bnext, tap_stride, kk_stride, lane16, bq, acc, none);
      if (more) activate_all(c0n, nbuf);
    }
    issue(c + 2, 2);
    if constexpr (QUARTERS) {
      grp[0] = grp[1]; grp[1] = grp[2];
      if (c + 3 < nchunks) { grp[2].a = next_group(); grp[2].b = next_group(); }
    }
    __syncthreads();          // other buffer staged; this one free for chunk c+2
  }

  // ---- epilogue: bias, residual, one rounding, store (through wavefront-private LDS patches over the tile buffers)
  if constexpr (!BIAS_EARLY) load_bias();
  float* patch = reinterpret_cast<float*>(smem) + wave * patch_floats(MI, NI);
  // statistics slot of this wavefront: [sample][group][spatial tile * WM + wave row], or by blocks of 4 rows x 8 pixels
  const int per_row = QUARTERS ? (p.w_out + 7) / 8 : p.tiles_x;   // slots of a row of blocks
  const int slot = QUARTERS ? ty0 / 4 * per_row + tx0 / 8 : tile * WM + wm;
  EpilogueParams ep;
  {
    const int elems = p.h * p.w_out * p.cout;   // of a sample
    char* y = reinterpret_cast<char*>(p.y) + (size_t)n * elems * sizeof(TO);
    ep.y = __builtin_amdgcn_make_buffer_rsrc(y, 0, (int)(elems * sizeof(TO)), 0x00020000);
    ep.planar = y;
    const char* res = reinterpret_cast<const char*>(p.res) + (size_t)n * elems * sizeof(T);
    ep.res = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(res), 0, (int)(elems * sizeof(T)), 0x00020000);
  }
  ep.h = p.h; ep.w = p.w_out; ep.cout = p.cout; ep.nchw = p.y_nchw != 0 && !p.res;
  ep.stats = p.stats ? p.stats + (size_t)n * p.stats_groups * p.stats_slots + slot : nullptr;
  ep.cpg = p.stats_cpg; ep.stats_stride = p.stats_slots; ep.pair_stride = per_row; ep.handed_over = p.rows_out != nullptr;
  auto store = [&](const f32x16 (&sums)[MI][NI]) {
    if (p.res) epilogue_store<T, TO, MI, NI, MTW, MTH, MT_PER_ROW, true, MODE>(sums, bias, patch, lane, wm * MI, ty0, tx0, co0 + wn * NI * 32, ep);
    else epilogue_store<T, TO, MI, NI, MTW, MTH, MT_PER_ROW, false, MODE>(sums, bias, patch, lane, wm * MI, ty0, tx0, co0 + wn * NI * 32, ep);
  };
  if constexpr (QUARTERS) store(total);
  else store(acc);

  if (p.rows_out) hand_over_row<NT>(p, n, wt.y, nt, co0, TN, WM, tid, lane);
}

template <typename T, typename TO, int TH, int TW, int WM, int WN, int NI, int KS, int KC, int RING = 0, int MODE = kPlain>
int launch_cfg(const ConvArgs& a, hipStream_t s) {
  constexpr int PAD = KS / 2;
  constexpr int TN = WN * NI * 32;
  MfmaParams p = conv_params(a, TH, TW, TN, WM, a.h, a.w);
  if (MODE == kQuarters) p.stats_slots = ((a.h + 3) / 4) * ((a.w + 7) / 8);
  WMDEC_REQUIRE(MODE != kQuarters || (!a.x2 && a.cin % 64 == 0), WMDEC_ERR_UNSUPPORTED, "conv_mfma: this form takes no shortcut");
  WMDEC_REQUIRE(MODE == kPlain || !a.rows_out, WMDEC_ERR_UNSUPPORTED, "conv_mfma: this tile hands over no rows");
  const int rc = check_hand_over(p);
  if (rc != WMDEC_OK) return rc;
  p.w = a.wt;
  p.w_bytes = (int)(packed_elems(KS * KS, a.cout, a.cin) * sizeof(T));
  if (a.x2) {
    WMDEC_REQUIRE(KS == 3 && a.w2 && a.cin2 > 0 && a.cin2 % KC == 0 && (long)a.h * a.w * a.cin2 < (1L << 29), WMDEC_ERR_UNSUPPORTED,
                  "conv_mfma: a folded shortcut needs a 3x3 convolution without upsampling and cin2 %% %d == 0", KC);
    p.x2 = a.x2; p.w2 = a.w2; p.bias2 = a.bias2; p.cin2 = a.cin2;
    p.w2_bytes = (int)(packed_elems(1, a.cout, a.cin2) * sizeof(T));
  }
  constexpr int NT = 64 * WM * WN;
  size_t smem = (((size_t)2 * tile_buf_elems(TH, TW, PAD, KC, m_tile_width(TW, MODE)) * 2 + 15) & ~(size_t)15) + (size_t)(a.cin + a.groups) * sizeof(float2);
  const size_t patch = (size_t)(WM * WN) * patch_floats(wave_m_tiles(TH, TW, WM), NI) * sizeof(float);   // epilogue patches of the wavefronts
  if (smem < patch) smem = patch;
  WMDEC_REQUIRE(smem <= 80 * 1024, WMDEC_ERR_UNSUPPORTED, "conv_mfma: %zu bytes of LDS needed", smem);
  void (*kern)(MfmaParams) = !p.norm ? conv_mfma_kernel<T, TO, TH, TW, WM, WN, NI, KS, KC, 0, MODE, RING>
                             : (a.silu ? conv_mfma_kernel<T, TO, TH, TW, WM, WN, NI, KS, KC, 2, MODE, RING>
                                       : conv_mfma_kernel<T, TO, TH, TW, WM, WN, NI, KS, KC, 1, MODE, RING>);
  // once per instantiation and activation mode (80 KiB: two workgroups per compute unit)
  static std::once_flag attr_once[3];
  hipError_t attr_err = hipSuccess;
  std::call_once(attr_once[!p.norm ? 0 : (a.silu ? 2 : 1)],
                 [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024); });
  WMDEC_HIP(attr_err);
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.total + warm_groups(p.next, WM * WN))), dim3(NT), smem, s, p);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

// Tile shapes: patch height x width, wavefront rows x columns, 32-channel tiles per wavefront.
struct TileShape { int th, tw, wm, wn, ni; };
enum TileId { T256x128 = 0, T128x128_ROW, T128x64_ROW, T128x64, T256x32, T128x128_1x4, T128x256, T64x128, T128x128_ROWS4, T96x128, T96x256, T128x128_PAIR, T128x256_PAIR, kNumTiles };
constexpr TileShape kTiles[kNumTiles] = {
    {8, 32, 2, 2, 2},    // T256x128: 256 pixels x 128 channels (large 1x1 convolutions)
    {4, 32, 2, 2, 2},    // T128x128_ROW: 128 x 128 on a 4x32 patch (1x1 convolutions)
    {4, 32, 4, 1, 2},    // T128x64_ROW: 128 x 64 on a 4x32 patch (1x1 convolutions)
    {8, 16, 4, 1, 2},    // T128x64: 128 x 64 on an 8x16 patch
    {8, 32, 4, 1, 1},    // T256x32: 256 x 32 (few output channels: the frame)
                         // the tiles of kernels_conv_rows.hip:
    {8, 16, 1, 4, 1},    // T128x128_1x4: 128 x 128, every wavefront all pixels x 32 channels: a weight fragment feeds all
                         //     rows, which keeps the fragment loads off the limit of the vector L1 (64 B/clk per compute unit)
    {8, 16, 1, 4, 2},    // T128x256: 128 x 256, every wavefront all pixels x 64 channels (see wide_channels); two workgroups per
                         //     compute unit
    {4, 16, 1, 4, 1},    // T64x128: 64 x 128, T128x128_1x4 at half the height, for launches of at most one workgroup per compute unit
    {8, 16, 1, 4, 1},    // T128x128_ROWS4: the same layers in larger batches
    {6, 16, 1, 4, 1},    // T96x128 and
    {6, 16, 1, 4, 2},    // T96x256: the two above at three quarters of the height, where a launch's last round is fuller with them (see six_eight_pair), and
    {8, 16, 1, 4, 1},    // T128x128_PAIR,
    {8, 16, 1, 4, 2},    // T128x256_PAIR: the same layers in other batches
};

// Layers whose 128 x 128 tiles leave half of the compute units empty at batch 1 and whose moments, per 4x16 block, are few
// enough for the consumer to merge: 64 x 128 tiles where the launch still fits one round, 128 x 128 otherwise, with the same
// order of summation and the same moments.  Measured, us, 64 x 128 against 128 x 128: 512 channels at 64x64 24.0 / 29.2, at
// 48x72 21.1 / 27.1, 256 channels at 68x92 11.7 / 16.0; past one round 31.3 / 29.1 (512 channels at 60x90).
// The smaller tile always has a whole chunk of weight fragments in flight: two MFMAs a k-step cover little of the latency of
// weights that are new to the L2 (256x256 frame 859 -> 853 us against half a chunk, 136x184 the same).
// The larger tile of the pair runs as T128x128_1x4 does (its moments take four rows each; ResBlocks of 2 to 8 samples within 0.6 % of each other).
bool four_row_slots(const ConvArgs& a) {
  const long blocks = (long)((a.h + 3) / 4) * ((a.w + 15) / 16);
  return a.ksize == 3 && !a.y_nchw && a.cout % 128 == 0 && !a.rows_out && !a.wide_tiles && blocks <= 128 && blocks * (a.cout / 128) <= 256;
}

// 128 or 256 channels a workgroup where the layer has both: whichever walks its rounds sooner.  With 256 a staged patch feeds twice the
// channels, half the normalise + SiLU work and input traffic per MFMA, so that a compute unit takes 1.8 times the time of a 128-channel tile per
// 256-channel tile instead of twice; but tiles are dealt to 256 compute units in larger pieces.  us, 128 / 256 channels,
// 256 -> 256 channels, by the number of 256-channel tiles: 180 29.1 / 26.7, 250 32.9 / 31.7, 260 42.3 / 48.2, 380 48.2 / 50.7, 420 57.9 / 52.6,
// 510 62.9 / 57.7, 520 70.8 / 75.8, 640 76.0 / 77.3, 700 86.4 / 80.5, 800 99.1 / 99.7, 900 111.8 / 102.6, 1100 129.2 / 126.5; 512 -> 512: 120
// 32.9 / 48.6, 220 56.6 / 52.9, 300 79.8 / 88.5, 480 113 / 102, 1440 320 / 290.  Both add a sum's products in the same order and leave the same
// moments per 8x16 block, so the batch may decide.  With a residual the epilogue of 256 channels waits for more of it: 256 channels lose where
// there are few products beside it (400x400, 128 / 256 channels: 32 -> 256 36.5 / 42.7, 128 -> 256 88.3 / 86.5; 256x256 16.8 / 18.5, 39.6 / 38.9).
// Where the rows' moments are merged by the launch itself, its ticket counters are sized for one sample's choice by its pixels alone (fits_wide)
// and the launch keeps to it: never more channel tiles than that.  (Between 513 and 640 tiles that is the slower of the two, by 4 to 9 %.)
bool fits_wide(const ConvArgs& a) { return a.cout % 256 == 0 && (((long)a.h * a.w + 127) / 128) * (a.cout / 256) >= 2 * 256; }
bool wide_channels(const ConvArgs& a) {
  if (a.cout % 256 != 0) return false;
  if (a.rows_out && fits_wide(a)) return true;
  if (a.res && a.cin < 128) return false;
  const long tiles = (long)((a.h + 7) / 8) * ((a.w + 15) / 16) * (a.cout / 256) * a.n;
  return 9 * ((tiles + 255) / 256) <= 5 * ((2 * tiles + 255) / 256);
}

// Tiles of six rows for launches of few rounds: a tile takes four fifths of the time of eight rows (the fixed parts and the weights are the same), and a launch takes
// as long as its fullest compute unit, so six rows are ahead where their tiles need no more rounds.  The estimate, which the batch may follow (y is the same with every
// tile, and both heights leave the same moments, see kSixEight), counts rounds of 256 tiles; tiles of 256 channels take 9 / 5 of 128.
// us, eight / six rows, SiLU, residual, without moments: 512 channels 60x90 29.0 / 27.2, two samples 47.9 / 43.0, three 75.6 / 67.4, four 85.2 / 81.1; 54x80 26.9 / 23.5, 50x90 27.0 / 23.6,
// 90x120 48.1 / 43.1, 80x100 47.3 / 43.8; 256 channels 100x100 15.7 / 13.9, 120x180 28.1 / 25.8; 512 -> 256 at 120x180 51.8 / 49.1; 128 channels 160x200 15.4 / 13.4;
// where the estimate says eight: 512 channels 62x90 27.6 / 37.9, 90x160 54.8 / 63.1, eight samples of 60x90 152.6 / 158.3; 128 channels 136x184 10.5 / 13.0, 240x360 24.7 / 26.6.
// Which layers may change their height is a function of the sample alone (its moments depend on it): those that gain at one sample, of at most two rounds (120x180 of
// 512 channels: 83.1 / 80.8, which larger batches would lose again), from 128 input channels on and not widening, where the products outweigh the fixed parts.
// Layers with fp32 output stay with eight rows, and so do a decoder's that leave moments where the launch merges its rows itself (256 channels at 120x180), where their consumer can read
// the fewer triples of eight rows only (512 channels at 72x128, 80x100, 90x120) or where the workspace would grow (see fuse_stats), and a caller's whose workspace holds those of eight.
// What the second triple of a tile costs the eight-row forms: ResBlocks of 512 channels at 60x90, eight samples, 329.5 -> 332, 128 channels at 160x200, three, 81.2 -> 82.8;
// with six rows, one sample, 512 channels at 60x90 67.5 -> 65.9, 54x80 70.0 -> 61.3, 90x120 113.5 -> 107.1, 512 -> 256 at 100x100 62.3 -> 60.0, 128 at 160x200 46.8 -> 43.7.
struct TileCost { int cost; bool wide; };
TileCost tile_cost(const ConvArgs& a, int th, int n) {   // in fifths of the time of a 128 x 128 tile
  const long tiles = (long)((a.h + th - 1) / th) * ((a.w + 15) / 16) * n, narrow = tiles * (a.cout / 128), wide = tiles * (a.cout / 256);
  const long c1 = (narrow + 255) / 256 * (th == 6 ? 4 : 5), c2 = (wide + 255) / 256 * (th == 6 ? 7 : 9);
  const bool only_wide = th == 6 && narrow > 2 * 256;    // (six rows of 128 channels come with the whole-chunk ring alone)
  if (a.cout % 256 != 0) return {only_wide ? 1 << 30 : (int)c1, false};
  return only_wide || c2 < c1 ? TileCost{(int)c2, true} : TileCost{(int)c1, false};
}
bool six_eight_pair(const ConvArgs& a) {
  if (a.ksize != 3 || a.cout % 128 != 0 || a.y_nchw || a.y_dtype == WMDEC_F32 || a.rows_out || a.wide_tiles || a.eight_rows) return false;
  if (a.cin < 128 || a.cin < a.cout) return false;
  if ((long)((a.h + 7) / 8) * ((a.w + 15) / 16) * (a.cout / 128) > 2 * 256) return false;
  return tile_cost(a, 6, 1).cost < tile_cost(a, 8, 1).cost;
}

// which tile shape a launch uses: a function of the per-sample shape only, so that the order of a summation does not depend on the
// batch, but for the pairs above
TileId pick_tile(const ConvArgs& a) {
  const long px = (long)a.h * a.w;
  const bool n128 = a.cout % 128 == 0;
  if (a.ksize == 3) {
    if (a.cout <= 32) return T256x32;
    if (four_row_slots(a))
      return (long)((a.h + 3) / 4) * ((a.w + 15) / 16) * (a.cout / 128) * a.n <= 256 ? T64x128 : T128x128_ROWS4;
    if (six_eight_pair(a)) {
      const TileCost six = tile_cost(a, 6, a.n);
      if (six.cost < tile_cost(a, 8, a.n).cost) return six.wide ? T96x256 : T96x128;
      return wide_channels(a) ? T128x256_PAIR : T128x128_PAIR;
    }
    if (wide_channels(a)) return T128x256;
    return n128 ? T128x128_1x4 : T128x64;
  }
  if (n128 && a.cin % 64 == 0 && px * (a.cout / 128) >= 256L * 256 * 2) return T256x128;
  return n128 ? T128x128_ROW : T128x64_ROW;
}

ConvMode mode_of(TileId t) { return t == T64x128 || t == T128x128_ROWS4 ? kRows4 : t >= T96x128 && t <= T128x256_PAIR ? kSixEight : kPlain; }

// The 128x128 tiles with a whole chunk of weight fragments in flight (see RING in kernels_conv_rows.hip): launches of at most two workgroups
// per compute unit, in their order of summation the same as the others, so that the batch may decide.  us, whole chunk / two steps ahead, with the
// weights in the L2: 512 channels at 60x90 32.4 / 34.1, two samples 53.4 / 54.5, 256 channels at 120x180 28.3 / 29.3; in a decoder run,
// where they are not, the difference is larger (the ten such layers of a 480x720 frame: 30 us when both rings were longer).
// The eight-row tiles that share their moments with six rows from 256 input channels on: below that a launch has too few chunks for it to pay.  us, whole
// chunk / two steps, three samples of 128 output channels at 131x145, with residual: f16 512 -> 128 59.0 / 60.4, bf16 58.6 / 59.0; four at 49x286, f16 256 -> 128 32.1 / 32.6, bf16 as
// fast; 128 -> 128 19.1 / 19.0 and 18.9 / 18.7, with moments 22.7 / 22.7 and 22.9 / 22.6.
bool whole_chunk_ring(const ConvArgs& a) {
  const TileId t = pick_tile(a);
  if (t == T96x128) return true;
  if (t != T128x128_1x4 && t != T128x128_ROWS4 && !(t == T128x128_PAIR && a.cin >= 256)) return false;
  const long wgs = (long)((a.h + 7) / 8) * ((a.w + 15) / 16) * (a.cout / 128) * a.n;
  return wgs <= 2 * 256;
}

template <typename T, typename TO>
int launch_3x3(const ConvArgs& a, hipStream_t s) {
  const TileId t = pick_tile(a);
  if (t == T128x64) return launch_cfg<T, TO, 8, 16, 4, 1, 2, 3, 32>(a, s);
  if (t == T256x32) return launch_cfg<T, TO, 8, 32, 4, 1, 1, 3, 32>(a, s);
  return launch_conv_rows(a, kTiles[t].th, kTiles[t].ni, mode_of(t), t == T64x128 || whole_chunk_ring(a), s);
}

// chunk of input channels a 1x1 launch stages at a time: 64 halves the barriers
int chunk_1x1(const ConvArgs& a) { return a.cin % 64 == 0 ? 64 : 32; }

template <typename T, typename TO>
int launch_1x1(const ConvArgs& a, hipStream_t s) {
  const TileId t = pick_tile(a);
  if (chunk_1x1(a) == 64) {
    if (t == T256x128) return launch_cfg<T, TO, 8, 32, 2, 2, 2, 1, 64>(a, s);
    if (t == T128x128_ROW) return launch_cfg<T, TO, 4, 32, 2, 2, 2, 1, 64>(a, s);
    return launch_cfg<T, TO, 4, 32, 4, 1, 2, 1, 64>(a, s);
  }
  if (t == T128x128_ROW) return launch_cfg<T, TO, 4, 32, 2, 2, 2, 1, 32>(a, s);
  return launch_cfg<T, TO, 4, 32, 4, 1, 2, 1, 32>(a, s);
}

template <typename T>
int launch_type(const ConvArgs& a, hipStream_t s) {
  if (a.y_dtype == WMDEC_F32) return a.ksize == 3 ? launch_3x3<T, float>(a, s) : launch_1x1<T, float>(a, s);
  return a.ksize == 3 ? launch_3x3<T, T>(a, s) : launch_1x1<T, T>(a, s);
}

}  // namespace

bool conv_mfma_supported(const ConvArgs& a) {
  if (!is_16bit(a.op_dtype) || a.x_dtype != a.op_dtype || a.upsample) return false;
  if (a.res && a.res_dtype != a.op_dtype) return false;
  if (a.y_dtype != a.op_dtype && a.y_dtype != WMDEC_F32) return false;
  if (a.x_nchw) return false;
  if (a.y_nchw && !(a.cout <= 32 && a.y_dtype == WMDEC_F32 && !a.res && a.ksize == 3)) return false;
  if (a.cin % 32 != 0) return false;
  if (a.cout % 64 != 0 && !(a.y_nchw && a.cout <= 32)) return false;
  if (a.cin > 2048) return false;   // scale/shift table lives in LDS
  if (a.ksize != 1 && a.ksize != 3) return false;
  if (!packed_offsets_fit(a.ksize * a.ksize, a.cout, a.cin, a.op_dtype) || !packed_offsets_fit(1, a.cout, a.cin2, a.op_dtype)) return false;
  if ((long)a.h * a.w * a.cin >= (long)kOutside || (long)a.h * a.w * a.cout >= (long)kOutside) return false;   // 32-bit byte offsets per sample
  return true;
}

int conv_mfma_stats_slots(const ConvArgs& a) {
  if (!conv_mfma_supported(a) || a.y_nchw || a.stats_groups <= 0 || a.cout % a.stats_groups != 0) return 0;
  const int cpg = a.cout / a.stats_groups;
  if ((cpg & (cpg - 1)) != 0 || cpg > 32) return 0;   // a group must sit inside one wavefront's 64-channel run
  const TileId t = pick_tile(a);
  const TileShape& ts = kTiles[t];
  if (mode_of(t) == kRows4) return ((a.h + 3) / 4) * ((a.w + 15) / 16);
  if (mode_of(t) == kSixEight) return (six_eight_run(a.h - 1) + 1) * ((a.w + 15) / 16);
  return ((a.w + ts.tw - 1) / ts.tw) * ((a.h + ts.th - 1) / ts.th) * ts.wm;
}

// tile rows / channel tiles of a launch: the extents of the row moments it can leave and of its ticket counters
void conv_mfma_row_extents(const ConvArgs& a, int* tile_rows, int* channel_tiles, int* tiles_per_row) {
  TileId t = pick_tile(a);
  if (t == T128x256 || t == T128x128_1x4 || mode_of(t) == kSixEight) t = fits_wide(a) ? T128x256 : T128x128_1x4;   // (launches that merge rows take no tile of that pair)
  const TileShape& ts = kTiles[t];
  const int tn = ts.wn * ts.ni * 32;
  *tile_rows = (a.h + ts.th - 1) / ts.th;
  *channel_tiles = (a.cout + tn - 1) / tn;
  *tiles_per_row = (a.w + ts.tw - 1) / ts.tw;
}

void conv_mfma_grid(const ConvArgs& a, NextWeights* next) {
  const TileShape& ts = kTiles[pick_tile(a)];
  next->per_tile = ((a.h + ts.th - 1) / ts.th) * ((a.w + ts.tw - 1) / ts.tw) * a.n;
  next->tile_blocks = ts.wn * ts.ni;
  next->total = next->per_tile * ((a.cout + 32 * next->tile_blocks - 1) / (32 * next->tile_blocks));
}

// the instantiation a launch would use, spelled like a profiler prints it
const char* conv_mfma_label(const ConvArgs& a) {
  static thread_local char buf[160];
  const TileId t = pick_tile(a);
  const int kc = a.ksize == 1 ? chunk_1x1(a) : 32;
  const TileShape& ts = kTiles[t];
  const char* ty = a.op_dtype == WMDEC_BF16 ? "wmdec::bf16_t" : "wmdec::f16_t";
  const int act = a.mean == nullptr && a.rows_in == nullptr && !a.groups_norm ? 0 : (a.silu ? 2 : 1);
  snprintf(buf, sizeof(buf), "conv_mfma_kernel<%s, %s, %d, %d, %d, %d, %d, %d, %d, %d, %d, %d>", ty,
           a.y_dtype == WMDEC_F32 ? "float" : ty, ts.th, ts.tw, ts.wm, ts.wn, ts.ni, a.ksize, kc, act,
           mode_of(t), a.ksize == 3 && whole_chunk_ring(a) ? 18 : t == T64x128 ? 18 : 0);
  return buf;
}

int launch_conv_quarters(const ConvArgs& a, hipStream_t s) {
  WMDEC_REQUIRE(conv_mfma_supported(a) && a.ksize == 3 && !a.y_nchw && a.cout % 128 == 0, WMDEC_ERR_UNSUPPORTED, "conv_mfma: no layer for this form");
  if (a.op_dtype == WMDEC_BF16)
    return a.y_dtype == WMDEC_F32 ? launch_cfg<bf16_t, float, 8, 16, 1, 4, 1, 3, 32, 9, kQuarters>(a, s) : launch_cfg<bf16_t, bf16_t, 8, 16, 1, 4, 1, 3, 32, 9, kQuarters>(a, s);
  return a.y_dtype == WMDEC_F32 ? launch_cfg<f16_t, float, 8, 16, 1, 4, 1, 3, 32, 9, kQuarters>(a, s) : launch_cfg<f16_t, f16_t, 8, 16, 1, 4, 1, 3, 32, 9, kQuarters>(a, s);
}

int launch_conv_mfma(const ConvArgs& a, hipStream_t s) {
  return a.op_dtype == WMDEC_BF16 ? launch_type<bf16_t>(a, s) : launch_type<f16_t>(a, s);
}

}  // namespace wmdec
