// 3x3 convolution on 16x16x32 MFMAs: a wavefront holds all rows of a 16-pixel-wide patch.
//
// The form that the large layers take (128 output channels and more a workgroup; tiles of 8, 6 or 4 rows).  GEMM view, staging, statistics and epilogue semantics
// are those of kernels_conv_mfma.hip: a workgroup of four wavefronts owns TH rows x 16 pixels and 128 * NI output channels, 32 * NI a
// wavefront; per chunk of 32 input channels the patch plus halo goes through one of two LDS buffers, normalised and
// activated once per element, and the nine taps are swept over it.
//
// Why this MFMA: the power limit decides the clock of these kernels, and 16x16x32 does a sixth more under it than 32x32x16
// (operands in registers, values as in a layer: 1.95 against 1.68 PFLOP/s, at 1.95 and 1.70 GHz).  One MFMA takes 32 channels of a row of
// 16 pixels and 16 output channels.
// A = pixels, B = weights: lane l then holds four consecutive pixels, 4 (l / 16) .. + 3, of one output channel of a tile; the two tiles of 32
// channels take the even and the odd ones, so that it is channels 2 (l % 16) and the next.  Residual and output move as pairs
// straight from the accumulators, 16 consecutive lanes on the 64 contiguous bytes of a pixel.  (With the operands the other way round a
// lane holds eight channels of one pixel, a 16-byte vector, but the four lanes on a pixel's 64 bytes are 16 lanes apart: every vector is
// a request of its own, and the moments of eight channels a lane spilled registers of the fullest forms.  us, that / this: plain input, 32 -> 128
// channels at 480x720 34.4 / 29.4, with residual 40.4 / 35.8; 32 -> 256 eight samples of 68x92 19.7 / 12.7, with moments 28.1 / 19.2; with
// SiLU, 256 -> 256 at the same size 58.3 / 56.9, 65.0 / 63.5.)
#include <stdio.h>

#include <mutex>

#include "conv_moments.hpp"

namespace wmdec {
namespace {

// LDS layout of a staged patch: 96 bytes from pixel to pixel.  A fragment is 16 pixels x 32 channels, lanes i and i + 16 a channel octet
// apart; 96 bytes serve that in one pass (4 cycles a KiB, measured), 64, 80 and 144 bytes in two.  One pixel slot behind the patch is spare:
// vectors outside the image are stored there.
constexpr int kChunk = 32;                 // input channels of a chunk
constexpr int PS = kChunk + 16;            // elements from pixel to pixel
constexpr int PW = 18, ROW = PW * PS;      // pixels, elements of a row of the patch
constexpr int buf_elems(int th) { return (th + 2) * ROW + PS; }

// Three workgroups per compute unit leave 168 registers: the offsets of the vectors that a thread stages then wait in LDS for their
// place in a sweep (the compiler would spill them, and wait for every load in flight where it takes them back).
constexpr int resident_workgroups(int th, int ni, int ring) { return th * ni <= 8 && ring == 0 ? 3 : 2; }
constexpr bool park_offsets(int th, int ni, int ring) { return resident_workgroups(th, ni, ring) == 3; }
constexpr size_t fixed_lds(int th, int ni, int ring) {   // patches, bias, parked offsets; the table of the activation lies behind them
  return (size_t)2 * buf_elems(th) * 2 + (size_t)128 * ni * sizeof(float) + (park_offsets(th, ni, ring) ? 2 * 256 * 16 : 0);
}

// byte offset, from the chunk's first fragment, of the weights of step s = (tap column, tap row, ni)
template <int NI> __device__ __forceinline__ int weight_offset(int s, int tap_stride) {
  return (s / NI % 3 * 3 + s / (3 * NI)) * tap_stride + s % NI * 1024;
}

// MFMA work of one staged chunk: 9 NI steps, each 2 R MFMAs with the weights of a tap and 32 output channels.
// One tap row further down, row r reads what row r + 1 reads here: R + 2 fragments serve the three taps of a column.  Steps
// run over ni innermost, then the tap rows, then the tap columns.  The fragments of the chunk's three columns are
// numbered on and kept in a ring: number q takes the place of q - SLOTS behind the last MFMA of that one (which is in the last of the NI
// steps of a tap: with two of them, all R fragments of a tap must have a place).  With eight rows
// seven places leave at least 12 MFMAs between a read and its use, eight 14, with four rows six leave 10.
// Weights are requested D - 1 steps ahead, into a ring that persists across chunks: on entry it holds steps 0 .. D - 2 of this chunk, on
// exit those of the chunk at `bnext` (LAST: there is none).
// The order is pinned as written, slice(m) behind MFMA m.
template <typename T, int R, int NI, int D, bool LAST, typename Slice>
__device__ __forceinline__ void sweep_chunk(const T* buf, __amdgpu_buffer_rsrc_t wrsrc, int bcur, int bnext, int tap_stride, int lane_w,
                                            u32x4 (&bq)[D][2], f32x4 (&acc)[R][2 * NI], Slice&& slice) {
  constexpr int STEPS = 9 * NI, FRAGS = R + 2, SLOTS = R < 8 ? FRAGS : NI == 1 ? R - 1 : R;
  static_assert(STEPS % D == 0, "the ring position must be the same at every chunk start");
  u32x4 af[SLOTS];
  auto read = [&](auto q_c) {
    constexpr int q = decltype(q_c)::value;
    af[q % SLOTS] = *reinterpret_cast<const u32x4*>(buf + q % FRAGS * ROW + q / FRAGS * PS);
  };
  static_for<SLOTS>(read);
  static_for<STEPS>([&](auto s_c) {
    constexpr int s = decltype(s_c)::value, g = s / (3 * NI), ky = s / NI % 3, ni = s % NI, sp = s + D - 1;
    if constexpr (!LAST || sp < STEPS) {
      const int at = (sp < STEPS ? bcur : bnext) + weight_offset<NI>(sp % STEPS, tap_stride);
#pragma unroll
      for (int h = 0; h < 2; ++h) bq[sp % D][h] = load_fragment(wrsrc, lane_w, at + 16 * h);
    }
    __builtin_amdgcn_sched_barrier(0);
    // row r is the last to read its fragment, and there is one to take its place
    constexpr auto last = [](int r) constexpr { return ni == NI - 1 && (ky == 2 || r == 0) && g * FRAGS + r + ky + SLOTS < 3 * FRAGS; };
    static_for<R>([&](auto r_c) {
      constexpr int r = decltype(r_c)::value;
      static_for<2>([&](auto h_c) {
        constexpr int h = decltype(h_c)::value;
        acc[r][2 * ni + h] = Mma<T>::m16(af[(g * FRAGS + r + ky) % SLOTS], bq[s % D][h], acc[r][2 * ni + h]);
        if constexpr (h == 1 && last(r)) read(std::integral_constant<int, g * FRAGS + r + ky + SLOTS>{});
        slice(std::integral_constant<int, (s * R + r) * 2 + h>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  });
}

// Rows of the residual that the last sweep requests, a pixel of the lane behind each of its last MFMAs; the epilogue requests the others in
// front of its first store.  (More of them in the sweep would be spilled where the accumulators are 128 registers, or the values to store as many as the
// accumulators.  Requested between the stores, each as the one four rows before it is used up, a row waits for the stores in front of it:
// what the residual costs 256-channel tiles, us, that way / this way: 256 -> 256 channels 150x150 4.9 / 2.1 beside 26 to 29, 480x480 34 / 14 beside 202 to 233, 32 -> 256 at
// 400x400 16 / 11 beside 31, 512 -> 512 at 106x82 3.4 / 1.6 beside 48 to 50.)
constexpr int asked_rows(int th, int ni, size_t out_size) { return ni == 1 && out_size == 2 ? th : 4; }

struct EpilogueParams {
  __amdgpu_buffer_rsrc_t res, y;           // the sample's residual and output, with its size: accesses outside are dropped
  int h, w, cout;
  Moments* stats; int cpg, stats_stride, row_stride;
  int cut;                                 // (kSixEight) row of the tile with which its second triple begins; R or more: there is none
  bool handed_over;
};

// element offset of a lane's channels at pixel i of its four, from channel 0 of the tile's first pixel; outside the image: kOutside
__device__ __forceinline__ unsigned lane_offset(const EpilogueParams& p, int lane, int tx0, int i) {
  const int px = 4 * (lane >> 4) + i;
  return tx0 + px < p.w ? (unsigned)(px * p.cout + 2 * (lane & 15)) : kOutside;
}
// the residual of channels co .. co + 31 of a row's pixels i (rows past the image take the last one's: no output is made of it)
template <typename T> __device__ __forceinline__ uint32_t load_residual(const EpilogueParams& p, unsigned at, int row, int tx0, int co) {
  return __builtin_amdgcn_raw_buffer_load_b32(p.res, (int)(at * sizeof(T)), vector_base(row, tx0, p.h, p.w, p.cout, co) * (int)sizeof(T), 0);
}

// Epilogue of one wavefront: bias, residual, one rounding, store.  (Through LDS
// patches, as in kernels_conv_mfma.hip, the same lanes write 64 values one by one and wait for them.)  The bias is added to
// the finished sums: accumulators that start from it round every partial sum at its exponent.
// rv: the residual; that of the first rows is on its way.
// Moments, of the values as stored: one triple per group for all R rows, or (kRows4) for every four of them, or (kSixEight) for the rows in front of
// `cut` and those from it on.  FULL: no pixel of the patch lies
// outside the image (the moments need no masks, and the rows are scheduled as one).
template <typename T, typename TO, int R, int NI, bool RES, bool STATS, bool FULL, int MODE>
__device__ __forceinline__ void epilogue(const f32x4 (&acc)[R][2 * NI], uint32_t (&rv)[NI * R][4], const float* s_bias, int lane, int ty0, int tx0, int co_w,
                                         const EpilogueParams& p) {
  constexpr int EMIT = MODE == kRows4 ? 4 : R;   // rows of a triple
  static_assert(R % EMIT == 0, "whole triples");
  const bool columns = tx0 + 16 <= p.w;                           // all columns lie inside the image,
  const int cols = min(max(p.w - tx0 - 4 * (lane >> 4), 0), 4);   // and of the lane's four so many
  unsigned at[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) at[i] = lane_offset(p, lane, tx0, i);
  if constexpr (RES) {
#pragma unroll
    for (int k = asked_rows(R, NI, sizeof(TO)); k < NI * R; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) rv[k][i] = load_residual<T>(p, at[i], ty0 + k % R, tx0, co_w + 32 * (k / R));
    __builtin_amdgcn_sched_barrier(0);
  }
  constexpr int TRIPLES = MODE == kSixEight ? 2 : R / EMIT;
  constexpr bool EACH = MODE == kSixEight && NI * R > 12;   // the triples are written 32 channels at a time: beside the accumulators those of all would be spilled
  LaneMoments<2> st[(EACH ? 1 : NI) * TRIPLES];
  Moments* dst[(EACH ? 1 : NI) * TRIPLES];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    const float2 bias = *reinterpret_cast<const float2*>(s_bias + 32 * ni + 2 * (lane & 15));
#pragma unroll
    for (int t = 0; t < R / EMIT; ++t) {
      float n = 0.f, shift[2] = {0.f, 0.f}, s[2][4] = {}, q[2][4] = {};
      auto close = [&](LaneMoments<2>& own) __attribute__((always_inline)) {
        if (STATS && !FULL) {   // a column outside the image has a sum of its own
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) { s[e][i] = i < cols ? s[e][i] : 0.f; q[e][i] = i < cols ? q[e][i] : 0.f; }
        }
        own.n = n;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          own.shift[e] = shift[e];
          own.s[e] = (s[e][0] + s[e][1]) + (s[e][2] + s[e][3]);
          own.q[e] = (q[e][0] + q[e][1]) + (q[e][2] + q[e][3]);
        }
      };
      LaneMoments<2> front{};   // (kSixEight) the rows in front of the cut, once it is behind
#pragma unroll
      for (int r = t * EMIT; r < (t + 1) * EMIT; ++r) {
        if (!FULL && ty0 + r >= p.h) continue;
        const int base = vector_base(ty0 + r, tx0, p.h, p.w, p.cout, co_w + 32 * ni) * (int)sizeof(TO);
        float v[4][2];   // as stored
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[i][0] = acc[r][2 * ni][i] + bias.x;
          v[i][1] = acc[r][2 * ni + 1][i] + bias.y;
          if constexpr (RES) { v[i][0] += unpack_lo<T>(rv[ni * R + r][i]); v[i][1] += unpack_hi<T>(rv[ni * R + r][i]); }
          if constexpr (sizeof(TO) == 4) {
            f32x2 pair{v[i][0], v[i][1]};
            asm volatile("" : "+v"(pair));   // (in this order: the compiler would form all pairs first)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, pair), p.y, (int)(at[i] * sizeof(TO)), base, 0);
            v[i][0] = pair[0]; v[i][1] = pair[1];
          } else {
            uint32_t word = pack2<T>(v[i][0], v[i][1]);
            asm("" : "+v"(word));   // (the stored values are taken from it: the compiler would convert each once more)
            __builtin_amdgcn_raw_buffer_store_b32(word, p.y, (int)(at[i] * sizeof(TO)), base, 0);
            v[i][0] = unpack_lo<T>(word); v[i][1] = unpack_hi<T>(word);
          }
        }
        if constexpr (STATS) {
          if constexpr (MODE == kSixEight) {
            if (r > 0 && r % 2 == 0 && r == p.cut) {   // (uniform)
              close(front);
              n = 0.f;
#pragma unroll
              for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) { s[e][i] = 0.f; q[e][i] = 0.f; }
            }
          }
          n += FULL ? 4.f : (float)cols;
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            // Shifted by the mean of the lane's first four pixels, a fourth of whichever is far off; in a ragged patch by the first (outside the image only if
            // all pixels of the lane are).
            if (r == t * EMIT || (MODE == kSixEight && r % 2 == 0 && r == p.cut)) shift[e] = FULL || columns ? 0.25f * ((v[0][e] + v[1][e]) + (v[2][e] + v[3][e])) : v[0][e];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float d = v[i][e] - shift[e];
              s[e][i] += d; q[e][i] = fmaf(d, d, q[e][i]);
            }
          }
        }
      }
      if constexpr (MODE == kSixEight) {
        const bool two = p.cut < R && (FULL || ty0 + p.cut < p.h);
        constexpr int STEP = EACH ? 0 : 2;
        LaneMoments<2> rear;
        close(rear);
        LaneMoments<2>& lead = st[STEP * ni];   // (value by value: of the two as a whole the compiler would select an address)
        lead.n = two ? front.n : rear.n;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          lead.shift[e] = two ? front.shift[e] : rear.shift[e];
          lead.s[e] = two ? front.s[e] : rear.s[e];
          lead.q[e] = two ? front.q[e] : rear.q[e];
        }
        rear.n = two ? rear.n : 0.f;
        st[STEP * ni + 1] = rear;
        dst[STEP * ni] = p.stats + (size_t)(32 * ni / p.cpg) * p.stats_stride;
        dst[STEP * ni + 1] = two ? dst[STEP * ni] + p.row_stride : nullptr;
        if constexpr (STATS && EACH) emit_pairs(st, false, lane, co_w, dst, p.cpg, p.stats_stride, p.handed_over);
      } else {
        close(st[ni * TRIPLES + t]);
        dst[ni * TRIPLES + t] = FULL || MODE != kRows4 || ty0 + t * EMIT < p.h   // (kRows4: rows past the image have no slot)
                                    ? p.stats + t * p.row_stride + (size_t)(32 * ni / p.cpg) * p.stats_stride : nullptr;
      }
    }
  }
  if constexpr (STATS && !EACH) emit_pairs(st, FULL && MODE != kSixEight, lane, co_w, dst, p.cpg, p.stats_stride, p.handed_over);
}

// ACT: what happens to an input element on its way into LDS: 0 nothing, 1 scale/shift, 2 scale/shift + SiLU
// RING: 0 = weights two steps ahead; otherwise the length of the weight ring in k-steps of 16 channels (18: a whole chunk).  The
// whole-chunk ring is for launches that leave a compute unit at most two workgroups: there a wavefront
// is alone on its SIMD, nothing else hides the latency of weights that come from beyond the L2 (every layer's weights
// are new to the L2 inside a decoder run), and the registers of the third workgroup are free for it.
// (TW, WM, WN, KS, KC: always 16, 1, 4, 3, 32; the name of an instantiation reads as those of kernels_conv_mfma.hip do.)
template <typename T, typename TO, int TH, int TW, int WM, int WN, int NI, int KS, int KC, int ACT, int MODE, int RING>
__global__ __launch_bounds__(256, resident_workgroups(TH, NI, RING)) void conv_mfma_kernel(MfmaParams p) {
  static_assert(TW == 16 && WM == 1 && WN == 4 && KS == 3 && KC == kChunk, "one layout");
  constexpr int NT = 256, HP = PW * (TH + 2), TN = 128 * NI;
  constexpr int VPP = KC / 8;                        // 16-byte vectors per pixel per chunk
  constexpr int NV = (HP * VPP + NT - 1) / NT;       // vectors a thread stages per chunk
  constexpr int BUF = buf_elems(TH), SPARE = (TH + 2) * ROW;
  constexpr int D = RING > 0 ? RING / 2 * NI : 3;    // weight ring, steps
  constexpr bool PARK = park_offsets(TH, NI, RING);
  static_assert(!PARK || NV == 3, "three offsets of either kind");

  fetch_arguments<sizeof(MfmaParams)>();
  extern __shared__ __align__(16) unsigned char smem[];
  T* s_a = reinterpret_cast<T*>(smem);                                          // [2][BUF]
  float* s_bias = reinterpret_cast<float*>(smem + 2 * BUF * 2);                 // [TN]
  u32x4* s_off = reinterpret_cast<u32x4*>(s_bias + TN);                         // [2][NT] offsets (PARK)
  float2* s_ab = reinterpret_cast<float2*>(smem + fixed_lds(TH, NI, RING));     // [cin] (scale, shift)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wn = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform: keeps the per-wave addresses scalar

  if (p.next.w && (int)blockIdx.x >= p.total) { warm_weights(p.next, p.total, WN, wn, lane); return; }   // (carries_weights: spilled registers of the fullest form)

  const WorkTile wt = workgroup_tile(p);
  const int nt = wt.nt, n = wt.n, tile = wt.tile;
  const int ty0 = wt.y * TH, tx0 = wt.x * TW;
  const int co0 = nt * TN, co_w = co0 + wn * NI * 32;

  if (tid < TN) s_bias[tid] = (p.bias ? p.bias[co0 + tid] : 0.f) + (p.bias2 ? p.bias2[co0 + tid] : 0.f);

  // ---- weights: the wavefront's fragment column (wave-uniform), and the lane's 16 bytes in tile 0 (the even channels) of a pair of fragments
  const int kk_stride = p.cout_blocks * 1024, tap_stride = p.cin_blocks * kk_stride;   // bytes
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, p.w_bytes, 0x00020000);
  const int wcol = (co_w >> 5) * 1024;
  const int lane_w = (lane >> 5) * kk_stride + (2 * (lane & 15) + 2 * (lane & 16)) * 16;
  u32x4 bq[D][2];
  f32x4 acc[TH][2 * NI];
  auto first_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int sp = 0; sp < D - 1; ++sp)
#pragma unroll
      for (int h = 0; h < 2; ++h) bq[sp][h] = load_fragment(wrsrc, lane_w, wcol + weight_offset<NI>(sp, tap_stride) + 16 * h);
  };
  // Two steps of weights come first; a whole chunk of them (RING) behind input and moments, which are needed before them: loads return in order, and
  // it is a thousand cycles of a compute unit's load path.  Without normalisation there is no table to wait for, and it comes first too (us, first / behind the
  // input, bf16: 1024 -> 384 channels at 40x120 30.9 / 34.1, 512 -> 384 at 53x149 25.0 / 27.2).
  if constexpr (RING == 0 || ACT == 0) first_weights();

  // ---- staging: a thread owns NV (pixel, channel-octet) vectors of the halo patch; the octet is the same for all.
  // Zero padding without per-element work: a vector outside the image is loaded from pixel 0 (a load under a lane
  // mask would make the compiler wait for it at the end of the branch), activated like any other, and stored to
  // the spare pixel slot behind the patch; its real slot is zeroed once, here, in both buffers.
  const int cvec = tid % VPP;
  const char* xin = reinterpret_cast<const char*>(p.x) + (size_t)n * p.h * p.w_out * p.cin * sizeof(T);   // uniform base
  int src_off[NV];          // byte offset of the vector in the first chunk of x
  int dst_off[NV];          // element offset of its slot in a patch
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int hp = (tid + i * NT) / VPP;
    const int hy = hp / PW, hx = hp % PW;
    const int gy = ty0 + hy - 1, gx = tx0 + hx - 1;
    const int at = hy * ROW + hx * PS;
    const bool in_patch = hp < HP, inside = in_patch & ((unsigned)gy < (unsigned)p.h) & ((unsigned)gx < (unsigned)p.w_out);   // (no branches)
    src_off[i] = (inside ? gy * p.w_out + gx : 0) * p.cin * (int)sizeof(T) + cvec * 16;
    dst_off[i] = (inside ? at : SPARE) + cvec * 8;
    if (in_patch & !inside) {
      *reinterpret_cast<u32x4*>(s_a + at + cvec * 8) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(s_a + BUF + at + cvec * 8) = u32x4{0u, 0u, 0u, 0u};
    }
  }
  // One register set of raw vectors: the loads of chunk c + 2 are issued behind the sweep of chunk c, and the vectors of chunk c + 1 are
  // activated and stored into the other LDS buffer in the last two thirds of that sweep.
  const int nchunks = p.cin / KC;
  u32x4 raw[NV];

  float zero = 0.f;
  asm volatile("" : "+v"(zero));   // (seen as a constant, it costs the fullest of these kernels spilled registers)
#pragma unroll
  for (int i = 0; i < TH; ++i)
#pragma unroll
    for (int j = 0; j < 2 * NI; ++j) acc[i][j] = f32x4{zero, zero, zero, zero};
  const int row_off = (lane & 15) * PS + (lane >> 4) * 8;   // the lane's pixel and octet in a row of the patch

  // ---- shortcut phase (a second input): acc = W2 * x2 over the tile's own pixels, a 1x1
  // contraction over cin2 channels taken as stored (no normalisation).  Chunks go through the same
  // two LDS buffers, to their pixels' slots in the patch; the main
  // loop below then adds the 3x3 contraction to the same accumulators, so the shortcut tensor never exists in
  // memory and the epilogue adds both biases.  A chunk is little work (16 MFMAs a wavefront and 32 channels), so input and weights travel three
  // chunks ahead.
  if (p.x2) {
    constexpr int ALL = TH * 16 * VPP, NC = (ALL + NT - 1) / NT, AHEAD = 3;   // vectors of a thread: the pixels without the halo
    const char* xin2 = reinterpret_cast<const char*>(p.x2) + (size_t)n * p.h * p.w_out * p.cin2 * sizeof(T);
    const int nch2 = p.cin2 / KC;
    int src2[NC], dst2[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int v = (tid + i * NT) / VPP, y = v / 16, x = v % 16;
      const bool inside = (NC * NT == ALL || v < TH * 16) && ty0 + y < p.h && tx0 + x < p.w_out;   // (the others' slots stay zero: the 3x3 taps read them)
      src2[i] = (inside ? (ty0 + y) * p.w_out + tx0 + x : 0) * p.cin2 * (int)sizeof(T) + cvec * 16;
      dst2[i] = (inside ? (y + 1) * ROW + (x + 1) * PS : SPARE) + cvec * 8;
    }
    const __amdgpu_buffer_rsrc_t wrsrc2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w2), 0, p.w2_bytes, 0x00020000);
    u32x4 x2[AHEAD][NC], w2[AHEAD][2 * NI];   // of chunk c in place c % AHEAD; past the last chunk: a harmless reload
    auto issue2 = [&](u32x4 (&v)[NC], int chunk) {
#pragma unroll
      for (int i = 0; i < NC; ++i) v[i] = *reinterpret_cast<const u32x4*>(xin2 + (unsigned)(src2[i] + min(chunk, nch2 - 1) * KC * (int)sizeof(T)));
    };
    auto load2 = [&](u32x4 (&f)[2 * NI], int chunk) {
#pragma unroll
      for (int j = 0; j < 2 * NI; ++j) f[j] = load_fragment(wrsrc2, lane_w, wcol + min(chunk, nch2 - 1) * 2 * kk_stride + j / 2 * 1024 + 16 * (j % 2));
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) { issue2(x2[k], k); load2(w2[k], k); }
    auto chunk2 = [&](auto k_c, int c) {
      constexpr int k = decltype(k_c)::value;
      T* buf = s_a + (c & 1) * BUF;
#pragma unroll
      for (int i = 0; i < NC; ++i) *reinterpret_cast<u32x4*>(buf + dst2[i]) = x2[k][i];
      issue2(x2[k], c + AHEAD);
      __syncthreads();   // (the other buffer is rewritten only behind the next barrier)
      const T* ctr = buf + row_off + ROW + PS;
#pragma unroll
      for (int r = 0; r < TH; ++r) {
        const u32x4 px = *reinterpret_cast<const u32x4*>(ctr + r * ROW);
#pragma unroll
        for (int j = 0; j < 2 * NI; ++j) acc[r][j] = Mma<T>::m16(px, w2[k][j], acc[r][j]);
      }
      load2(w2[k], c + AHEAD);
    };
    for (int c = 0; c < nch2; c += AHEAD) {
      chunk2(std::integral_constant<int, 0>{}, c);
      if (c + 1 < nch2) chunk2(std::integral_constant<int, 1>{}, c + 1);
      if (c + 2 < nch2) chunk2(std::integral_constant<int, 2>{}, c + 2);
    }
  }

#pragma unroll
  for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const u32x4*>(xin + (unsigned)src_off[i]);
  // ---- per-channel scale/shift table: a = gamma*rstd, b = beta - mean*a (built behind the first chunk's loads, so that its own
  // global loads overlap them).  With SiLU the table holds -log2(e) * (a, b):
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
      // round-robin; (mean, rstd) parked behind the table
      float2* s_stat = s_ab + p.cin;
      // Launches that leave a wavefront alone on its SIMD (RING): gamma / beta of this thread's first two table
      // entries are requested together with the triples, one memory round trip less in front of the first chunk
      // (elsewhere other workgroups cover that latency and the registers are better left to the main loop).
      constexpr int PRE = RING > 0 ? 2 : 0;
      float gpre[2] = {0.f, 0.f}, bpre[2] = {0.f, 0.f};
      int group[2] = {0, 0};
#pragma unroll
      for (int j = 0; j < PRE; ++j) {
        const int c = min(tid + j * NT, p.cin - 1);
        gpre[j] = p.gamma[c]; bpre[j] = p.beta[c];
        group[j] = quotient_of(c, p.cpg_in, p.inv_cpg_in);
      }
      constexpr int LANES = 8;
      merge_sample<LANES, NT>(p.rows_in + (size_t)n * p.groups * p.rows_in_count, p.groups, p.rows_in_count, tid, p.eps, s_stat);
      if constexpr (RING > 0) first_weights();
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PRE; ++j)
        if (tid + j * NT < p.cin) entry(tid + j * NT, s_stat[group[j]], gpre[j], bpre[j]);
      for (int c = tid + PRE * NT; c < p.cin; c += NT) entry(c, s_stat[quotient_of(c, p.cpg_in, p.inv_cpg_in)], p.gamma[c], p.beta[c]);
    } else {
      if constexpr (RING > 0) first_weights();
      for (int c = tid; c < p.cin; c += NT) {
        const int g = n * p.groups + quotient_of(c, p.cpg_in, p.inv_cpg_in);
        entry(c, make_float2(p.mean[g], p.rstd[g]), p.gamma[c], p.beta[c]);
      }
    }
  }
  __syncthreads();            // scale/shift table complete
  auto table = [&](const float2* tab, int part) -> f32x4 {   // entries of word `part` of the thread's octet
    if constexpr (ACT > 0) return *reinterpret_cast<const f32x4*>(tab + 2 * part);
    else return f32x4{0.f, 0.f, 0.f, 0.f};
  };
#pragma unroll
  for (int part = 0; part < 4; ++part) {
    const f32x4 ab = table(s_ab + cvec * 8, part);
#pragma unroll
    for (int i = 0; i < NV; ++i) raw[i][part] = activate_word<T, ACT, true>(raw[i][part], ab);
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) *reinterpret_cast<u32x4*>(s_a + dst_off[i]) = raw[i];
  if (nchunks > 1) {
#pragma unroll
    for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const u32x4*>(xin + (unsigned)(src_off[i] + KC * (int)sizeof(T)));
  }
  if constexpr (PARK) {
    s_off[tid] = u32x4{(unsigned)dst_off[0], (unsigned)dst_off[1], (unsigned)dst_off[NV - 1], 0u};
    s_off[NT + tid] = u32x4{(unsigned)src_off[0], (unsigned)src_off[1], (unsigned)src_off[NV - 1], 0u};
  }
  __syncthreads();

  EpilogueParams ep;
  {
    const int elems = p.h * p.w_out * p.cout;   // of a sample
    char* y = reinterpret_cast<char*>(p.y) + (size_t)n * elems * sizeof(TO);
    ep.y = __builtin_amdgcn_make_buffer_rsrc(y, 0, (int)(elems * sizeof(TO)), 0x00020000);
    const char* res = reinterpret_cast<const char*>(p.res) + (size_t)n * elems * sizeof(T);
    ep.res = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(res), 0, p.res ? (int)(elems * sizeof(T)) : 0, 0x00020000);   // (none: reads zeros)
  }
  ep.h = p.h; ep.w = p.w_out; ep.cout = p.cout;
  // statistics slot of this tile: [sample][group][spatial tile], or by blocks of 4 rows x 16 pixels
  ep.stats = p.stats ? p.stats + (size_t)n * p.stats_groups * p.stats_slots + (MODE == kRows4 ? ty0 / 4 * p.tiles_x + tx0 / TW : MODE == kSixEight ? six_eight_run(ty0) * p.tiles_x + tx0 / TW : tile) : nullptr;
  ep.cut = MODE == kSixEight ? six_eight_rows_left(ty0) : TH;
  ep.cpg = p.stats_cpg; ep.stats_stride = p.stats_slots; ep.row_stride = p.tiles_x; ep.handed_over = p.rows_out != nullptr;

  // ---- the chunks.  In the last two thirds of a sweep the words (two channels) of the next chunk's vectors are activated: all vectors of a
  // thread hold the same channel octet, so they are taken part by part (word `part` of every vector, then the next part), with the
  // table entries of a part read from LDS once, ahead of their first use.  A word's operations are dealt to the MFMAs from
  // its start on, so that none waits for the one before it.
  const T* rows_at = s_a + row_off;          // what a sweep reads, advanced from chunk to chunk
  const float2* tab = s_ab + cvec * 8;       // the table entries of the chunk that a sweep activates
  float k;
  asm("s_mov_b32 %0, 0xbfb8aa3b" : "=s"(k));   // -log2(e), see silu_from_scaled: the compiler would keep it in a vector register
  for (int c = 0; c + 1 < nchunks; ++c) {
    T* nbuf = s_a + ((c + 1) & 1) * BUF;
    tab += KC;
    u32x4 off;                                 // (PARK) the offsets at hand: dst_off towards the end of the sweep, src_off behind it
    f32x4 ab;
    float t0, t1, e0, e1;                      // a word's values on their way
    auto slice = [&](auto m_c) {
      constexpr int m = decltype(m_c)::value, ALL = 18 * NI * TH, FIRST = ALL / 3, SPAN = ALL - FIRST, NW = NV * 4;
      constexpr bool FINE = SPAN / NW >= 8;    // eight MFMAs a word, otherwise six
      static_assert(SPAN / NW >= 6, "a word takes six MFMAs");
      if constexpr (m == FIRST - 8) ab = table(tab, 0);
      if constexpr (PARK && m == FIRST + NV * 3 * SPAN / NW - 8) off = s_off[tid];
      if constexpr (m >= FIRST) {
        constexpr int wi = ((m - FIRST + 1) * NW - 1) / SPAN;        // the last word that starts at this MFMA or before it:
        constexpr int at = m - FIRST - wi * SPAN / NW;               // word wi starts at FIRST + wi * SPAN / NW
        constexpr int stage = FINE ? at : at == 0 ? 0 : at == 1 ? 12 : at == 2 ? 3 : at == 3 ? 45 : at + 2;
        constexpr int part = wi / NV, i = wi % NV;
        if constexpr (ACT > 0 && stage == 0) {
          t0 = fmaf(unpack_lo<T>(raw[i][part]), ab[0], ab[1]);
          t1 = fmaf(unpack_hi<T>(raw[i][part]), ab[2], ab[3]);
        }
        if constexpr (stage == 0 && i == NV - 1 && part < 3) ab = table(tab, part + 1);
        if constexpr (ACT == 2) {
          if constexpr (stage == 1 || stage == 12) e0 = __builtin_amdgcn_exp2f(t0);
          if constexpr (stage == 2 || stage == 12) e1 = __builtin_amdgcn_exp2f(t1);
          if constexpr (stage == 3) { e0 = fmaf(e0, k, k); e1 = fmaf(e1, k, k); }
          if constexpr (stage == 4 || stage == 45) e0 = __builtin_amdgcn_rcpf(e0);
          if constexpr (stage == 5 || stage == 45) e1 = __builtin_amdgcn_rcpf(e1);
          if constexpr (stage == 6) { t0 *= e0; t1 *= e1; }
        }
        if constexpr (stage == 7) {
          if constexpr (ACT > 0) {
            asm("" : "+v"(t0), "+v"(t1));   // the roundings stay apart, see activate_word
            raw[i][part] = pack_word<T>(t0, t1);
          }
          if constexpr (part == 3) *reinterpret_cast<u32x4*>(nbuf + (PARK ? (int)off[i] : dst_off[i])) = raw[i];
        }
      }
    };
    const int bcur = wcol + c * 2 * kk_stride;
    sweep_chunk<T, TH, NI, D, false>(rows_at, wrsrc, bcur, bcur + 2 * kk_stride, tap_stride, lane_w, bq, acc, slice);
    if (c + 2 < nchunks) {
      if constexpr (PARK) off = s_off[NT + tid];
#pragma unroll
      for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const u32x4*>(xin + (unsigned)((PARK ? (int)off[i] : src_off[i]) + (c + 2) * KC * (int)sizeof(T)));
    }
    rows_at += c & 1 ? -BUF : BUF;
    __syncthreads();          // other buffer staged; this one free for chunk c + 2
  }
  // the last one: nothing to activate, and behind its last weights the residual is requested, so that the epilogue does not wait for it
  constexpr int ASKED = asked_rows(TH, NI, sizeof(TO));
  uint32_t rv[NI * TH][4];
  unsigned at[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) at[i] = lane_offset(ep, lane, tx0, i);
  auto ask = [&](auto m_c) {
    constexpr int m = decltype(m_c)::value, AFTER = (9 * NI - (D - 1)) * TH * 2, FROM = NI == 1 ? AFTER : 18 * NI * TH - 4 * ASKED, j = m - FROM;
    static_assert(FROM >= AFTER && FROM + 4 * ASKED <= 18 * NI * TH, "behind the last weights, and all of them");
    if constexpr (j >= 0 && j < 4 * ASKED) rv[j / 4][j % 4] = load_residual<T>(ep, at[j % 4], ty0 + j / 4, tx0, co_w);
  };
  sweep_chunk<T, TH, NI, D, true>(rows_at, wrsrc, wcol + (nchunks - 1) * 2 * kk_stride, 0, tap_stride, lane_w, bq, acc, ask);

  int last = lane;
  asm volatile("" : "+v"(last));   // (what the epilogue derives from it is not held through the sweeps)
  const float* bias_w = s_bias + wn * NI * 32;
  auto finish = [&](auto res_c, auto stats_c, auto full_c) __attribute__((always_inline)) {
    epilogue<T, TO, TH, NI, decltype(res_c)::value, decltype(stats_c)::value, decltype(full_c)::value, MODE>(acc, rv, bias_w, last, ty0, tx0, co_w, ep);
  };
  const std::true_type yes{};
  const std::false_type no{};
  if (!p.stats) {
    if (p.res) finish(yes, no, no);
    else finish(no, no, no);
  } else if (sizeof(TO) == 2 && ty0 + TH <= p.h && tx0 + 16 <= p.w_out) {   // (fp32 values of all rows at once would be spilled)
    if constexpr (sizeof(TO) == 2) {
      if (p.res) finish(yes, yes, yes);
      else finish(no, yes, yes);
    }
  } else {
    if (p.res) finish(yes, yes, no);
    else finish(no, yes, no);
  }

  if (p.rows_out) hand_over_row<NT>(p, n, wt.y, nt, co0, TN, WM, tid, lane);
}

template <typename T, typename TO, int TH, int NI, int MODE, int RING>
int launch_cfg(const ConvArgs& a, hipStream_t s) {
  MfmaParams p = conv_params(a, TH, 16, 128 * NI, 1, a.h, a.w);
  if (MODE == kRows4) p.stats_slots = ((a.h + 3) / 4) * p.tiles_x;
  if (MODE == kSixEight) p.stats_slots = (six_eight_run(a.h - 1) + 1) * p.tiles_x;
  WMDEC_REQUIRE(a.cin % kChunk == 0 && a.cout % (128 * NI) == 0 && !a.y_nchw, WMDEC_ERR_UNSUPPORTED, "conv_rows: channels do not fit the tile");
  WMDEC_REQUIRE(MODE == kPlain || !a.rows_out, WMDEC_ERR_UNSUPPORTED, "conv_rows: this tile hands over no rows");
  const int rc = check_hand_over(p);
  if (rc != WMDEC_OK) return rc;
  p.w = a.wt;
  p.w_bytes = (int)(packed_elems(9, a.cout, a.cin) * sizeof(T));
  if (a.x2) {
    WMDEC_REQUIRE(a.w2 && a.cin2 > 0 && a.cin2 % kChunk == 0 && (long)a.h * a.w * a.cin2 < (1L << 29), WMDEC_ERR_UNSUPPORTED,
                  "conv_rows: a folded shortcut needs cin2 %% %d == 0", kChunk);
    p.x2 = a.x2; p.w2 = a.w2; p.bias2 = a.bias2; p.cin2 = a.cin2;
    p.w2_bytes = (int)(packed_elems(1, a.cout, a.cin2) * sizeof(T));
  }
  const size_t smem = fixed_lds(TH, NI, RING) + (size_t)(a.cin + a.groups) * sizeof(float2);
  WMDEC_REQUIRE(smem <= 80 * 1024, WMDEC_ERR_UNSUPPORTED, "conv_rows: %zu bytes of LDS needed", smem);
  void (*kern)(MfmaParams) = !p.norm ? conv_mfma_kernel<T, TO, TH, 16, 1, 4, NI, 3, kChunk, 0, MODE, RING>
                             : (a.silu ? conv_mfma_kernel<T, TO, TH, 16, 1, 4, NI, 3, kChunk, 2, MODE, RING>
                                       : conv_mfma_kernel<T, TO, TH, 16, 1, 4, NI, 3, kChunk, 1, MODE, RING>);
  // once per instantiation and activation mode (80 KiB: two workgroups per compute unit)
  static std::once_flag attr_once[3];
  hipError_t attr_err = hipSuccess;
  std::call_once(attr_once[!p.norm ? 0 : (a.silu ? 2 : 1)],
                 [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024); });
  WMDEC_HIP(attr_err);
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.total + warm_groups(p.next, 4))), dim3(256), smem, s, p);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

template <typename T, typename TO>
int launch_form(const ConvArgs& a, int th, int ni, ConvMode mode, bool whole_ring, hipStream_t s) {
  if constexpr (sizeof(TO) == 2) {
    if (th == 6) return ni == 2 ? launch_cfg<T, TO, 6, 2, kSixEight, 0>(a, s) : launch_cfg<T, TO, 6, 1, kSixEight, 18>(a, s);
    if (mode == kSixEight && ni == 2) return launch_cfg<T, TO, 8, 2, kSixEight, 0>(a, s);
    if (mode == kSixEight) return whole_ring ? launch_cfg<T, TO, 8, 1, kSixEight, 18>(a, s) : launch_cfg<T, TO, 8, 1, kSixEight, 0>(a, s);
  }
  if (th == 4) return launch_cfg<T, TO, 4, 1, kRows4, 18>(a, s);
  if (ni == 2) return launch_cfg<T, TO, 8, 2, kPlain, 0>(a, s);
  if (mode == kRows4) return whole_ring ? launch_cfg<T, TO, 8, 1, kRows4, 18>(a, s) : launch_cfg<T, TO, 8, 1, kRows4, 0>(a, s);
  return whole_ring ? launch_cfg<T, TO, 8, 1, kPlain, 18>(a, s) : launch_cfg<T, TO, 8, 1, kPlain, 0>(a, s);
}

template <typename T> int launch_type(const ConvArgs& a, int th, int ni, ConvMode mode, bool whole_ring, hipStream_t s) {
  return a.y_dtype == WMDEC_F32 ? launch_form<T, float>(a, th, ni, mode, whole_ring, s) : launch_form<T, T>(a, th, ni, mode, whole_ring, s);
}

}  // namespace

// bf16 is compiled by kernels_conv_rows_bf16.hip, which includes this file: the two types beside each other take half of the time.
#ifdef WMDEC_CONV_ROWS_BF16
int launch_conv_rows_bf16(const ConvArgs& a, int th, int ni, int mode, bool whole_ring, hipStream_t s) { return launch_type<bf16_t>(a, th, ni, (ConvMode)mode, whole_ring, s); }
#else
int launch_conv_rows_bf16(const ConvArgs& a, int th, int ni, int mode, bool whole_ring, hipStream_t s);
int launch_conv_rows(const ConvArgs& a, int th, int ni, int mode, bool whole_ring, hipStream_t s) {
  WMDEC_REQUIRE(mode != kSixEight || a.y_dtype != WMDEC_F32, WMDEC_ERR_UNSUPPORTED, "conv_rows: this tile stores 16 bits");
  return a.op_dtype == WMDEC_BF16 ? launch_conv_rows_bf16(a, th, ni, mode, whole_ring, s) : launch_type<f16_t>(a, th, ni, (ConvMode)mode, whole_ring, s);
}
#endif

}  // namespace wmdec
