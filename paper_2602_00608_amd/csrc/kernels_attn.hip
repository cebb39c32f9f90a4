// Mid-block attention: one head of dimension 512, softmax(q k^T / sqrt(d)) v over the tokens of a sample.
//
// Three launches hand over 32-token tiles in MFMA fragment order, so that every one of them loads and stores runs of 1 KiB:
//   attn_qkv_kernel                               [q|k|v] = W norm(x) + b, straight from its accumulators into fragments
//   flash_attn_kernel                             streams the keys, online softmax, unnormalised partial outputs
//   attn_combine_kernel                           merges the partial outputs of the key ranges, normalises, rows of o (where one
//                                                 range holds all keys, the core writes these rows itself)
//
// Fragments (16-bit type T, tile = 32 tokens x 512 = 32 KiB, 32 runs of 64 lanes x 16 bytes), lane = l32 + 32 * lk:
//   q, k  [step 0..31][lane]     token l32, channels 16 * step + 8 * lk + 0..7: operand of the 32x32x16 MFMA as it is
//   v     [ks 0..1][dt 0..15][lane]   channel 32 * dt + l32, tokens 16 * ks + 4 * lk + {0..3, 8..11}: the token order in which
//         an accumulator tile S^T[key][query] holds its keys, so that the probabilities become the other operand of the
//         second product without leaving their registers
// Tokens past the end have zero fragments of v (their probability is zero, and zero times what a fresh buffer holds is not).
#include <stdio.h>

#include <mutex>

#include "conv_device.hpp"

namespace wmdec {
namespace {

constexpr int D = 512;            // head dimension
constexpr int KB = 32;            // tokens per tile
constexpr int TILE = KB * D;      // elements of a tile

// lane l: its own a and the a of lane l + 32 (l < 32), or the b of lane l - 32 and its own b: four channels of eight become
// eight of four when a and b hold an accumulator tile's channels 8 * g + 4 * lk + 0..3 for g and g + 1
__device__ __forceinline__ u32x4 join_halves(u32x2 a, u32x2 b) {
  const u32x2 lo = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
  const u32x2 hi = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
  return u32x4{lo.x, hi.x, lo.y, hi.y};
}

// ---------------------------------------------------------------- q, k, v projection
// A workgroup takes 64 tokens and the 512 channels of one of q, k, v: the normalised input (64 KiB) is staged once, after
// which eight wavefronts (64 tokens x 64 channels each) walk the contraction without a barrier.  Bound by the 512 KiB of
// weights that every workgroup streams through the vector L1 (64 B per cycle: half of the launch at 5400 tokens) and the load
// and table in front of it.  5400 tokens 25.1 -> 16.2 us against the general 1x1 kernel, and the 8.4 us pass that laid v out
// for the second product is gone.
constexpr int QT = 64;            // tokens per workgroup
constexpr int QNT = 512;          // threads
constexpr int QRING = 8;          // weight fragments travel this many contraction steps ahead
struct QkvParams {
  const void* x; const float* mean; const float* rstd; const float* gamma; const float* beta;
  const Moments* rows_in; int rows_in_count; float eps;
  const void* w; const float* bias; void* frag;
  int n, t, groups, tiles, w_bytes;   // tiles: workgroups along the tokens of a sample
};

template <typename T>
__global__ __launch_bounds__(QNT, 2) void attn_qkv_kernel(QkvParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* s_x = reinterpret_cast<T*>(smem);                                   // [2][32 steps][64 lanes][8]
  float2* s_ab = reinterpret_cast<float2*>(smem + QT * D * sizeof(T));   // [D] (scale, shift)
  float2* s_stat = s_ab + D;                                             // [groups]
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroup id -> (q / k / v, sample, token tile); the ids of one XCD (id % 8) are neighbours and share their weights
  int L;
  {
    const int i = blockIdx.x, total = gridDim.x, per = total / 8, rem = total % 8, x = i % 8, j = i / 8;
    L = x * per + (x < rem ? x : rem) + j;
  }
  const int tile = L % p.tiles, n = L / p.tiles % p.n, part = L / (p.tiles * p.n);
  const int t0 = tile * QT;

  // ---- the input, all requests at once: a vector is 8 channels of a token, a wavefront's load 16 tokens x 64 bytes
  const T* x = reinterpret_cast<const T*>(p.x) + (size_t)n * p.t * D;
  const int tok16 = lane & 15, c4 = lane >> 4;
  u32x4 raw[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int tok = min(t0 + (i % 4) * 16 + tok16, p.t - 1), chunk = (wave * 2 + i / 4) * 4 + c4;
    raw[i] = *reinterpret_cast<const u32x4*>(x + (size_t)tok * D + chunk * 8);
  }
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.w), 0, p.w_bytes, 0x00020000);
  constexpr int STEP = 3 * D / 32 * 1024;                 // bytes of the weights of a contraction step
  const int wcol = (part * (D / 32) + wave * 2) * 1024, lane16 = lane * 16;
  u32x4 wq[QRING][2];
  // The first weights, 112 KiB of a workgroup, behind the input and the moments, which are needed before them: loads return in order.
  auto first_weights = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < QRING - 1; ++s)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) wq[s][ni] = load_fragment(wrsrc, lane16, wcol + s * STEP + ni * 1024);
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- scale/shift table
  {
    const float ga = p.gamma[tid], be = p.beta[tid];      // one channel per thread
    static_assert(QNT == D, "one channel per thread");
    if (p.rows_in) {
      merge_sample<8, QNT>(p.rows_in + (size_t)n * p.groups * p.rows_in_count, p.groups, p.rows_in_count, tid, p.eps, s_stat);
    } else {
      for (int g = tid; g < p.groups; g += QNT) s_stat[g] = make_float2(p.mean[n * p.groups + g], p.rstd[n * p.groups + g]);
    }
    first_weights();
    __syncthreads();
    const float2 st = s_stat[tid / (D / p.groups)];
    const float a = ga * st.y;
    s_ab[tid] = make_float2(a, be - st.x * a);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int chunk = (wave * 2 + i / 4) * 4 + c4, tok = (i % 4) * 16 + tok16;
    const f32x4* tab = reinterpret_cast<const f32x4*>(s_ab + chunk * 8);
#pragma unroll
    for (int k = 0; k < 4; ++k) raw[i][k] = activate_word<T, 1>(raw[i][k], tab[k]);   // (scale and shift)
    *reinterpret_cast<u32x4*>(s_x + (size_t)((tok / 32) * 32 + chunk / 2) * 512 + (tok % 32 + 32 * (chunk % 2)) * 8) = raw[i];
  }
  __syncthreads();

  // ---- contraction.  q, k: A = weights, B = tokens (a lane holds channels of one token); v: exchanged
  f32x16 acc[2][2];   // [token tile][channel tile]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i / 2][i % 2][r] = 0.f;
  auto contract = [&](auto tokens_first_c) {
    constexpr bool TOKENS_FIRST = decltype(tokens_first_c)::value;
    u32x4 xf[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) xf[0][mi] = *reinterpret_cast<const u32x4*>(s_x + mi * TILE + lane * 8);
    static_for<D / 16>([&](auto s_c) {
      constexpr int s = decltype(s_c)::value;
      if constexpr (s + QRING - 1 < D / 16) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) wq[(s + QRING - 1) % QRING][ni] = load_fragment(wrsrc, lane16, wcol + (s + QRING - 1) * STEP + ni * 1024);
      }
      if constexpr (s + 1 < D / 16) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) xf[(s + 1) % 2][mi] = *reinterpret_cast<const u32x4*>(s_x + mi * TILE + (s + 1) * 512 + lane * 8);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
          acc[mi][ni] = TOKENS_FIRST ? Mma<T>::m32(xf[s % 2][mi], wq[s % QRING][ni], acc[mi][ni]) : Mma<T>::m32(wq[s % QRING][ni], xf[s % 2][mi], acc[mi][ni]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  const int nkb = (p.t + KB - 1) / KB;
  T* dst = reinterpret_cast<T*>(p.frag) + ((size_t)(part * p.n + n) * nkb + tile * 2) * TILE + lane * 8;
  const float* bias = p.bias + part * D + wave * 64;
  if (part < 2) {
    f32x4 bq[2][4];   // (requested in front of the contraction: behind it they would be a trip of their own)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int g = 0; g < 4; ++g) bq[ni][g] = f32x4{bias[ni * 32 + 8 * g + 4 * lk], bias[ni * 32 + 8 * g + 4 * lk + 1], bias[ni * 32 + 8 * g + 4 * lk + 2], bias[ni * 32 + 8 * g + 4 * lk + 3]};
    contract(std::false_type{});
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      const f32x4 (&b)[4] = bq[ni];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) {
        if (tile * 2 + mi >= nkb) continue;
        const f32x16& c = acc[mi][ni];
        u32x2 w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) w[g] = u32x2{pack2<T>(c[4 * g] + b[g][0], c[4 * g + 1] + b[g][1]), pack2<T>(c[4 * g + 2] + b[g][2], c[4 * g + 3] + b[g][3])};
#pragma unroll
        for (int k = 0; k < 2; ++k) *reinterpret_cast<u32x4*>(dst + (size_t)mi * TILE + (wave * 4 + ni * 2 + k) * 512) = join_halves(w[2 * k], w[2 * k + 1]);
      }
    }
  } else {
    const float bv[2] = {bias[l32], bias[32 + l32]};
    contract(std::true_type{});
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      const float b = bv[ni];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) {
        if (tile * 2 + mi >= nkb) continue;
        const int tok = t0 + mi * 32 + 4 * lk;
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = tok + 8 * (r / 4) + r % 4 < p.t ? acc[mi][ni][r] + b : 0.f;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          *reinterpret_cast<u32x4*>(dst + (size_t)mi * TILE + (ks * 16 + wave * 2 + ni) * 512) =
              u32x4{pack2<T>(v[8 * ks], v[8 * ks + 1]), pack2<T>(v[8 * ks + 2], v[8 * ks + 3]), pack2<T>(v[8 * ks + 4], v[8 * ks + 5]), pack2<T>(v[8 * ks + 6], v[8 * ks + 7])};
      }
    }
  }
}

// ---------------------------------------------------------------- attention core
// A workgroup takes 128 queries, a wavefront 32 of them with all 512 channels of their output in registers; k and v stream
// through LDS in blocks of 32 keys, two blocks each (128 KiB), and every wavefront reads all of both.  Per block a wavefront
// has 32 MFMAs of scores and 32 of output, with one 1 KiB LDS read each; the wavefronts share nothing but the tiles.
// Earlier 64 queries were the workgroup's, with the scores in other wavefronts than the output: twice the tile traffic per
// query and the probabilities through LDS.  128 queries x 32 keys take 2300 cycles where the MFMAs take 2048; 5400 tokens
// 91 -> 78 us, of which 60 us are the blocks (at 1 PFLOP/s the chip lowers its clock: with fewer compute units busy a block
// takes less, but not by as much as there are more of them each, see splits_of), 10 us the partial outputs (55 MB) and 9 us the
// first tiles.  Measured and not kept: tile requests dealt to one wavefront at a time with three buffers of k (86 us),
// 4 or 16 fragments ahead (82, 125).
constexpr int NT = 256;           // threads: four wavefronts of 32 queries
constexpr int R = 8;              // fragments read from LDS ahead of their MFMAs, a divisor of 32
constexpr float kSlack = 8.0f;    // log2 of how far a block's maximum may exceed the running reference before it moves
constexpr size_t kSmemBytes = (size_t)4 * TILE * 2;

__device__ __forceinline__ float max3(float a, float b, float c) {   // (fmaxf would quiet its operands first: twice the instructions)
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// max over lanes l and l ^ 32 (the results of the swap are made opaque: this compiler otherwise takes both for the first one)
__device__ __forceinline__ float half_max(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const u32x2 r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  unsigned a = r.x, b = r.y;
  asm volatile("" : "+v"(a), "+v"(b));
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}

// Registers.  The output accumulators of a wavefront (32 queries x 512) are 256 registers, exactly the accumulation half of the
// register file; its query fragments are 128 of the other half.  The compiler gives every MFMA of a kernel its result in the
// accumulation half, which the scores' 16 registers would overflow (336 registers spilled); so the scores' MFMAs are written
// out, with the result in the other half.  The compiler does not see them as MFMAs: settle_scores() is the wait before
// their result is read (11 wait states are due behind a 32x32x16 MFMA), and the build fails where the compiler touches one earlier or
// spills (asm_check.py).  Nor does it keep the accumulators in place where a
// branch multiplies them (234 spilled): rescale_tile is one statement per tile that names the tile's registers and jumps to
// the multiplications, out of line, only if a lane's reference has moved.
template <typename T> __device__ __forceinline__ void score_first(f32x16& s, const u32x4& k, const u32x4& q) {
  if constexpr (std::is_same<T, f16_t>::value) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "v"(q));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "v"(q));
}
template <typename T> __device__ __forceinline__ void score_next(f32x16& s, const u32x4& k, const u32x4& q) {
  if constexpr (std::is_same<T, f16_t>::value) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "v"(q));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(k), "v"(q));
}
__device__ __forceinline__ void settle_scores(f32x16& s) { asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s)); }

#define WMDEC_RESCALE(I_, LO, HI)                                                                                                    \
  if constexpr (I == I_)                                                                                                             \
  asm volatile("s_cmp_lg_u64 %3, 0\n\ts_cbranch_scc1 2f\n1:\n\t.subsection 1\n2:\n\ts_nop 15\n\t.set wmdec_r, " #LO "\n\t.rept 16\n\t" \
               "v_accvgpr_read_b32 %1, a[wmdec_r]\n\tv_mul_f32 %1, %2, %1\n\tv_accvgpr_write_b32 a[wmdec_r], %1\n\t"                 \
               ".set wmdec_r, wmdec_r + 1\n\t.endr\n\ts_nop 7\n\ts_branch 1b\n\t.subsection 0"                                       \
               : "+{a[" #LO ":" #HI "]}"(o), "=&v"(t) : "v"(factor), "s"(moved) : "scc")
// o *= factor if any bit of `moved` is set
template <int I> __device__ __forceinline__ void rescale_tile(f32x16& o, float factor, unsigned long long moved) {
  float t;
  WMDEC_RESCALE(0, 0, 15); WMDEC_RESCALE(1, 16, 31); WMDEC_RESCALE(2, 32, 47); WMDEC_RESCALE(3, 48, 63);
  WMDEC_RESCALE(4, 64, 79); WMDEC_RESCALE(5, 80, 95); WMDEC_RESCALE(6, 96, 111); WMDEC_RESCALE(7, 112, 127);
  WMDEC_RESCALE(8, 128, 143); WMDEC_RESCALE(9, 144, 159); WMDEC_RESCALE(10, 160, 175); WMDEC_RESCALE(11, 176, 191);
  WMDEC_RESCALE(12, 192, 207); WMDEC_RESCALE(13, 208, 223); WMDEC_RESCALE(14, 224, 239); WMDEC_RESCALE(15, 240, 255);
}
#undef WMDEC_RESCALE

// A lane's 16 channels (8 * (r / 4) + 4 * lk + r % 4) of 32 of its token's, divided by the sum of its probabilities: two runs of eight
// channels, of which the second is 16 further.
template <typename T> __device__ __forceinline__ void normalised_runs(const f32x4 (&num)[4], float inv, u32x4& first, u32x4& second) {
  u32x2 w[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) w[g] = u32x2{pack2<T>(num[g][0] * inv, num[g][1] * inv), pack2<T>(num[g][2] * inv, num[g][3] * inv)};
  first = join_halves(w[0], w[1]);
  second = join_halves(w[2], w[3]);
}

// WHOLE: one range holds all keys, `out` is o; otherwise the partial outputs.
template <typename T, bool WHOLE>
__global__ __launch_bounds__(NT, 1) void flash_attn_kernel(const T* __restrict__ qf, const T* __restrict__ kf, const T* __restrict__ vf, size_t sample_stride,
                                                           void* __restrict__ out, float* __restrict__ ml, int t, int nqb, int splits, float scale_log2e) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* s_k = reinterpret_cast<T*>(smem);   // [2] tiles of k
  T* s_v = s_k + 2 * TILE;               // [2] tiles of v
  const int tid = threadIdx.x, lane = tid & 63, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroup id -> (sample, key range, query block); the ids of one XCD (id % 8) are neighbours and share their keys
  int L;
  {
    const int i = blockIdx.x, total = gridDim.x, per = total / 8, rem = total % 8, x = i % 8, j = i / 8;
    L = x * per + (x < rem ? x : rem) + j;
  }
  const int qb = L % nqb, split = L / nqb % splits, n = L / (nqb * splits);
  const int nkb = (t + KB - 1) / KB;
  const int kb0 = (int)((long)split * nkb / splits), nb = (int)((long)(split + 1) * nkb / splits) - kb0;   // key blocks of this range, at least one
  const int qt = qb * 4 + wave;          // this wavefront's query tile (past the last one: computed from the last, not stored)

  // tile loads: straight into LDS, a KiB at a time; a block past the range reloads its last one, harmlessly
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  constexpr int SHARE = TILE / 4;        // a wavefront's share of a tile
  const size_t first = n * sample_stride + (size_t)kb0 * TILE + wave * SHARE + lane * 8;
  auto load_k = [&](int i, int b) {
    __builtin_amdgcn_global_load_lds((gptr_t)(kf + first + (size_t)min(b, nb - 1) * TILE + i * 512), (lptr_t)(s_k + (b & 1) * TILE + wave * SHARE + i * 512), 16, 0, 0);
  };
  auto load_v = [&](int i, int b) {
    __builtin_amdgcn_global_load_lds((gptr_t)(vf + first + (size_t)min(b, nb - 1) * TILE + i * 512), (lptr_t)(s_v + (b & 1) * TILE + wave * SHARE + i * 512), 16, 0, 0);
  };
  // every load this wavefront issued has landed, everything it read from LDS has arrived, and so for the other wavefronts
  auto sync_tiles = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < 8; ++i) load_k(i, 0);
  u32x4 q[32];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(qf + n * sample_stride + (size_t)min(qt, nkb - 1) * TILE) + lane;
#pragma unroll
    for (int i = 0; i < 32; ++i) q[i] = src[i * 64];
    // (held in registers: left alone, the compiler reads them again for every key block)
#pragma unroll
    for (int i = 0; i < 32; ++i) asm volatile("" : "+v"(q[i]));
  }
  f32x16 s;             // scores, then probabilities, of a key block: keys 8 * (r / 4) + 4 * lk + r % 4 of the block, query lane % 32
  u32x4 p[2];           // probabilities as operands
  u32x4 kr[R], vr[R];   // fragments on their way from LDS
  float m_run = -INFINITY, l_run = 0.f, mx = 0.f, m_new = 0.f, alpha = 1.f, ps = 0.f;
  // Softmax of s in slices 0..31, which ride behind the MFMAs of the output.  The reference only moves when the block's
  // maximum exceeds it by more than 2^kSlack: until then the probabilities are taken against the old one (they may reach
  // 2^kSlack, well inside both 16-bit types).  Sums and outputs share the reference, so the normalised result is the same.
  auto soft = [&](auto i_c, bool live) {
    constexpr int i = decltype(i_c)::value;
    if constexpr (i == 3) mx = max3(max3(s[0], s[1], s[2]), s[3], s[3]);
    if constexpr (i >= 4 && i <= 6) { constexpr int e = (i - 3) * 4; mx = max3(max3(mx, s[e], s[e + 1]), s[e + 2], s[e + 3]); }
    if constexpr (i == 7) mx = half_max(mx) * scale_log2e;
    if constexpr (i == 8) { m_new = live && mx > m_run + kSlack ? mx : m_run; alpha = __builtin_amdgcn_exp2f(m_run - m_new); m_run = m_new; ps = 0.f; }
    if constexpr (i >= 9 && i < 25) { constexpr int r = i - 9; s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2e, -m_new)); ps += s[r]; }
    if constexpr (i == 25) { if (live) l_run = fmaf(l_run, alpha, ps); }
  };
  auto mask = [&](int b) {   // keys past the last token
    if (kb0 + b != nkb - 1) return;
    settle_scores(s);
    const int key = (kb0 + b) * KB + 4 * lk;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = key + 8 * (r / 4) + r % 4 < t ? s[r] : -INFINITY;
  };
  auto pack = [&]() {
#pragma unroll
    for (int k = 0; k < 2; ++k)
      p[k] = u32x4{pack2<T>(s[8 * k], s[8 * k + 1]), pack2<T>(s[8 * k + 2], s[8 * k + 3]), pack2<T>(s[8 * k + 4], s[8 * k + 5]), pack2<T>(s[8 * k + 6], s[8 * k + 7])};
  };
  auto head = [&](u32x4 (&ring)[R], const T* tiles, int b) {
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = *reinterpret_cast<const u32x4*>(tiles + (b & 1) * TILE + lane * 8 + r * 512);
  };
  // Scores of key block b.  The wait for the tiles stands in front of the last R - 1 MFMAs, whose fragments are in registers
  // by then, so that the first reads of v behind it have their latency covered.
  auto scores = [&](int b) {
    const T* kl = s_k + (b & 1) * TILE + lane * 8;
    static_for<32>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      if constexpr (i == 32 - R + 1) {
        sync_tiles();
        head(vr, s_v, b - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (i == 0) score_first<T>(s, kr[i % R], q[i]);
      else score_next<T>(s, kr[i % R], q[i]);
      if constexpr (i + R < 32) kr[i % R] = *reinterpret_cast<const u32x4*>(kl + (i + R) * 512);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // prologue: scores and probabilities of block 0, scores of block 1
  sync_tiles();
#pragma unroll
  for (int i = 0; i < 8; ++i) { load_k(i, 1); load_v(i, 0); }
  head(kr, s_k, 0);
  scores(0);
#pragma unroll
  for (int i = 0; i < 8; ++i) load_k(i, 2);
  head(kr, s_k, 1);
  settle_scores(s);
  mask(0);
  static_for<32>([&](auto i_c) { soft(i_c, true); });
  pack();
  if (nb > 1) scores(1);
  else { sync_tiles(); head(vr, s_v, 0); }
  f32x16 o[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  unsigned long long moved = 0;
  float factor = 1.f;
  // (puts the loop where the other form has it, 36 bytes into a line of 64: a wavefront alone on its SIMD waits for its instructions;
  // 16 770 tokens 965 -> 930 us)
  if constexpr (WHOLE) asm volatile("s_nop 0\n\ts_nop 0\n\ts_nop 0");
#pragma unroll 1
  for (int j = 0; j < nb; ++j) {
    // output of block j, with the softmax of block j + 1 and the requests of v of block j + 1 and k of block j + 3 in between
    // (their buffers were read up to the wait of the iteration before)
    const T* vl = s_v + (j & 1) * TILE + lane * 8;
    const T* kl = s_k + (j & 1) * TILE + lane * 8;      // k of block j + 2
    const bool live = j + 1 < nb;
    if (live) mask(j + 1);
    static_for<32>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      if constexpr (i < 16) rescale_tile<i>(o[i], factor, moved);
      o[i % 16] = Mma<T>::m32(vr[i % R], p[i / 16], o[i % 16]);
      if constexpr (i + R < 32) vr[i % R] = *reinterpret_cast<const u32x4*>(vl + (i + R) * 512);
      else kr[i % R] = *reinterpret_cast<const u32x4*>(kl + (i + R - 32) * 512);
      if constexpr (i == 1) settle_scores(s);
      soft(i_c, live);
      if constexpr (i % 2 == 0 && i < 16) load_v(i / 2, j + 1);
      if constexpr (i % 2 == 0 && i >= 16) load_k(i / 2 - 8, j + 3);
      __builtin_amdgcn_sched_barrier(0);
    });
    pack();
    moved = __ballot(alpha != 1.f);
    factor = alpha;
    __builtin_amdgcn_sched_barrier(0);
    if (j + 2 < nb) scores(j + 2);
    else { sync_tiles(); head(vr, s_v, j + 1); }
  }

  l_run += __shfl_xor(l_run, 32);
  if (qt >= nkb) return;
  int id = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));   // the lane once more: no register is left to hold it up to here
  asm volatile("" : "+v"(id));
  if constexpr (WHOLE) {
    const float inv = 1.0f / l_run;
    const int row = qt * KB + (id & 31);
    T* dst = reinterpret_cast<T*>(out) + ((size_t)n * t + row) * D + (id >> 5) * 8;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const f32x4 num[4] = {{o[i][0], o[i][1], o[i][2], o[i][3]}, {o[i][4], o[i][5], o[i][6], o[i][7]},
                            {o[i][8], o[i][9], o[i][10], o[i][11]}, {o[i][12], o[i][13], o[i][14], o[i][15]}};
      u32x4 first, second;
      normalised_runs<T>(num, inv, first, second);
      if (row < t) {
        *reinterpret_cast<u32x4*>(dst + i * 32) = first;
        *reinterpret_cast<u32x4*>(dst + i * 32 + 16) = second;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    const size_t row = ((size_t)n * splits + split) * nkb + qt;
    if (id < KB) reinterpret_cast<float2*>(ml)[row * KB + id] = make_float2(m_run, l_run);
    float* dst = reinterpret_cast<float*>(out) + row * TILE + id * 4;   // [dt][group of 8 channels][lane][4 channels]: what attn_combine_kernel reads
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(dst + (i * 4 + g) * 256) = f32x4{o[i][4 * g], o[i][4 * g + 1], o[i][4 * g + 2], o[i][4 * g + 3]};
  }
}

// o[n][token][:] = sum_s O_s 2^(m_s - M) / sum_s l_s 2^(m_s - M), key ranges merged in index order.  A wavefront takes 32 channels of
// a tile's 32 tokens; all partial outputs it needs are requested at once.
template <typename T, int SPLITS>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ opart, const float* __restrict__ ml, T* __restrict__ o, int t, int nkb) {
  const int tile = blockIdx.x, n = blockIdx.z, lane = threadIdx.x & 63, l32 = lane & 31, lk = lane >> 5;
  const int dt = blockIdx.y * 4 + (threadIdx.x >> 6);
  f32x4 part[SPLITS][4];
  float m[SPLITS], l[SPLITS];
#pragma unroll
  for (int s = 0; s < SPLITS; ++s) {
    const size_t row = ((size_t)n * SPLITS + s) * nkb + tile;
    const float2 st = reinterpret_cast<const float2*>(ml)[row * KB + l32];
    m[s] = st.x; l[s] = st.y;
#pragma unroll
    for (int g = 0; g < 4; ++g) part[s][g] = *reinterpret_cast<const f32x4*>(opart + row * TILE + (dt * 4 + g) * 256 + lane * 4);
  }
  float mx = m[0], den = 0.f;
#pragma unroll
  for (int s = 1; s < SPLITS; ++s) mx = fmaxf(mx, m[s]);
  f32x4 num[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) num[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < SPLITS; ++s) {
    const float w = __builtin_amdgcn_exp2f(m[s] - mx);
    den += w * l[s];
#pragma unroll
    for (int g = 0; g < 4; ++g) num[g] += w * part[s][g];
  }
  const float inv = 1.0f / den;
  u32x4 first, second;
  normalised_runs<T>(num, inv, first, second);
  const int row = tile * KB + l32;
  if (row >= t) return;
  T* dst = o + ((size_t)n * t + row) * D + dt * 32 + lk * 8;
  *reinterpret_cast<u32x4*>(dst) = first;
  *reinterpret_cast<u32x4*>(dst + 16) = second;
}

constexpr int kMaxSplits = 8;
int tiles_of(int t) { return (t + KB - 1) / KB; }

// ranges of keys per query block: as many workgroups as compute units, two key blocks at least; independent of the batch, so
// that a frame's bits do not depend on what it is batched with.  A whole call in us, by ranges: 1024 tokens 4 46.8, 6 43.3, 7 42.6,
// 8 42.8; 3600 tokens 5 76.2, 6 74.1, 7 73.4, 8 74.5; 5400 tokens 3 135.5, 4 120.8, 5 114.0, 6 (past one round) 151.7; 8372 tokens 2
// 270, 3 217, 4 287; 12 000 tokens 1 647, 2 404, 3 500.  A range costs t * 2 KiB of workspace: 5400 tokens take 78 MB with five,
// 56 with three.
int splits_of(int t) {
  const int nkb = tiles_of(t), nqb = (nkb + 3) / 4;
  return max(1, min(min(256 / nqb, kMaxSplits), (nkb + 1) / 2));
}

template <typename T, int S = 2>
void combine(const float* opart, const float* ml, T* o, int n, int t, int splits, hipStream_t s) {
  if constexpr (S <= kMaxSplits) {
    if (splits == S) hipLaunchKernelGGL((attn_combine_kernel<T, S>), dim3((unsigned)tiles_of(t), D / 128, (unsigned)n), dim3(256), 0, s, opart, ml, o, t, tiles_of(t));
    else combine<T, S + 1>(opart, ml, o, n, t, splits, s);
  }
}

template <typename T, bool WHOLE>
int launch_flash(const void* frag, void* o, void* scratch, int n, int t, float scale, hipStream_t s) {
  const int splits = splits_of(t), nkb = tiles_of(t), nqb = (nkb + 3) / 4;
  const size_t per = (size_t)nkb * TILE;
  const T* q = (const T*)frag;
  float* opart = (float*)scratch;
  float* ml = WHOLE ? nullptr : opart + (size_t)n * splits * per;
  static std::once_flag attr_once;
  hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void*)flash_attn_kernel<T, WHOLE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmemBytes); });
  WMDEC_HIP(attr_err);
  hipLaunchKernelGGL((flash_attn_kernel<T, WHOLE>), dim3((unsigned)(nqb * splits * n)), dim3(NT), kSmemBytes, s, q, q + n * per, q + 2 * n * per, per,
                     WHOLE ? o : scratch, ml, t, nqb, splits, scale * 1.4426950408889634f);
  WMDEC_HIP(hipGetLastError());
  if (!WHOLE) combine<T>(opart, ml, (T*)o, n, t, splits, s);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

template <typename T>
int launch_qkv_t(const ConvArgs& a, void* frag, hipStream_t s) {
  QkvParams p;
  p.x = a.x; p.mean = a.mean; p.rstd = a.rstd; p.gamma = a.gamma; p.beta = a.beta;
  p.rows_in = (const Moments*)a.rows_in; p.rows_in_count = a.rows_in_count; p.eps = a.eps;
  p.w = a.wt; p.bias = a.bias; p.frag = frag;
  p.n = a.n; p.t = a.h * a.w; p.groups = a.groups; p.tiles = (p.t + QT - 1) / QT;
  p.w_bytes = (int)(packed_elems(1, 3 * D, D) * sizeof(T));
  const size_t smem = (size_t)QT * D * sizeof(T) + (size_t)(D + a.groups) * sizeof(float2);
  static std::once_flag attr_once;
  hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void*)attn_qkv_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024); });
  WMDEC_HIP(attr_err);
  hipLaunchKernelGGL(attn_qkv_kernel<T>, dim3((unsigned)(p.tiles * 3 * p.n)), dim3(QNT), smem, s, p);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

}  // namespace

size_t attention_fragment_bytes(int n, int t) { return (size_t)n * 3 * tiles_of(t) * TILE * 2; }

size_t flash_attention_scratch_bytes(int n, int t) { return splits_of(t) == 1 ? 0 : (size_t)n * splits_of(t) * tiles_of(t) * KB * (D + 2) * sizeof(float); }

int flash_attention_num_launches(int t) { return splits_of(t) == 1 ? 1 : 2; }

const char* attention_qkv_label(int dtype) { return dtype == WMDEC_BF16 ? "attn_qkv_kernel<wmdec::bf16_t>" : "attn_qkv_kernel<wmdec::f16_t>"; }

void attention_qkv_grid(const ConvArgs& a, NextWeights* next) {
  next->per_tile = (a.h * a.w + QT - 1) / QT * a.n;
  next->tile_blocks = D / 32;
  next->total = next->per_tile * 3;
}

int launch_attention_qkv(const ConvArgs& a, void* frag, hipStream_t s) {
  WMDEC_REQUIRE(a.cin == D && a.cout == 3 * D && a.ksize == 1 && is_16bit(a.op_dtype) && a.x_dtype == a.op_dtype && a.bias && !a.res, WMDEC_ERR_UNSUPPORTED,
                "attention: the projection takes %d channels in a 16-bit type", D);
  WMDEC_REQUIRE((a.mean || a.rows_in) && !a.silu && a.groups > 0 && D % a.groups == 0, WMDEC_ERR_SHAPE, "attention: bad normalisation");
  WMDEC_REQUIRE(!a.rows_in || (a.rows_in_count >= 1 && a.rows_in_count <= 128), WMDEC_ERR_UNSUPPORTED, "attention: at most 128 triples per group can be merged in the prologue");
  return a.op_dtype == WMDEC_BF16 ? launch_qkv_t<bf16_t>(a, frag, s) : launch_qkv_t<f16_t>(a, frag, s);
}

int launch_flash_attention(const void* frag, void* o, void* scratch, int dtype, int n, int t, float scale, hipStream_t s) {
  WMDEC_REQUIRE(is_16bit(dtype) && n > 0 && t > 0 && frag && o && (scratch || splits_of(t) == 1), WMDEC_ERR_INVALID_ARG, "attention: bad arguments");
  if (splits_of(t) == 1) return dtype == WMDEC_BF16 ? launch_flash<bf16_t, true>(frag, o, scratch, n, t, scale, s) : launch_flash<f16_t, true>(frag, o, scratch, n, t, scale, s);
  return dtype == WMDEC_BF16 ? launch_flash<bf16_t, false>(frag, o, scratch, n, t, scale, s) : launch_flash<f16_t, false>(frag, o, scratch, n, t, scale, s);
}

}  // namespace wmdec
