// Horizontal fusion of the DiT's AdaLN projections (Sec. IV-B-2): the shift, scale and gate vectors of a block are
// three small products of the same conditioning vector; with the three weight matrices stored as one row-concatenated
// matrix they are one product, one launch, one pass over the weights.
//
// With a handful of conditioning vectors per call (one per frame) the product is a matrix-vector product: every weight
// is used `batch` times, far below the ridge point, so the bound is the single read of the weights from HBM and the
// matrix cores have nothing to add.  A wavefront owns two or four weight rows: a lane reads 16 contiguous bytes of
// each row per step (a wavefront's load is 1 KiB of one row), the activated conditioning vectors sit in LDS as fp32
// and are read once per step for all of them, partial sums stay in registers and are reduced over the 64 lanes at
// the end in a fixed order.  What a call takes beside the weights (22 MB at 1920, 4.3 us) is the launch, the trip to memory and the vectors' activation:
// asked for behind the weights, stored word by word and read two ways into the same banks they were most of it.  us at 1920 bf16, before / now, by the
// vectors: one 8.2 / 5.6, two 10.8 / 6.3, four 16.8 / 8.6, eight 28.6 / 14.0; 384: 3.5 / 2.3 to 12.0 / 3.9.
#include "conv_device.hpp"

namespace wmdec {
namespace {

constexpr int kWaves = 4;
constexpr int kMaxBatch = 16;
constexpr int kMaxLdsFloats = 16384;   // batch * d_cond fp32 values of the conditioning vectors (64 KiB)
constexpr int kMaxSteps = 8;           // 16-byte steps of a lane along a row: d_cond <= 8 * 64 * (16 / sizeof(weight))

template <typename T> struct Vec8 { static constexpr int N = 16 / sizeof(T); T v[16 / sizeof(T)]; };

// B: conditioning vectors the accumulators are sized for (batch rounded up); STEPS: 16-byte steps per lane and row.
// All RW x STEPS weight vectors of a wavefront are requested before the first is used: the kernel lives on loads in
// flight, and a loop that waits for one step before it asks for the next would pay the HBM latency STEPS times.  Loads return in order, so what is
// needed before the weights (the first conditioning vectors) and what would be a trip of its own behind them (the bias) are asked for in front of them.
template <typename TW, int B, int STEPS, int RW>
__global__ __launch_bounds__(64 * kWaves) void adaln_projection_kernel(const void* __restrict__ c, int c_dtype, const TW* __restrict__ w,
                                                                       const float* __restrict__ bias, float* __restrict__ out,
                                                                       int batch, int d_cond, int rows, int apply_silu) {
  constexpr int V = 16 / sizeof(TW), NT = 64 * kWaves;   // weights per 16-byte load
  // [B][d_cond], vectors past `batch` are zero; four values a place.  A lane takes V of them at a time: where that is eight, all first fours come
  // first and the others behind them, so that the lanes' reads are next to each other.
  extern __shared__ __align__(16) float s_a[];
  const int fours = B * d_cond / 4;
  auto place = [&](int f) -> float4& { return reinterpret_cast<float4*>(s_a)[V == 8 ? (f & 1) * (fours / 2) + f / 2 : f]; };
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = (blockIdx.x * kWaves + wave) * RW;
  const int per = c_dtype == WMDEC_F32 ? 4 : 8;            // elements per 16-byte load of the conditioning vectors, four loads in flight per thread
  const int nvec = batch * d_cond / per, total = B * d_cond / per;
  uint4 q[4];
  auto ask = [&](int i0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = reinterpret_cast<const uint4*>(c)[min(i0 + u * NT, nvec - 1)];
  };
  ask(tid);
  float bv[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) bv[r] = bias ? bias[min(row0 + r, rows - 1)] : 0.f;
  __builtin_amdgcn_sched_barrier(0);
  Vec8<TW> wv[RW][STEPS];
#pragma unroll
  for (int r = 0; r < RW; ++r)   // rows and columns past the end re-read valid elements; they are masked below
#pragma unroll
    for (int st = 0; st < STEPS; ++st)
      wv[r][st] = *reinterpret_cast<const Vec8<TW>*>(w + (size_t)min(row0 + r, rows - 1) * d_cond + min((st * 64 + lane) * V, d_cond - V));
  __builtin_amdgcn_sched_barrier(0);
  // conditioning vectors -> LDS as fp32, activated
  for (int i0 = tid; i0 < total; i0 += 4 * NT) {
    if (i0 != tid) ask(i0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * NT;
      if (i >= total) continue;
      auto act = [&](float v) -> float {
        if (i >= nvec) return 0.f;
        return apply_silu ? silu_f(v) : v;
      };
      if (c_dtype == WMDEC_F32) {
        place(i) = make_float4(act(__uint_as_float(q[u].x)), act(__uint_as_float(q[u].y)), act(__uint_as_float(q[u].z)), act(__uint_as_float(q[u].w)));
      } else {
        const uint32_t wd[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
        float t[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (c_dtype == WMDEC_BF16) { t[2 * e] = to_float(bf16_t{(uint16_t)(wd[e] & 0xffffu)}); t[2 * e + 1] = to_float(bf16_t{(uint16_t)(wd[e] >> 16)}); }
          else { t[2 * e] = to_float(f16_t{(uint16_t)(wd[e] & 0xffffu)}); t[2 * e + 1] = to_float(f16_t{(uint16_t)(wd[e] >> 16)}); }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
          place(2 * i + h) = make_float4(act(t[4 * h]), act(t[4 * h + 1]), act(t[4 * h + 2]), act(t[4 * h + 3]));
      }
    }
  }
  __syncthreads();
  if (row0 >= rows) return;
  float acc[RW][B];
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[r][b] = 0.f;
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    const int k0 = (st * 64 + lane) * V;
    if (k0 < d_cond) {
#pragma unroll
      for (int b = 0; b < B; ++b) {
        float a[V];
#pragma unroll
        for (int j = 0; j < V; j += 4) {
          const float4 t = place((b * d_cond + k0 + j) / 4);
          a[j] = t.x; a[j + 1] = t.y; a[j + 2] = t.z; a[j + 3] = t.w;
        }
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
          for (int j = 0; j < V; ++j) acc[r][b] = fmaf(to_float(wv[r][st].v[j]), a[j], acc[r][b]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const float v = swap_sum<32>(swap_sum<16>(lane_group_sum<16>(acc[r][b])));
      if (lane == 0 && row0 + r < rows && b < batch) out[(size_t)b * rows + row0 + r] = v + bv[r];
    }
}

template <typename TW, int B, int STEPS, int RW>
int launch_rows(const void* c, int c_dtype, const void* w, const float* bias, float* out, int batch, int d_cond, int rows, int silu, hipStream_t s) {
  const dim3 grid((unsigned)((rows + kWaves * RW - 1) / (kWaves * RW)));
  const size_t smem = (size_t)B * d_cond * sizeof(float);
  auto kern = adaln_projection_kernel<TW, B, STEPS, RW>;
  if (smem > 48 * 1024) WMDEC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  hipLaunchKernelGGL(kern, grid, dim3(64 * kWaves), smem, s, c, c_dtype, (const TW*)w, bias, out, batch, d_cond, rows, silu);
  WMDEC_HIP(hipGetLastError());
  return WMDEC_OK;
}

template <typename TW, int B, int STEPS>
int launch_k(const void* c, int c_dtype, const void* w, const float* bias, float* out, int batch, int d_cond, int rows, int silu, hipStream_t s) {
  // Rows of a wavefront: two, so that the rows of most layers are dealt to the compute units more evenly, as long as three workgroups' vectors fit a compute
  // unit's LDS; beyond that four, which activate the vectors half as often.  us, four / two rows: bf16 1920 one vector 6.39 / 5.61, four 9.70 / 8.55, eight
  // 13.95 / 16.5; 1472 eight 11.3 / 10.4; 384 one 2.47 / 2.28; f32 1920 one 10.75 / 9.28, eight 18.4 / 19.4.
  if ((long)B * d_cond <= 12288) return launch_rows<TW, B, STEPS, 2>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  return launch_rows<TW, B, STEPS, 4>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
}

template <typename TW, int B>
int launch_s(const void* c, int c_dtype, const void* w, const float* bias, float* out, int batch, int d_cond, int rows, int silu, hipStream_t s) {
  const int steps = (d_cond + 64 * (16 / (int)sizeof(TW)) - 1) / (64 * (16 / (int)sizeof(TW)));
  if (steps <= 1) return launch_k<TW, B, 1>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  if (steps <= 2) return launch_k<TW, B, 2>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  if (steps <= 4) return launch_k<TW, B, 4>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  return launch_k<TW, B, 8>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
}

template <typename TW>
int launch_b(const void* c, int c_dtype, const void* w, const float* bias, float* out, int batch, int d_cond, int rows, int silu, hipStream_t s) {
  if (batch <= 1) return launch_s<TW, 1>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  if (batch <= 2) return launch_s<TW, 2>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  if (batch <= 4) return launch_s<TW, 4>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  if (batch <= 8) return launch_s<TW, 8>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
  return launch_s<TW, 16>(c, c_dtype, w, bias, out, batch, d_cond, rows, silu, s);
}

}  // namespace

// conditioning vectors one launch can take: the accumulators are sized for the batch rounded up to a power of two, and
// that many vectors of d_cond fp32 values must fit the LDS budget
int adaln_max_batch(int d_cond) {
  if (d_cond <= 0) return 0;
  int b = kMaxBatch;
  while (b > 1 && (long)b * d_cond > kMaxLdsFloats) b >>= 1;
  return (long)b * d_cond > kMaxLdsFloats ? 0 : b;
}

int adaln_max_d_cond(int w_dtype) { return kMaxSteps * 64 * (int)(16 / dtype_size(w_dtype)); }

int launch_adaln_projection(const void* c, int c_dtype, const void* w, int w_dtype, const float* bias, float* out, int batch,
                            int d_cond, int rows, int apply_silu, hipStream_t s) {
  switch (w_dtype) {
    case WMDEC_F32: return launch_b<float>(c, c_dtype, w, bias, out, batch, d_cond, rows, apply_silu, s);
    case WMDEC_BF16: return launch_b<bf16_t>(c, c_dtype, w, bias, out, batch, d_cond, rows, apply_silu, s);
    default: return launch_b<f16_t>(c, c_dtype, w, bias, out, batch, d_cond, rows, apply_silu, s);
  }
}

}  // namespace wmdec
