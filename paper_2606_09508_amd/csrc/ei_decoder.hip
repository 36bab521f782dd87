// The passes of a decoder layer between its matrix products, one pass over
// memory each (prefill.py's layer around the attention):
//
//  add_rmsnorm_kernel  s = x + y (rounded to bf16), h = RMSNorm(s) * gain: the
//                      residual sum and the norm that reads it, a row held in
//                      registers between the two
//  rope_heads_kernel   q, k, v as the projections leave them ([B][N][H][128])
//                      to head-major [B][H][N][128], q and k rotated
//  swiglu_kernel       silu(g) * u
//  rope_tables_kernel  the rotary embedding's cosines and sines
//
// The first three are bound by HBM.  Written as separate tensor operations the same
// passes widened every operand to fp32 in memory and read and wrote it again
// per operation: 1.27 ms of the 4.2 ms of an 8B-shaped layer at 8192 tokens.
// Here each operand is read once and each result written once:
//   add_rmsnorm, 8192 x 4096:                    43 us, 6.3 TB/s (23 us without the sum)
//   rope_heads, 8192 tokens, 32 + 8 + 8 heads:   42 us, 4.8 TB/s
//   swiglu, 8192 x 14336:                        124 us, 5.7 TB/s
// Every value is computed in fp32 with the roundings to bf16 where the tensor
// operations have them (the sum, silu, the product, the rotated pair), so the
// results differ from theirs only by the order of a row's sum of squares.
#include "../../include/entropyinfer.h"
#include "ei_internal.h"

#include <limits.h>

// a cos - b sin keeps its two rounded products, as two tensor operations do
#pragma clang fp contract(off)

namespace ei {
namespace {

constexpr int kThreads = 256;
constexpr int kNormMaxCols = 16384;
// A launch's threads are counted in 32 bits and one of more does less without
// an error, so work of more workgroups than these takes several launches.
constexpr int64_t kMaxGrid = (1ll << 31) / kThreads;
unsigned launch_grid(int64_t left) { return (unsigned)(left < kMaxGrid ? left : kMaxGrid); }

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  const f32x2 x = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));   // round to nearest even
}
__device__ __forceinline__ void widen8(uint4 w, float (&f)[8]) {
  const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = bf16_lo(ww[e]);
    f[2 * e + 1] = bf16_hi(ww[e]);
  }
}
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// T threads per row (a wave for rows of up to 1024 columns, which leaves no
// barrier; else the workgroup), CH chunks of 8 columns per thread.  sum_out
// may be x or y (so none of the three is restrict): a thread stores a chunk
// after it has loaded its chunks of both.
template <int T, int CH, bool ADD>
__global__ __launch_bounds__(kThreads) void add_rmsnorm_kernel(
    const uint16_t* x, const uint16_t* y, const uint16_t* __restrict__ gain, int64_t rows,
    int cols, float eps, uint16_t* sum_out, uint16_t* __restrict__ out) {
  __shared__ float part[kThreads / kWave];
  const int t = threadIdx.x % T;
  const int64_t row = (int64_t)blockIdx.x * (kThreads / T) + threadIdx.x / T;
  if (T < kThreads && row >= rows) return;   // T == kThreads: the grid is the rows
  const int nch = cols / 8;
  const size_t base = (size_t)row * nch;
  uint4 w[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (t + c * T < nch) w[c] = ((const uint4*)x)[base + t + c * T];
  if constexpr (ADD) {
    uint4 z[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (t + c * T < nch) z[c] = ((const uint4*)y)[base + t + c * T];
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (t + c * T < nch) {
        float a[8], b[8];
        widen8(w[c], a);
        widen8(z[c], b);
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] += b[e];
        w[c] = pack8(a);
        ((uint4*)sum_out)[base + t + c * T] = w[c];
      }
  }
  float ss = 0.0f;
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (t + c * T < nch) {
      float a[8];
      widen8(w[c], a);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss += a[e] * a[e];
    }
  ss = wave_sum(ss);
  if constexpr (T > kWave) {
    if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = ss;
    __syncthreads();
    ss = (part[0] + part[1]) + (part[2] + part[3]);
  }
  const float r = rsqrtf(ss / (float)cols + eps);
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (t + c * T < nch) {
      float a[8], g[8];
      widen8(w[c], a);
      widen8(((const uint4*)gain)[t + c * T], g);
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = (a[e] * r) * g[e];
      ((uint4*)out)[base + t + c * T] = pack8(a);
    }
}

// One workgroup: 32 positions of up to kRopeHeads heads (q's, then k's, then
// v's).  Eight lanes hold a position: dims 8c .. 8c+7 and their partners 64
// further on, with the position's 16 table values kept in registers over the
// heads (reloaded per head the table would be read twice as often as the
// data).  Each head's 32 rows are written as one 8 KB run.
constexpr int kRopeHeads = 8, kRopePos = kThreads / 8;

__global__ __launch_bounds__(kThreads) void rope_heads_kernel(
    const uint16_t* __restrict__ qi, const uint16_t* __restrict__ ki,
    const uint16_t* __restrict__ vi, const float* __restrict__ cosv,
    const float* __restrict__ sinv, int N, int Hq, int Hkv, int n_pos, unsigned g0,
    uint16_t* __restrict__ qo, uint16_t* __restrict__ ko, uint16_t* __restrict__ vo) {
  const unsigned wg = g0 + blockIdx.x;   // (g0: the launch's first)
  const int pb = (int)(wg % (unsigned)n_pos), hb = (int)(wg / (unsigned)n_pos);
  const int groups = (Hq + 2 * Hkv + kRopeHeads - 1) / kRopeHeads;
  const int b = hb / groups, h0 = (hb % groups) * kRopeHeads;
  const int c = threadIdx.x & 7;
  const int n = pb * kRopePos + (threadIdx.x >> 3);
  if (n >= N) return;
  float cs[8], sn[8];
  {
    const float4* cp = (const float4*)(cosv + (size_t)n * 64 + 8 * c);
    const float4* sp = (const float4*)(sinv + (size_t)n * 64 + 8 * c);
    const float4 c0 = cp[0], c1 = cp[1], s0 = sp[0], s1 = sp[1];
    cs[0] = c0.x; cs[1] = c0.y; cs[2] = c0.z; cs[3] = c0.w;
    cs[4] = c1.x; cs[5] = c1.y; cs[6] = c1.z; cs[7] = c1.w;
    sn[0] = s0.x; sn[1] = s0.y; sn[2] = s0.z; sn[3] = s0.w;
    sn[4] = s1.x; sn[5] = s1.y; sn[6] = s1.z; sn[7] = s1.w;
  }
  uint4 w[kRopeHeads][2];
  // which tensor head h belongs to (workgroup-uniform)
  auto place = [&](int h, const uint16_t*& in, uint16_t*& out, int& H, int& hh) {
    if (h < Hq) { in = qi; out = qo; H = Hq; hh = h; }
    else if (h < Hq + Hkv) { in = ki; out = ko; H = Hkv; hh = h - Hq; }
    else { in = vi; out = vo; H = Hkv; hh = h - Hq - Hkv; }
  };
#pragma unroll
  for (int i = 0; i < kRopeHeads; ++i)
    if (h0 + i < Hq + 2 * Hkv) {
      const uint16_t* in; uint16_t* out; int H, hh;
      place(h0 + i, in, out, H, hh);
      const uint16_t* p = in + (((size_t)b * N + n) * H + hh) * kHeadDim + 8 * c;
      w[i][0] = *(const uint4*)p;
      w[i][1] = *(const uint4*)(p + 64);
    }
#pragma unroll
  for (int i = 0; i < kRopeHeads; ++i)
    if (h0 + i < Hq + 2 * Hkv) {
      const uint16_t* in; uint16_t* out; int H, hh;
      place(h0 + i, in, out, H, hh);
      if (h0 + i < Hq + Hkv) {
        float a[8], d[8], u[8], v[8];
        widen8(w[i][0], a);
        widen8(w[i][1], d);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          u[e] = a[e] * cs[e] - d[e] * sn[e];
          v[e] = a[e] * sn[e] + d[e] * cs[e];
        }
        w[i][0] = pack8(u);
        w[i][1] = pack8(v);
      }
      uint16_t* p = out + (((size_t)b * H + hh) * N + n) * kHeadDim + 8 * c;
      *(uint4*)p = w[i][0];
      *(uint4*)(p + 64) = w[i][1];
    }
}

// cos / sin of position * theta^(-2i / D), [N][half], the fp32 operations of
// the tensor form one after another (power, reciprocal, product, cos, sin) in
// one launch: as ten, the tables of a short prompt took 45 us of it.
// (e0: the launch's first element)
__global__ __launch_bounds__(kThreads) void rope_tables_kernel(int64_t e0, int64_t n, int half,
                                                              float D, float theta,
                                                              float* __restrict__ cosv,
                                                              float* __restrict__ sinv) {
  const int64_t e = e0 + (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= n) return;
  const int64_t pos = e / half;
  const int i = (int)(e - pos * half);
  // (the tensor's division by a number is a product with its reciprocal)
  const float inv = 1.0f / powf(theta, (float)(2 * i) * (1.0f / D));
  const float ang = (float)pos * inv;
  cosv[e] = cosf(ang);
  sinv[e] = sinf(ang);
}

// x / (1 + exp(-x)), every bf16 value of x rounding to the tensor operation's
// result.  That takes the IEEE division (an approximate reciprocal misrounds
// x = 5.9375); the exponential may be the base-2 instruction of a rounded
// product (2047 x 14336, operands in cache: 26.5 us, with expf 29.1).
__device__ __forceinline__ float silu(float x) {
  return x / (1.0f + __builtin_amdgcn_exp2f(x * -1.4426950408889634f));
}

// Two chunks of 8 elements per thread.
constexpr int kSwigluChunks = 2;

__global__ __launch_bounds__(kThreads) void swiglu_kernel(const uint16_t* g, const uint16_t* u,
                                                          int64_t n_chunks, uint16_t* out) {
  const int64_t i0 = (int64_t)blockIdx.x * (kThreads * kSwigluChunks) + threadIdx.x;
  uint4 wg[kSwigluChunks], wu[kSwigluChunks];
#pragma unroll
  for (int c = 0; c < kSwigluChunks; ++c)
    if (i0 + c * kThreads < n_chunks) {
      wg[c] = ((const uint4*)g)[i0 + c * kThreads];
      wu[c] = ((const uint4*)u)[i0 + c * kThreads];
    }
#pragma unroll
  for (int c = 0; c < kSwigluChunks; ++c)
    if (i0 + c * kThreads < n_chunks) {
      float a[8], b[8];
      widen8(wg[c], a);
      widen8(wu[c], b);
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = silu(a[e]);
      widen8(pack8(a), a);   // silu is rounded to bf16 before the product
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] *= b[e];
      ((uint4*)out)[i0 + c * kThreads] = pack8(a);
    }
}

template <int T, int CH>
void launch_norm_t(const uint16_t* x, const uint16_t* y, const uint16_t* gain, int64_t rows,
                   int cols, float eps, uint16_t* sum_out, uint16_t* out, hipStream_t stream) {
  constexpr int64_t per = kThreads / T;
  const int64_t groups = (rows + per - 1) / per;
  for (int64_t g0 = 0; g0 < groups; g0 += kMaxGrid) {
    const dim3 grid(launch_grid(groups - g0));
    const int64_t left = rows - g0 * per;
    const size_t at = (size_t)(g0 * per) * cols;
    if (y)
      hipLaunchKernelGGL((add_rmsnorm_kernel<T, CH, true>), grid, dim3(kThreads), 0, stream, x + at,
                         y + at, gain, left, cols, eps, sum_out + at, out + at);
    else
      hipLaunchKernelGGL((add_rmsnorm_kernel<T, CH, false>), grid, dim3(kThreads), 0, stream,
                         x + at, nullptr, gain, left, cols, eps, nullptr, out + at);
  }
}

hipError_t launch_add_rmsnorm(const uint16_t* x, const uint16_t* y, const uint16_t* gain,
                              int64_t rows, int cols, float eps, uint16_t* sum_out, uint16_t* out,
                              hipStream_t stream) {
  if (cols <= 512) launch_norm_t<kWave, 1>(x, y, gain, rows, cols, eps, sum_out, out, stream);
  else if (cols <= 1024) launch_norm_t<kWave, 2>(x, y, gain, rows, cols, eps, sum_out, out, stream);
  else if (cols <= 2048) launch_norm_t<kThreads, 1>(x, y, gain, rows, cols, eps, sum_out, out, stream);
  else if (cols <= 4096) launch_norm_t<kThreads, 2>(x, y, gain, rows, cols, eps, sum_out, out, stream);
  else if (cols <= 8192) launch_norm_t<kThreads, 4>(x, y, gain, rows, cols, eps, sum_out, out, stream);
  else launch_norm_t<kThreads, 8>(x, y, gain, rows, cols, eps, sum_out, out, stream);
  return hipGetLastError();
}

hipError_t launch_rope_heads(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                             const float* cosv, const float* sinv, int B, int N, int Hq, int Hkv,
                             uint16_t* qo, uint16_t* ko, uint16_t* vo, hipStream_t stream) {
  const int n_pos = (N + kRopePos - 1) / kRopePos;
  const int groups = (Hq + 2 * Hkv + kRopeHeads - 1) / kRopeHeads;
  const int64_t total = (int64_t)B * groups * n_pos;
  for (int64_t g0 = 0; g0 < total; g0 += kMaxGrid)
    hipLaunchKernelGGL(rope_heads_kernel, dim3(launch_grid(total - g0)), dim3(kThreads), 0, stream,
                       q, k, v, cosv, sinv, N, Hq, Hkv, n_pos, (unsigned)g0, qo, ko, vo);
  return hipGetLastError();
}

hipError_t launch_swiglu(const uint16_t* g, const uint16_t* u, int64_t n, uint16_t* out,
                         hipStream_t stream) {
  constexpr int64_t per = kThreads * kSwigluChunks;
  const int64_t chunks = n / 8, groups = (chunks + per - 1) / per;
  for (int64_t g0 = 0; g0 < groups; g0 += kMaxGrid) {
    const size_t at = (size_t)(g0 * per * 8);
    hipLaunchKernelGGL(swiglu_kernel, dim3(launch_grid(groups - g0)), dim3(kThreads), 0, stream,
                       g + at, u + at, chunks - g0 * per, out + at);
  }
  return hipGetLastError();
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }
template <class... P>
bool aligned16(const void* p, P... more) { return aligned16(p) && aligned16(more...); }
ei_status from_hip(hipError_t e) { return e == hipSuccess ? EI_OK : EI_ERR_LAUNCH; }

}  // namespace
}  // namespace ei

extern "C" {

ei_status ei_add_rmsnorm(const uint16_t* x, const uint16_t* y, const uint16_t* gain, int64_t rows,
                         int32_t cols, float eps, uint16_t* sum_out, uint16_t* out, void* stream) {
  if (rows < 0 || cols <= 0 || rows > INT_MAX) return EI_ERR_SHAPE;
  if (cols % 8 || cols > ei::kNormMaxCols) return EI_ERR_UNSUPPORTED;
  if (rows == 0) return EI_OK;
  if (!x || !gain || !out || (y && !sum_out)) return EI_ERR_NULL;
  if (!ei::aligned16(x, y, gain, out) || (y && !ei::aligned16(sum_out))) return EI_ERR_UNSUPPORTED;
  return ei::from_hip(
      ei::launch_add_rmsnorm(x, y, gain, rows, cols, eps, sum_out, out, (hipStream_t)stream));
}

ei_status ei_rope_heads(const uint16_t* q_in, const uint16_t* k_in, const uint16_t* v_in,
                        const float* cos_table, const float* sin_table, ei_dims d, uint16_t* q_out,
                        uint16_t* k_out, uint16_t* v_out, void* stream) {
  if (d.batch < 0 || d.seq_len < 0 || d.n_q_heads <= 0 || d.n_kv_heads <= 0 || d.head_dim <= 0 ||
      d.n_q_heads % d.n_kv_heads)
    return EI_ERR_SHAPE;
  // workgroups: eight heads of 32 positions of a batch entry each
  const int64_t heads = (int64_t)d.n_q_heads + 2 * (int64_t)d.n_kv_heads;
  const int64_t groups = (heads + ei::kRopeHeads - 1) / ei::kRopeHeads;
  const int64_t n_pos = ((int64_t)d.seq_len + ei::kRopePos - 1) / ei::kRopePos;
  if (heads > INT_MAX / 2 || d.batch * groups > INT_MAX || d.batch * groups * n_pos > INT_MAX)
    return EI_ERR_SHAPE;
  if (d.head_dim != ei::kHeadDim) return EI_ERR_UNSUPPORTED;
  if (d.batch == 0 || d.seq_len == 0) return EI_OK;
  if (!q_in || !k_in || !v_in || !cos_table || !sin_table || !q_out || !k_out || !v_out)
    return EI_ERR_NULL;
  if (!ei::aligned16(q_in, k_in, v_in, cos_table, sin_table, q_out, k_out, v_out))
    return EI_ERR_UNSUPPORTED;
  return ei::from_hip(ei::launch_rope_heads(q_in, k_in, v_in, cos_table, sin_table, d.batch,
                                            d.seq_len, d.n_q_heads, d.n_kv_heads, q_out, k_out,
                                            v_out, (hipStream_t)stream));
}

ei_status ei_rope_tables(int32_t seq_len, int32_t head_dim, float theta, float* cos_table,
                         float* sin_table, void* stream) {
  if (seq_len < 0 || head_dim <= 0 || !(theta > 0.0f)) return EI_ERR_SHAPE;
  const int32_t half = (int32_t)(((int64_t)head_dim + 1) / 2);
  const int64_t n = (int64_t)seq_len * half, groups = (n + ei::kThreads - 1) / ei::kThreads;
  if (groups > INT_MAX) return EI_ERR_SHAPE;
  if (n == 0) return EI_OK;
  if (!cos_table || !sin_table) return EI_ERR_NULL;
  if (((uintptr_t)cos_table | (uintptr_t)sin_table) & 3) return EI_ERR_UNSUPPORTED;
  for (int64_t g0 = 0; g0 < groups; g0 += ei::kMaxGrid)
    hipLaunchKernelGGL(ei::rope_tables_kernel, dim3(ei::launch_grid(groups - g0)),
                       dim3(ei::kThreads), 0, (hipStream_t)stream, g0 * ei::kThreads, n, half,
                       (float)head_dim, theta, cos_table, sin_table);
  return ei::from_hip(hipGetLastError());
}

ei_status ei_swiglu(const uint16_t* g, const uint16_t* u, int64_t n, uint16_t* out, void* stream) {
  if (n < 0 || n / 4096 > INT_MAX) return EI_ERR_SHAPE;
  if (n % 8) return EI_ERR_UNSUPPORTED;
  if (n == 0) return EI_OK;
  if (!g || !u || !out) return EI_ERR_NULL;
  if (!ei::aligned16(g, u, out)) return EI_ERR_UNSUPPORTED;
  return ei::from_hip(ei::launch_swiglu(g, u, n, out, (hipStream_t)stream));
}

}  // extern "C"
