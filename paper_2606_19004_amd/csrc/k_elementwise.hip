// Memory-bound and latency-bound kernels of the denoise step for gfx950:
//   flow_update    fused Euler / SDE latent update (fp32, 16-byte vector access)
//   flow_logprob   per-sample Gaussian log-density of an SDE step (fp64 sums)
//   ln_modulate    LayerNorm (fp32 statistics) + adaLN modulate, one wave per row
//   gemv           batched GEMV for the adaLN / timestep / final modulation vectors
//   reward_stats   per prompt-group mean, std, advantages, stable descending ranks
//   small helpers  fp32->bf16 cast, timestep sinusoid, RoPE cos/sin table
#include <type_traits>

#include "internal.h"

namespace dit {

template <typename T> struct Vec8;
template <> struct Vec8<u16> {
  static __device__ __forceinline__ void load(const u16* p, float* f) {
    uint4 u = *(const uint4*)p;
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void store(u16* p, const float* f) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; i++)
      w[i] = (uint32_t)from_f32<u16>(f[2 * i]) | ((uint32_t)from_f32<u16>(f[2 * i + 1]) << 16);
    *(uint4*)p = make_uint4(w[0], w[1], w[2], w[3]);
  }
};
template <> struct Vec8<float> {
  static __device__ __forceinline__ void load(const float* p, float* f) {
    float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
  static __device__ __forceinline__ void store(float* p, const float* f) {
    *(float4*)p = make_float4(f[0], f[1], f[2], f[3]);
    *(float4*)(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
  }
};

__device__ __forceinline__ float silu(float x) { return x / (1.0f + __expf(-x)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---------------------------------------------------------------------------
// flow update: x' = cx*x + cv*v + ce*noise. The host folds the sampler step
// (Euler ODE or reverse-time SDE, both linear in x, v and noise) into these
// three coefficients in double precision.
// ---------------------------------------------------------------------------
template <bool NOISE>
__global__ void __launch_bounds__(256) flow_update_vec(float4* __restrict__ x, const float4* __restrict__ v,
                                                       const float4* __restrict__ e, int64_t n4,
                                                       float cx, float cv, float ce) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    float4 a = x[i], b = v[i];
    float4 r;
    r.x = fmaf(cx, a.x, cv * b.x);
    r.y = fmaf(cx, a.y, cv * b.y);
    r.z = fmaf(cx, a.z, cv * b.z);
    r.w = fmaf(cx, a.w, cv * b.w);
    if (NOISE) {
      float4 c = e[i];
      r.x = fmaf(ce, c.x, r.x);
      r.y = fmaf(ce, c.y, r.y);
      r.z = fmaf(ce, c.z, r.z);
      r.w = fmaf(ce, c.w, r.w);
    }
    x[i] = r;
  }
}

__global__ void flow_update_tail(float* x, const float* v, const float* e, int64_t start, int64_t n,
                                 float cx, float cv, float ce) {
  int64_t i = start + threadIdx.x;
  if (i < n) {
    float r = fmaf(cx, x[i], cv * v[i]);
    if (e) r = fmaf(ce, e[i], r);
    x[i] = r;
  }
}

__global__ void flow_update_scalar(float* x, const float* v, const float* e, int64_t n,
                                   float cx, float cv, float ce) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    float r = fmaf(cx, x[i], cv * v[i]);
    if (e) r = fmaf(ce, e[i], r);
    x[i] = r;
  }
}

// Log-density of an SDE step's output, one 1024-thread workgroup per sample: each thread sums
// (x_next - mean)^2 over a strided share of the sample in fp64 (the mean too is formed in fp64
// from the fp32 inputs), then the workgroup reduces in a fixed order.
template <bool VEC>
__global__ void __launch_bounds__(1024) flow_logprob_kernel(const float* __restrict__ x, const float* __restrict__ v,
                                                            const float* __restrict__ xn, int64_t n, double h,
                                                            double k1, double omt, double inv2var, double cst,
                                                            double* __restrict__ logp) {
  __shared__ double part[16];
  const int64_t base = (int64_t)blockIdx.x * n;
  double acc = 0.0;
  auto term = [&](float xf, float vf, float nf) {
    const double xd = xf, vd = vf;
    const double mean = xd + h * (vd + k1 * (xd + omt * vd));
    const double r = (double)nf - mean;
    acc = fma(r, r, acc);
  };
  if (VEC) {
    const float4* x4 = (const float4*)(x + base);
    const float4* v4 = (const float4*)(v + base);
    const float4* n4 = (const float4*)(xn + base);
    for (int64_t i = threadIdx.x; i < n / 4; i += 1024) {
      const float4 a = x4[i], b = v4[i], c = n4[i];
      term(a.x, b.x, c.x);
      term(a.y, b.y, c.y);
      term(a.z, b.z, c.z);
      term(a.w, b.w, c.w);
    }
  } else {
    for (int64_t i = threadIdx.x; i < n; i += 1024) term(x[base + i], v[base + i], xn[base + i]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < 16; w++) s += part[w];
    logp[blockIdx.x] = -s * inv2var + cst;
  }
}

hipError_t flow_logprob_launch(const float* x, const float* v, const float* xn, int batch, int64_t n, double h,
                               double k1, double omt, double inv2var, double cst, double* logp, hipStream_t s) {
  const bool vec = n % 4 == 0 && ((uintptr_t)x | (uintptr_t)v | (uintptr_t)xn) % 16 == 0;
  if (vec) flow_logprob_kernel<true><<<batch, 1024, 0, s>>>(x, v, xn, n, h, k1, omt, inv2var, cst, logp);
  else flow_logprob_kernel<false><<<batch, 1024, 0, s>>>(x, v, xn, n, h, k1, omt, inv2var, cst, logp);
  return hipGetLastError();
}

template <typename T, int MODE>
__global__ void __launch_bounds__(256) teacache_residual_kernel(T* __restrict__ x, float* __restrict__ r, int64_t n4) {
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n4; q += (int64_t)gridDim.x * 256) {
    float a[4];
    load4<T>(x + 4 * q, a);
    float4 rv = MODE == 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : *(const float4*)(r + 4 * q);
    if (MODE == 0) {
      *(float4*)(r + 4 * q) = make_float4(a[0], a[1], a[2], a[3]);
    } else if (MODE == 1) {
      *(float4*)(r + 4 * q) = make_float4(a[0] - rv.x, a[1] - rv.y, a[2] - rv.z, a[3] - rv.w);
    } else {
      float o[4] = {a[0] + rv.x, a[1] + rv.y, a[2] + rv.z, a[3] + rv.w};
      store4<T>(x + 4 * q, o);
    }
  }
}

hipError_t teacache_residual(void* x, float* r, int64_t n, int mode, int dtype, hipStream_t s) {
  const int64_t n4 = n / 4;
  if (n4 == 0) return hipSuccess;
  const int grid = (int)std::min<int64_t>(2048, cdiv(n4, (int64_t)256));
  if (dtype == DT_BF16) {
    if (mode == 0) teacache_residual_kernel<u16, 0><<<grid, 256, 0, s>>>((u16*)x, r, n4);
    else if (mode == 1) teacache_residual_kernel<u16, 1><<<grid, 256, 0, s>>>((u16*)x, r, n4);
    else teacache_residual_kernel<u16, 2><<<grid, 256, 0, s>>>((u16*)x, r, n4);
  } else {
    if (mode == 0) teacache_residual_kernel<float, 0><<<grid, 256, 0, s>>>((float*)x, r, n4);
    else if (mode == 1) teacache_residual_kernel<float, 1><<<grid, 256, 0, s>>>((float*)x, r, n4);
    else teacache_residual_kernel<float, 2><<<grid, 256, 0, s>>>((float*)x, r, n4);
  }
  return hipGetLastError();
}

hipError_t flow_update(float* x, const float* v, const float* noise, int64_t n, float cx, float cv, float ce,
                       hipStream_t s) {
  if (n <= 0) return hipSuccess;
  bool aligned = ((uintptr_t)x % 16 == 0) && ((uintptr_t)v % 16 == 0) && (!noise || (uintptr_t)noise % 16 == 0);
  if (aligned) {
    int64_t n4 = n / 4;
    if (n4 > 0) {
      int grid = (int)std::min<int64_t>(cdiv(n4, 256), 4096);
      if (noise)
        flow_update_vec<true><<<grid, 256, 0, s>>>((float4*)x, (const float4*)v, (const float4*)noise, n4, cx, cv, ce);
      else
        flow_update_vec<false><<<grid, 256, 0, s>>>((float4*)x, (const float4*)v, nullptr, n4, cx, cv, ce);
    }
    if (n % 4) flow_update_tail<<<1, 64, 0, s>>>(x, v, noise, n4 * 4, n, cx, cv, ce);
  } else {
    int grid = (int)std::min<int64_t>(cdiv(n, 256), 4096);
    flow_update_scalar<<<grid, 256, 0, s>>>(x, v, noise, n, cx, cv, ce);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__global__ void silu_kernel(const float* __restrict__ in, float* __restrict__ out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = silu(in[i]);
}
hipError_t silu_f32(const float* in, float* out, int64_t n, hipStream_t s) {
  if (n > 0) silu_kernel<<<cdiv(n, 256), 256, 0, s>>>(in, out, n);
  return hipGetLastError();
}

__global__ void cast_bf16_kernel(const float* __restrict__ in, u16* __restrict__ out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = from_f32<u16>(in[i]);
}
hipError_t cast_f32_to_bf16(const float* in, u16* out, int64_t n, hipStream_t s) {
  if (n > 0) cast_bf16_kernel<<<cdiv(n, 256), 256, 0, s>>>(in, out, n);
  return hipGetLastError();
}

// the two bf16 parts of x, hi + lo = x to 2^-16 relative
__device__ __forceinline__ void split_hilo(float x, u16& hi, u16& lo) {
  const __bf16 h = (__bf16)x, l = (__bf16)(x - (float)h);
  hi = __builtin_bit_cast(u16, h);
  lo = __builtin_bit_cast(u16, l);
}

// e = [cos(1000 t f_j) ; sin(1000 t f_j)], f_j = 10000^(-j/128), evaluated in fp64
__device__ __forceinline__ void sinusoid(double t, int j, float& c, float& s) {
  const double f = exp(-log(10000.0) * (double)j / 128.0);
  const double arg = 1000.0 * t * f;
  c = (float)cos(arg);
  s = (float)sin(arg);
}
__global__ void sinusoid_kernel(const float* t_dev, float t_scalar, float* e, int B) {
  int b = blockIdx.x, j = threadIdx.x;  // 128 threads
  sinusoid(t_dev ? (double)t_dev[b] : (double)t_scalar, j, e[(int64_t)b * 256 + j], e[(int64_t)b * 256 + 128 + j]);
}
hipError_t timestep_sinusoid(const float* t_dev, float t_scalar, float* e, int B, hipStream_t s) {
  if (B > 0) sinusoid_kernel<<<B, 128, 0, s>>>(t_dev, t_scalar, e, B);
  return hipGetLastError();
}

// The start of a step in one launch: workgroups 0..15 write the sinusoid of sample b, split, in the
// MFMA GEMV's input layout ([2][16][256], zeros for b >= B); the others round the latent to bf16, 8
// elements per thread.
__global__ void __launch_bounds__(256) step_prep_kernel(const float* t_dev, float t_scalar, int B, u16* __restrict__ xs,
                                                        const float* __restrict__ latent, u16* __restrict__ lat16,
                                                        int64_t n8) {
  if (blockIdx.x < 16) {
    const int b = blockIdx.x, j = threadIdx.x;
    if (j >= 128) return;
    float c = 0.f, s = 0.f;
    if (b < B) sinusoid(t_dev ? (double)t_dev[b] : (double)t_scalar, j, c, s);
    split_hilo(c, xs[b * 256 + j], xs[(16 + b) * 256 + j]);
    split_hilo(s, xs[b * 256 + 128 + j], xs[(16 + b) * 256 + 128 + j]);
    return;
  }
  const int64_t i = ((int64_t)blockIdx.x - 16) * 256 + threadIdx.x;
  if (i < n8) {
    float f[8];
    Vec8<float>::load(latent + 8 * i, f);
    Vec8<u16>::store(lat16 + 8 * i, f);
  }
}
hipError_t step_prep(const float* t_dev, float t_scalar, int B, u16* xs, const float* latent, u16* lat16, int64_t n,
                     hipStream_t s) {
  step_prep_kernel<<<16 + cdiv(n / 8, 256), 256, 0, s>>>(t_dev, t_scalar, B, xs, latent, lat16, n / 8);
  return hipGetLastError();
}

// tab[pos][i] = (cos, sin)(pos * theta^(-2i/m)), m = head_dim/2, i < m/2, in fp64.
__device__ __forceinline__ void rope_entry(const RopeArgs& r, int idx) {
  int pairs = r.head_dim / 4;
  if (idx >= r.npos * pairs) return;
  int pos = idx / pairs, i = idx % pairs;
  double m = r.head_dim / 2;
  double ang = (double)pos * pow((double)r.theta, -2.0 * i / m);
  r.tab[2 * idx] = (float)cos(ang);
  r.tab[2 * idx + 1] = (float)sin(ang);
}
__global__ void rope_table_kernel(RopeArgs r) { rope_entry(r, blockIdx.x * 256 + threadIdx.x); }
hipError_t rope_table(const RopeArgs& r, hipStream_t s) {
  int n = r.npos * (r.head_dim / 4);
  if (n > 0) rope_table_kernel<<<cdiv(n, 256), 256, 0, s>>>(r);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// LayerNorm + modulate. One 64-lane wave per row; each lane owns CH chunks of
// 8 consecutive elements (16-byte bf16 or 32-byte fp32 accesses), so a row of
// D <= 512*CH stays in registers for the two-pass mean / variance.
// ---------------------------------------------------------------------------
template <typename T, int CH>
__global__ void __launch_bounds__(256) ln_modulate_kernel(LnArgs a) {
  if (a.zero && blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.nzero; i += 256) a.zero[i] = 0;
  int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  int64_t total = a.rows[0] + a.rows[1];
  if (row >= total) return;
  int s = row < a.rows[0] ? 0 : 1;
  int64_t m = s == 0 ? row : row - a.rows[0];
  int64_t b = m / a.xmap[s].rows_per_batch;
  const T* x = (const T*)a.x[s] + row_offset(a.xmap[s], m);
  T* out = (T*)a.out + row_offset(a.omap[s], m);
  const float* shift = a.mod[s] + b * a.mod_bstride + a.shift_off;
  const float* scale = a.mod[s] + b * a.mod_bstride + a.scale_off;
  const int D = a.D;

  float v[CH][8];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < CH; c++) {
    int k = (c * 64 + lane) * 8;
    if (k < D) {
      Vec8<T>::load(x + k, v[c]);
#pragma unroll
      for (int i = 0; i < 8; i++) sum += v[c][i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; i++) v[c][i] = 0.f;
    }
  }
  float mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < CH; c++) {
    int k = (c * 64 + lane) * 8;
    if (k < D) {
#pragma unroll
      for (int i = 0; i < 8; i++) {
        float d = v[c][i] - mean;
        sq += d * d;
      }
    }
  }
  float rstd = rsqrtf(wave_sum(sq) / (float)D + a.eps);
#pragma unroll
  for (int c = 0; c < CH; c++) {
    int k = (c * 64 + lane) * 8;
    if (k < D) {
      float4 sh0 = *(const float4*)(shift + k), sh1 = *(const float4*)(shift + k + 4);
      float4 sc0 = *(const float4*)(scale + k), sc1 = *(const float4*)(scale + k + 4);
      float sh[8] = {sh0.x, sh0.y, sh0.z, sh0.w, sh1.x, sh1.y, sh1.z, sh1.w};
      float sc[8] = {sc0.x, sc0.y, sc0.z, sc0.w, sc1.x, sc1.y, sc1.z, sc1.w};
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; i++) o[i] = fmaf((v[c][i] - mean) * rstd, 1.0f + sc[i], sh[i]);
      Vec8<T>::store(out + k, o);
    }
  }
}

template <typename T>
static hipError_t ln_launch(const LnArgs& a, hipStream_t s) {
  int64_t total = a.rows[0] + a.rows[1];
  if (total == 0) return hipSuccess;
  int grid = cdiv(total, 4);
  int ch = cdiv(a.D, 512);
  if (ch <= 1) ln_modulate_kernel<T, 1><<<grid, 256, 0, s>>>(a);
  else if (ch <= 2) ln_modulate_kernel<T, 2><<<grid, 256, 0, s>>>(a);
  else if (ch <= 4) ln_modulate_kernel<T, 4><<<grid, 256, 0, s>>>(a);
  else if (ch <= 6) ln_modulate_kernel<T, 6><<<grid, 256, 0, s>>>(a);
  else ln_modulate_kernel<T, 8><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t ln_modulate(const LnArgs& a, int dtype, hipStream_t s) {
  return dtype == DT_BF16 ? ln_launch<u16>(a, s) : ln_launch<float>(a, s);
}

// Keeps a packed row packed: the compiler would otherwise carry the fp32 expansion (twice the registers)
// from one pass over the row to the next.
__device__ __forceinline__ void opaque(uint4& u) { asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w)); }

// ---------------------------------------------------------------------------
// TeaCache distance, fused with the LayerNorm + modulate that makes the compared input: a wave takes
// rows of the image stream as in ln_modulate_kernel, rounds h to the storage type, adds |h - h_prev| and
// |h_prev| in fp64 and replaces h_prev, so h itself is never stored. One partial pair per workgroup
// (at most TEACACHE_PARTS; the host, which needs the distance, sums them). Bound by HBM: x and h_prev read, h_prev written.
// ---------------------------------------------------------------------------
template <typename T, int CH>
__global__ void __launch_bounds__(256) teacache_ln_distance_kernel(LnArgs a, T* __restrict__ hp, int measure,
                                                                   double* __restrict__ part) {
  __shared__ double sd[4], sp[4];
  constexpr int Q = sizeof(T) / 2;   // 16-byte registers per chunk of 8 elements
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int D = a.D;
  const int64_t step = (int64_t)gridDim.x * 4;
  double ad = 0.0, ap = 0.0;
  uint4 xr[CH][Q], pr[CH][Q];   // the row as stored; bf16 rows are fetched one row ahead
  auto fetch = [&](int64_t row, uint4 (*x)[Q], uint4 (*p)[Q]) {
    const T* xp = (const T*)a.x[0] + row_offset(a.xmap[0], row);
    const T* hrow = hp + row * D;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int k = (c * 64 + lane) * 8;
#pragma unroll
      for (int q = 0; q < Q; q++) {
        x[c][q] = k < D ? ((const uint4*)(xp + k))[q] : make_uint4(0u, 0u, 0u, 0u);
        p[c][q] = k < D && measure ? ((const uint4*)(hrow + k))[q] : make_uint4(0u, 0u, 0u, 0u);
      }
    }
  };
  auto expand = [](const uint4* u, float* f) {
    if constexpr (Q == 1) {
      const uint32_t w[4] = {u[0].x, u[0].y, u[0].z, u[0].w};
#pragma unroll
      for (int i = 0; i < 4; i++) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 2; q++) {
        f[4 * q] = __uint_as_float(u[q].x);
        f[4 * q + 1] = __uint_as_float(u[q].y);
        f[4 * q + 2] = __uint_as_float(u[q].z);
        f[4 * q + 3] = __uint_as_float(u[q].w);
      }
    }
  };
  int64_t row = (int64_t)blockIdx.x * 4 + wave;
  if (row < a.rows[0]) fetch(row, xr, pr);
  for (; row < a.rows[0]; row += step) {
    const float* mod = a.mod[0] + (row / a.xmap[0].rows_per_batch) * a.mod_bstride;
    T* hrow = hp + row * D;
    uint4 xn[CH][Q], pn[CH][Q];
    if constexpr (Q == 1) fetch(min(row + step, a.rows[0] - 1), xn, pn);
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < CH; c++) {   // (zeros past the row's end)
      float v[8];
      expand(xr[c], v);
#pragma unroll
      for (int i = 0; i < 8; i++) sum += v[i];
    }
    const float mean = wave_sum(sum) / (float)D;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < CH; c++)
      if ((c * 64 + lane) * 8 < D) {
        float v[8];
#pragma unroll
        for (int q = 0; q < Q; q++) opaque(xr[c][q]);
        expand(xr[c], v);
#pragma unroll
        for (int i = 0; i < 8; i++) {
          const float d = v[i] - mean;
          sq += d * d;
        }
      }
    const float rstd = rsqrtf(wave_sum(sq) / (float)D + a.eps);
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int k = (c * 64 + lane) * 8;
      if (k < D) {
        float v[8], p[8], sh[8], sc[8], o[8];
#pragma unroll
        for (int q = 0; q < Q; q++) opaque(xr[c][q]);
        expand(xr[c], v);
        expand(pr[c], p);
        Vec8<float>::load(mod + a.shift_off + k, sh);
        Vec8<float>::load(mod + a.scale_off + k, sc);
#pragma unroll
        for (int i = 0; i < 8; i++) {
          o[i] = to_f32(from_f32<T>(fmaf((v[i] - mean) * rstd, 1.0f + sc[i], sh[i])));
          if (measure) {
            ad += fabs((double)o[i] - (double)p[i]);
            ap += fabs((double)p[i]);
          }
        }
        Vec8<T>::store(hrow + k, o);
        __builtin_amdgcn_sched_barrier(0);   // one chunk's shift and scale at a time in registers
      }
    }
    if constexpr (Q == 1) {
#pragma unroll
      for (int c = 0; c < CH; c++) {
        xr[c][0] = xn[c][0];
        pr[c][0] = pn[c][0];
      }
    } else if (row + step < a.rows[0]) {
      fetch(row + step, xr, pr);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ad += __shfl_xor(ad, o, 64);
    ap += __shfl_xor(ap, o, 64);
  }
  if (lane == 0) {
    sd[wave] = ad;
    sp[wave] = ap;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double d = 0.0, q = 0.0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
      d += sd[w];
      q += sp[w];
    }
    part[2 * blockIdx.x] = d;
    part[2 * blockIdx.x + 1] = q;
  }
}

template <typename T>
static void teacache_ln_launch(const LnArgs& a, T* hp, bool measure, double* partials, int grid, hipStream_t s) {
  const int ch = cdiv(a.D, 512);
  if (ch <= 1) teacache_ln_distance_kernel<T, 1><<<grid, 256, 0, s>>>(a, hp, measure, partials);
  else if (ch <= 2) teacache_ln_distance_kernel<T, 2><<<grid, 256, 0, s>>>(a, hp, measure, partials);
  else if (ch <= 4) teacache_ln_distance_kernel<T, 4><<<grid, 256, 0, s>>>(a, hp, measure, partials);
  else if (ch <= 6) teacache_ln_distance_kernel<T, 6><<<grid, 256, 0, s>>>(a, hp, measure, partials);
  else teacache_ln_distance_kernel<T, 8><<<grid, 256, 0, s>>>(a, hp, measure, partials);
}
int teacache_parts(int64_t rows) { return (int)std::min<int64_t>(TEACACHE_PARTS, cdiv(rows, 4)); }
hipError_t teacache_ln_distance(const LnArgs& a, void* h_prev, bool measure, double* partials, int dtype, hipStream_t s) {
  if (a.rows[0] == 0) return hipSuccess;
  const int grid = teacache_parts(a.rows[0]);
  if (dtype == DT_BF16) teacache_ln_launch<u16>(a, (u16*)h_prev, measure, partials, grid, s);
  else teacache_ln_launch<float>(a, (float*)h_prev, measure, partials, grid, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Velocity head in one pass (bf16): x (+ the TeaCache residual, rounded to bf16 as if stored) ->
// LayerNorm + modulate -> bf16 -> W_out h + b_out, fp32 out. A workgroup takes 16 rows; its 8 waves take
// every 8th 64-deep pair of k steps of them (whole 128-byte lines of a row), so that a lane's share (row
// lane % 16, 8 elements at 8 (lane / 16) of each 32-deep step) is at once the LayerNorm input and, once modulated, operand B of
// v_mfma_f32_16x16x32_bf16: the modulated row never leaves the registers. W_out (64 output features per
// workgroup) is read from L2 straight into operand A. Row sums and the eight partial tiles meet in LDS, in a
// fixed order. Reads x (and the fp32 residual) once from HBM, and W_out from L2 again for every 16 rows: 16384 x 3072 with
// the residual, 302 MB and 403 MB, 103 us (2.9 TB/s of HBM).
// ---------------------------------------------------------------------------
// FULL: every wave has exactly NS steps, no test per step. ONE: no tile crosses samples, so a tile's
// modulation vectors come through LDS once per workgroup (read from L2 by every wave for itself they are
// half of the loads that a CU has to issue).
template <int NS, bool RES, bool FULL, bool ONE>
__global__ void __launch_bounds__(512, 4) final_head_kernel(FinalArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist only in the device pass
  constexpr int NW = 8;
  __shared__ float red[2][NW][16];
  // the partial tiles, and before them the sample's shift and scale (at most 2 x 4096 floats)
  __shared__ union { f32x4 part[NW][4][64]; float mod[2 * 4096]; } sm;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
  const int D = a.D, nks = D / 32;
  const int np = nks / 2, nloc = np > wave ? 2 * ((np - wave + NW - 1) / NW) : 0;   // this wave's k steps
  const int64_t m0 = (int64_t)blockIdx.x * 16, mrow = min(m0 + r16, a.M - 1);
  // step i of this wave starts at element koff(i) of a row; loads go through buffer descriptors with that
  // part of the address in a scalar, since per-access 64-bit pointers would take most of the registers
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  auto koff = [&](int i) { return 64 * wave_s + 64 * NW * (i >> 1) + 32 * (i & 1); };
  auto rsrc = [](const void* p) { return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, 0x7fffffff, 0x00020000); };
  auto load16 = [](__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  };
  auto load_f8 = [&](__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float* f) {
    const f32x4 lo = __builtin_bit_cast(f32x4, load16(r, voff, soff)), hi = __builtin_bit_cast(f32x4, load16(r, voff + 16, soff));
#pragma unroll
    for (int e = 0; e < 4; e++) {
      f[e] = lo[e];
      f[4 + e] = hi[e];
    }
  };
  const uint32_t row = (uint32_t)(mrow - m0);
  const int64_t b0 = m0 / a.rows_per_batch;
  const auto rx = rsrc((const u16*)a.x + m0 * D), rr = rsrc(RES ? a.resid + m0 * D : nullptr), rm = rsrc(a.mod + b0 * 2 * D);
  const uint32_t xo = (row * D + 8 * kq) * 2, ro = (row * D + 8 * kq) * 4;
  const uint32_t mo = (uint32_t)(mrow / a.rows_per_batch - b0) * 8u * D + 32 * kq, wo = (uint32_t)(r16 * D + 8 * kq) * 2;
  uint4 xv[NS];
  float sum = 0.f;
  auto unpack = [](const uint4& u, float* f) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  };
  auto pack = [](const float* f) {
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
  };
#pragma unroll
  for (int i = 0; i < NS; i++) {
    if (FULL || i < nloc) xv[i] = load16(rx, xo, koff(i) * 2);
    else xv[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  if constexpr (ONE)
    for (int q = threadIdx.x; q < D / 2; q += 64 * NW) ((uint4*)sm.mod)[q] = load16(rm, q * 16, 0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (RES) {
#pragma unroll
    for (int i = 0; i < NS; i++)
      if (FULL || i < nloc) {
        float f[8], q[8];
        unpack(xv[i], f);
        load_f8(rr, ro, koff(i) * 4, q);
#pragma unroll
        for (int e = 0; e < 8; e++) f[e] += q[e];
        xv[i] = pack(f);
        if (i % 6 == 5) __builtin_amdgcn_sched_barrier(0);   // six steps' residuals in flight
      }
  }
#pragma unroll
  for (int i = 0; i < NS; i++) {   // (zeros past the wave's steps)
    float f[8];
    opaque(xv[i]);
    unpack(xv[i], f);
#pragma unroll
    for (int e = 0; e < 8; e++) sum += f[e];
    __builtin_amdgcn_sched_barrier(0);
  }
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  if (kq == 0) red[0][wave][r16] = sum;
  __syncthreads();
  auto total = [&](int k) {   // the waves' sums of row r16, in a fixed order
    float t = red[k][0][r16];
#pragma unroll
    for (int w = 1; w < NW; w++) t += red[k][w][r16];
    return t / (float)D;
  };
  const float mean = total(0);
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NS; i++)
    if (FULL || i < nloc) {
      float f[8];
      opaque(xv[i]);
      unpack(xv[i], f);
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const float d = f[e] - mean;
        sq += d * d;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  sq += __shfl_xor(sq, 16, 64);
  sq += __shfl_xor(sq, 32, 64);
  if (kq == 0) red[1][wave][r16] = sq;
  __syncthreads();
  const float rstd = rsqrtf(total(1) + a.eps);
#pragma unroll
  for (int i = 0; i < NS; i++)
    if (FULL || i < nloc) {
      float f[8], sh[8], sc[8];
      opaque(xv[i]);
      unpack(xv[i], f);
      if constexpr (ONE) {
        Vec8<float>::load(sm.mod + koff(i) + 8 * kq, sh);
        Vec8<float>::load(sm.mod + D + koff(i) + 8 * kq, sc);
      } else {
        load_f8(rm, mo, koff(i) * 4, sh);
        load_f8(rm, mo, (D + koff(i)) * 4, sc);
      }
#pragma unroll
      for (int e = 0; e < 8; e++) f[e] = fmaf((f[e] - mean) * rstd, 1.0f + sc[e], sh[e]);
      xv[i] = pack(f);
      if (i & 1) __builtin_amdgcn_sched_barrier(0);   // two steps' shift and scale at a time in registers
    }
  const int c0 = blockIdx.y * 64;
  const auto rw = rsrc((const u16*)a.W + (int64_t)c0 * D);
  f32x4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // W fragments one step ahead
  bf16x8 fw[2][4];
  auto load_w = [&](int i, int slot) {
#pragma unroll
    for (int j = 0; j < 4; j++) fw[slot][j] = __builtin_bit_cast(bf16x8, load16(rw, wo, (16 * j * D + koff(i)) * 2));
  };
  if (FULL || nloc > 0) load_w(0, 0);
#pragma unroll
  for (int i = 0; i < NS; i++)
    if (FULL || i < nloc) {
      if (FULL ? i + 1 < NS : i + 1 < nloc) load_w(i + 1, (i + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; j++)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i & 1][j], __builtin_bit_cast(bf16x8, xv[i]), acc[j], 0, 0, 0);
    }
  __syncthreads();   // every wave is done with the modulation vectors
#pragma unroll
  for (int j = 0; j < 4; j++) sm.part[wave][j][lane] = acc[j];
  __syncthreads();
  if (wave >= 4) return;
  // wave j finishes features c0 + 16 j + 4 kq + 0..3 of row r16
  f32x4 o = sm.part[0][wave][lane];
#pragma unroll
  for (int q = 1; q < NW; q++) {
    const f32x4 p = sm.part[q][wave][lane];
#pragma unroll
    for (int r = 0; r < 4; r++) o[r] += p[r];
  }
  const int n = c0 + 16 * wave + 4 * kq;
  float b[4] = {0.f, 0.f, 0.f, 0.f};
  if (a.bias) {
#pragma unroll
    for (int q = 0; q < 4; q++) b[q] = to_f32(((const u16*)a.bias)[n + q]);
  }
  if ((int64_t)blockIdx.x * 16 + r16 < a.M)
    *(float4*)(a.v + mrow * a.C + n) = make_float4(o[0] + b[0], o[1] + b[1], o[2] + b[2], o[3] + b[3]);
#endif
}

template <int NS, bool RES>
static void final_head_ns(const FinalArgs& a, dim3 grid, hipStream_t s) {
  const bool one = a.rows_per_batch % 16 == 0;
  if constexpr (RES || NS < 8) {   // (rows of 2048 without a residual take two kernels)
    if (a.D == 256 * NS && one) {
      final_head_kernel<NS, RES, true, true><<<grid, 512, 0, s>>>(a);
      return;
    }
  }
  if (one) final_head_kernel<NS, RES, false, true><<<grid, 512, 0, s>>>(a);
  else final_head_kernel<NS, RES, false, false><<<grid, 512, 0, s>>>(a);
}
template <bool RES>
static hipError_t final_head_launch(const FinalArgs& a, hipStream_t s) {
  const dim3 grid(cdiv(a.M, 16), a.C / 64);
  const int ns = 2 * cdiv(a.D, 512);   // k steps of the wave that has most
  if (ns <= 2) final_head_ns<2, RES>(a, grid, s);
  else if (ns <= 4) final_head_ns<4, RES>(a, grid, s);
  else if (ns <= 8) final_head_ns<8, RES>(a, grid, s);
  else if constexpr (!RES) return hipErrorInvalidValue;   // wider rows without a residual take two kernels too
  else if (ns <= 12) final_head_ns<12, RES>(a, grid, s);
  else final_head_ns<16, RES>(a, grid, s);
  return hipGetLastError();
}
// One pass, or LayerNorm + modulate and a GEMM. Every 64 output features have a workgroup of their own, which reads
// x and normalises it again, and W_out is read again for every 16 rows; where tiles span samples (tokens not a
// multiple of 16) each wave reads the modulation from L2. So one pass wins while all of that stays small, and loses
// to the latency of its own chain at widths past 1024 with few workgroups. Measured (us, two kernels / one pass,
// modulation GEMV included): 1024 rows x 512 -> 64 features: 13.0 / 11.3; 8192 x 1024 -> 64: 27.8 / 19.8;
// 16384 x 3072 -> 64: 76.9 / 80.9; 16384 x 1024 -> 64: 34.5 / 31.6, in tiles that span samples 34.9 / 36.5;
// 8192 x 1024 -> 128: 29.7 / 29.7; 2048 x 2048 -> 192: 25.9 / 31.6; 14820 x 1664 -> 1024: 81 / 540. With a residual to
// add, one pass also saves a pass over x and wins at 64 features throughout (16384 x 3072: by 42 us).
bool final_head_in_one_pass(const FinalArgs& a) {
  const int64_t groups = a.C / 64, wgs = cdiv(a.M, 16) * groups;
  if (a.resid && groups == 1) return true;
  if (a.D > 1024 && (a.D > 1792 || wgs < 100)) return false;
  return wgs * groups * a.D * (a.rows_per_batch % 16 ? 1.5 : 1.0) <= 1.2e6;
}
hipError_t final_head(const FinalArgs& a, hipStream_t s) {
  if (a.D % 64 || a.C % 64) return hipErrorInvalidValue;   // whole pairs of k steps, whole feature groups
  if (a.M == 0) return hipSuccess;
  return a.resid ? final_head_launch<true>(a, s) : final_head_launch<false>(a, s);
}

// ---------------------------------------------------------------------------
// batched GEMV: out[s][b][n] = W[s][n][:] . in[b][:] + bias[s][n], B <= 16 per
// pass. A wave owns 4 weight rows and streams them once (16-byte loads), with
// the fp32 input read through L1/L2; lanes split K and reduce at the end.
// ---------------------------------------------------------------------------
// (fp32 weights; act: SiLU on the input as it is read)
template <int BMAX>
__global__ void __launch_bounds__(256) gemv_kernel(GemvArgs a, int b0, int nb, int act) {
  typedef float T;
  constexpr int R = 4;
  int s = blockIdx.y;
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int n0 = (blockIdx.x * 4 + wave) * R;
  if (n0 >= a.N) return;
  const T* W = (const T*)a.W[s];
  float acc[R][BMAX];
#pragma unroll
  for (int r = 0; r < R; r++)
#pragma unroll
    for (int b = 0; b < BMAX; b++) acc[r][b] = 0.f;
  for (int k = lane * 8; k < a.K; k += 512) {
    float w[R][8];
#pragma unroll
    for (int r = 0; r < R; r++) {
      if (n0 + r < a.N) Vec8<T>::load(W + (int64_t)(n0 + r) * a.K + k, w[r]);
      else
#pragma unroll
        for (int i = 0; i < 8; i++) w[r][i] = 0.f;
    }
#pragma unroll
    for (int b = 0; b < BMAX; b++) {
      if (b < nb) {
        float x[8];
        Vec8<float>::load(a.in + (int64_t)(b0 + b) * a.in_bstride + k, x);
        if (act) {
#pragma unroll
          for (int i = 0; i < 8; i++) x[i] = silu(x[i]);
        }
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
          for (int i = 0; i < 8; i++) acc[r][b] = fmaf(w[r][i], x[i], acc[r][b]);
      }
    }
  }
  const T* bias = (const T*)a.bias[s];
#pragma unroll
  for (int r = 0; r < R; r++) {
#pragma unroll
    for (int b = 0; b < BMAX; b++) {
      float v = wave_sum(acc[r][b]);
      if (lane == 0 && b < nb && n0 + r < a.N) {
        if (bias) v += to_f32(bias[n0 + r]);
        a.out[s][(int64_t)(b0 + b) * a.out_bstride + n0 + r] = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 weights: an MFMA skinny GEMM. The fp32 input (at most 16 samples per
// pass) is split once into bf16 hi + lo parts (x = hi + lo to ~2^-16), laid out
// [2][16][K]; each wave then streams 32 weight rows once and multiplies them
// against both parts with v_mfma_f32_16x16x32_bf16 (samples are the MFMA's
// 16-wide N dimension), so HBM bandwidth, not VALU FMAs, sets the time.
// A workgroup owns 32 weight rows and splits K over its 4 waves.
// ---------------------------------------------------------------------------
// Workgroups past the first 16 cdiv(K, 256) fill the RoPE table of a block instead, which saves a launch
// (r.tab null: none).
__global__ void __launch_bounds__(256) split_hilo_kernel(const float* __restrict__ in, int64_t stride, int b0, int nb, int K,
                                                         int act, u16* __restrict__ out, RopeArgs r) {
  const int kb = (K + 255) / 256;
  if ((int)blockIdx.x >= 16 * kb) {
    rope_entry(r, (blockIdx.x - 16 * kb) * 256 + threadIdx.x);
    return;
  }
  const int k = (blockIdx.x % kb) * 256 + threadIdx.x, b = blockIdx.x / kb;
  if (k >= K) return;
  float x = 0.f;
  if (b < nb) {
    x = in[(int64_t)(b0 + b) * stride + k];
    if (act) x = silu(x);
  }
  split_hilo(x, out[(int64_t)b * K + k], out[(int64_t)(16 + b) * K + k]);
}

// Both kernels below are bound by HBM while their weights stream, and next by what a CU takes in besides:
// every 32-deep k step of a wave also reads the split input (2 KB from L2 for 16 samples) against 1 KB of
// weights per 16 rows. Rows past the batch are therefore left out of those loads (ALL = false, their
// lanes zero): for one sample that alone takes 226 MB of weights from 70 to 52 us.

// sums of a wave's accumulators (register r of lane l in block j: weight row n0 + 16 j + 4 (l / 16) + r,
// sample l % 16) plus bias into out and, when asked, SiLU of them into the next GEMV's split input
template <int RB>
__device__ __forceinline__ void gemv_finish(const GemvArgs& a, int s, int n0, f32x4* acc, int b0, int nb) {
  const int lane = threadIdx.x & 63, b = lane & 15;
  const u16* bias = (const u16*)a.bias[s];
  if (b < nb && bias) {
#pragma unroll
    for (int j = 0; j < RB; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) acc[j][r] += to_f32(bias[min(n0 + 16 * j + 4 * (lane >> 4) + r, a.N - 1)]);
  }
  if (a.xs_out) {   // (zeros past the batch)
#pragma unroll
    for (int j = 0; j < RB; j++) {
      const int n = n0 + 16 * j + 4 * (lane >> 4);
      if (n >= a.N) continue;
      u16 h[4], l[4];
#pragma unroll
      for (int r = 0; r < 4; r++) split_hilo(b < nb ? silu(acc[j][r]) : 0.f, h[r], l[r]);
      *(uint2*)(a.xs_out + (int64_t)b * a.N + n) = make_uint2(h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16);
      *(uint2*)(a.xs_out + (int64_t)(16 + b) * a.N + n) = make_uint2(l[0] | (uint32_t)l[1] << 16, l[2] | (uint32_t)l[3] << 16);
    }
  }
  if (b >= nb || !a.out[s]) return;
  float* out = a.out[s] + (int64_t)(b0 + b) * a.out_bstride;
#pragma unroll
  for (int j = 0; j < RB; j++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      int n = n0 + 16 * j + 4 * (lane >> 4) + r;
      if (n < a.N) out[n] = acc[j][r];
    }
}

// The loads of U k steps, step u at element k0 + u * kstep: RB row blocks of weights and the split input.
template <int RB, int U, bool ALL>
struct GemvGroup {
  bf16x8 fw[U][RB], fh[U], fl[U];
  __device__ __forceinline__ void load(const u16* const* w, const u16* xh, const u16* xl, bool on, int k0, int kstep) {
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int j = 0; j < RB; j++) fw[u][j] = *(const bf16x8*)(w[j] + k0 + u * kstep);
    if constexpr (!ALL) {
      const bf16x8 z = {};
#pragma unroll
      for (int u = 0; u < U; u++) fh[u] = fl[u] = z;
    }
    if (ALL || on) {
#pragma unroll
      for (int u = 0; u < U; u++) {
        fh[u] = *(const bf16x8*)(xh + k0 + u * kstep);
        fl[u] = *(const bf16x8*)(xl + k0 + u * kstep);
      }
    }
  }
  __device__ __forceinline__ void mma(f32x4* acc) const {
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int j = 0; j < RB; j++) {
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[u][j], fh[u], acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[u][j], fl[u], acc[j], 0, 0, 0);
      }
  }
};

// One workgroup = 16 RB weight rows (RB row blocks of 16, each the A operand of its own MFMA
// chain); its 4 waves take every 4th 32-deep k step and the partial sums meet in LDS, so each
// row block streams with 4 independent load chains. Small GEMVs (the timestep and final-layer ones, a few
// MB of weights) are bound by the latency of each wave's chain of k steps instead: they take fewer rows
// per workgroup (more workgroups) and, with DEPTH > 0, keep DEPTH of a wave's k steps in flight (the
// loads of step i + DEPTH - 1 are issued before the MFMAs of step i; loads past the wave's last step are
// clamped to that step, so that every load is unconditional and the compiler can count the loads in
// flight). The sums run in the same order either way.
template <int RB, int U, int DEPTH, bool ALL>
__global__ void __launch_bounds__(256) gemv_mfma_kernel(GemvArgs a, const u16* __restrict__ xs, int b0, int nb) {
  __shared__ f32x4 part[4][RB][64];
  const int s = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n0 = blockIdx.x * 16 * RB;
  const int K = a.K, nks = K / 32;
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  const bool on = r16 < nb;
  // operand A: rows n0 + 16 j + r16 (clamped; results of clamped rows are dropped)
  const u16* W = (const u16*)a.W[s];
  const u16* w[RB];
#pragma unroll
  for (int j = 0; j < RB; j++) w[j] = W + (int64_t)min(n0 + 16 * j + r16, a.N - 1) * K + kq;
  // operand B: sample r16, hi and lo parts
  const u16* xh = xs + (int64_t)r16 * K + kq;
  const u16* xl = xs + (int64_t)(16 + r16) * K + kq;
  f32x4 acc[RB];
#pragma unroll
  for (int j = 0; j < RB; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (DEPTH == 0) {
    int ks = wave;
    for (; ks + 4 * (U - 1) < nks; ks += 4 * U) {
      GemvGroup<RB, U, ALL> g;
      g.load(w, xh, xl, on, 32 * ks, 128);
      g.mma(acc);
    }
    for (; ks < nks; ks += 4) {
      GemvGroup<RB, 1, ALL> g;
      g.load(w, xh, xl, on, 32 * ks, 0);
      g.mma(acc);
    }
  } else {
    // this wave's k steps are wave + 4 i, i < nloc; the first nmain of them run pipelined
    const int nloc = nks > wave ? (nks - wave + 3) / 4 : 0;
    const int nmain = nloc - nloc % DEPTH;
    GemvGroup<RB, 1, ALL> g[DEPTH];
    auto load = [&](int i, int slot) { g[slot].load(w, xh, xl, on, 32 * (wave + 4 * i), 0); };
    if (nmain > 0) {
#pragma unroll
      for (int d = 0; d < DEPTH - 1; d++) load(d, d);
      __builtin_amdgcn_sched_barrier(0);
      for (int i = 0; i < nmain; i += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; u++) {
          load(min(i + u + DEPTH - 1, nloc - 1), (u + DEPTH - 1) % DEPTH);
          __builtin_amdgcn_sched_barrier(0);   // keep the loads ahead of this step's MFMAs
          g[u].mma(acc);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    for (int i = nmain; i < nloc; i++) {
      load(i, 0);
      g[0].mma(acc);
    }
  }
#pragma unroll
  for (int j = 0; j < RB; j++) part[wave][j][lane] = acc[j];
  __syncthreads();
  if (wave != 0) return;
  // sum the 4 partials in a fixed order (deterministic)
#pragma unroll
  for (int q = 1; q < 4; q++)
#pragma unroll
    for (int j = 0; j < RB; j++) {
      f32x4 p = part[q][j][lane];
#pragma unroll
      for (int r = 0; r < 4; r++) acc[j][r] += p[r];
    }
  gemv_finish<RB>(a, s, n0, acc, b0, nb);
}

// Many weight matrices at once (a step's batched modulation): a wave takes 16 RB rows over the whole of
// K, the next two k steps loaded ahead, and the four waves of a workgroup walk the same k together, so
// that the split input comes from L2 once for their 64 RB rows and from the CU's cache otherwise. Needs
// many workgroups to fill the chip evenly (K a multiple of 64).
template <int RB, bool ALL>
__global__ void __launch_bounds__(256) gemv_rows_kernel(GemvArgs a, const u16* __restrict__ xs, int b0, int nb) {
  constexpr int U = 2;
  const int s = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n0 = (blockIdx.x * 4 + wave) * 16 * RB, K = a.K, ng = K / (32 * U);
  if (n0 >= a.N) return;
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  const bool on = r16 < nb;
  const u16* w[RB];
#pragma unroll
  for (int j = 0; j < RB; j++) w[j] = (const u16*)a.W[s] + (int64_t)min(n0 + 16 * j + r16, a.N - 1) * K + kq;
  const u16* xh = xs + (int64_t)r16 * K + kq;
  const u16* xl = xs + (int64_t)(16 + r16) * K + kq;
  f32x4 acc[RB];
#pragma unroll
  for (int j = 0; j < RB; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  GemvGroup<RB, U, ALL> g[2];
  auto load = [&](int i, int slot) { g[slot].load(w, xh, xl, on, 32 * U * min(i, ng - 1), 32); };
  load(0, 0);
  for (int i = 0; i < ng; i += 2) {
    load(i + 1, 1);
    __builtin_amdgcn_sched_barrier(0);
    g[0].mma(acc);
    __builtin_amdgcn_sched_barrier(0);
    load(i + 2, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (i + 1 < ng) g[1].mma(acc);
    __builtin_amdgcn_sched_barrier(0);
  }
  gemv_finish<RB>(a, s, n0, acc, b0, nb);
}

template <int RB, int U, int DEPTH>
static void gemv_mfma_launch(const GemvArgs& a, const u16* xs, int b0, int nb, hipStream_t s) {
  const dim3 grid(cdiv(a.N, 16 * RB), a.nstreams);
  if (nb == 16) gemv_mfma_kernel<RB, U, DEPTH, true><<<grid, 256, 0, s>>>(a, xs, b0, nb);
  else gemv_mfma_kernel<RB, U, DEPTH, false><<<grid, 256, 0, s>>>(a, xs, b0, nb);
}

hipError_t gemv_bf16(const GemvArgs& a, u16* xs, int input, const RopeArgs& rope, hipStream_t s) {
  if (a.N == 0 || a.B == 0) return hipSuccess;
  for (int b0 = 0; b0 < a.B; b0 += 16) {
    int nb = std::min(16, a.B - b0);
    if (input != GEMV_SPLIT) {
      RopeArgs r{};
      if (b0 == 0 && rope.tab) r = rope;
      split_hilo_kernel<<<16 * cdiv(a.K, 256) + (r.tab ? cdiv((int64_t)r.npos * (r.head_dim / 4), 256) : 0), 256, 0, s>>>(
          a.in, a.in_bstride, b0, nb, a.K, input == GEMV_SILU, xs, r);
    }
    // By grid size and batch. Measured with cold weights of 18432 x 3072 per slot (us for 2 / 4 / 8 / 12 / 16
    // slots): 64 rows per workgroup 70 / 115 / 220 / 335 / 445 with 16 samples, 64 / 111 / 206 / 315 / 414
    // with 8; 32 rows with four k steps in flight 62 / 113 / 221 / 329 / 435 with 8, 57 / 102 / - / - / 385 with
    // 4, 52 / 91 / 176 / 260 / 345 with 1; whole-K waves 75 / 146 / 222 / 298 / 374 with 16, 58 / 122 / 188 /
    // 252 / 322 with 1. The timestep and final-layer GEMVs (a few MB) need more workgroups and a pipelined
    // k chain (30 -> 18 us for 3072 x 3072).
    const int64_t ns = a.nstreams;
    if ((int64_t)cdiv(a.N, 256) * ns >= 768) {
      const dim3 grid(cdiv(a.N, 256), a.nstreams);
      if (nb == 16) gemv_rows_kernel<4, true><<<grid, 256, 0, s>>>(a, xs, b0, nb);
      else gemv_rows_kernel<4, false><<<grid, 256, 0, s>>>(a, xs, b0, nb);
    } else if ((int64_t)cdiv(a.N, 64) * ns >= 256) {
      if (nb <= 8 && (int64_t)cdiv(a.N, 64) * ns < (nb <= 4 ? 4096 : 1024)) gemv_mfma_launch<2, 4, 0>(a, xs, b0, nb, s);
      else gemv_mfma_launch<4, 2, 0>(a, xs, b0, nb, s);
    } else if ((int64_t)cdiv(a.N, 32) * ns >= 192) {
      gemv_mfma_launch<2, 1, 2>(a, xs, b0, nb, s);
    } else {
      gemv_mfma_launch<1, 1, 4>(a, xs, b0, nb, s);
    }
  }
  return hipGetLastError();
}

// Every wave applies SiLU to the whole input for its 4 rows, 8 values per lane, sample and 512 elements, against
// one more launch. Timestep embedding (us, SiLU apart / folded): 14.7 / 13.2 for 1 sample at hidden 512, 16.9 / 16.3
// for 2 at 768, 19.2 / 18.5 for 4 at 448; 20.9 / 21.8 for 4 at 640, 33.5 / 35.4 for 8 at 1024; with half a wave or
// less at work (hidden 64) 15.9 / 16.3 for 2 (18.3 / 17.2 launched from the host), 17.5 / 18.6 for 3.
bool gemv_f32_folds_silu(const GemvArgs& a) { return (int64_t)a.B * cdiv(a.K, 512) <= (a.K < 128 ? 2 : 4); }
hipError_t gemv_f32(const GemvArgs& a, bool silu_in, hipStream_t s) {
  if (a.N == 0 || a.B == 0) return hipSuccess;
  dim3 grid(cdiv(a.N, 16), a.nstreams);
  for (int b0 = 0; b0 < a.B; b0 += 16) {
    int nb = std::min(16, a.B - b0);
    if (nb <= 4) gemv_kernel<4><<<grid, 256, 0, s>>>(a, b0, nb, silu_in);
    else if (nb <= 8) gemv_kernel<8><<<grid, 256, 0, s>>>(a, b0, nb, silu_in);
    else gemv_kernel<16><<<grid, 256, 0, s>>>(a, b0, nb, silu_in);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// per-group reward statistics. One workgroup per group; rewards of the group in LDS; fp64 sums.
// The order is the stable descending one (ties by index). Up to SORT_MIN seeds it comes from ranks, rank
// of seed i = #{j : r_j > r_i or (r_j == r_i and j < i)}; past that from a bitonic sort in LDS of
// 64-bit keys (value, descending, above the index), which are all different, so the result is as unique.
// ---------------------------------------------------------------------------
__device__ double block_sum_f64(double v, double* red) {
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// whether any of the `count` rewards is not finite, seen by the whole workgroup (NT threads)
template <int NT>
__device__ bool any_bad(const float* __restrict__ rw, int64_t count) {
  __shared__ int any[NT / 64];
  int bad = 0;
  int64_t i = threadIdx.x;
  for (; i + 7 * NT < count; i += 8 * NT) {
    float f[8];
#pragma unroll
    for (int u = 0; u < 8; u++) f[u] = rw[i + u * NT];
#pragma unroll
    for (int u = 0; u < 8; u++) bad |= !isfinite(f[u]);
  }
  for (; i < count; i += NT) bad |= !isfinite(rw[i]);
  bad = __any(bad);
  if ((threadIdx.x & 63) == 0) any[threadIdx.x >> 6] = bad;
  __syncthreads();
  int r = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; w++) r |= any[w];
  return r != 0;
}

// status[0] = 0 when every one of the `count` rewards is finite, else the non-finite code; one
// workgroup strides over the input (the reward matrix is small: groups x seeds)
__global__ void __launch_bounds__(1024) reward_check_kernel(const float* __restrict__ rw, int64_t count,
                                                            int32_t bad_code, int32_t* status) {
  const bool bad = any_bad<1024>(rw, count);
  if (threadIdx.x == 0) status[0] = bad ? bad_code : 0;
}

// Ranks cost n LDS reads per seed, the sort a pass and a barrier per stage: 36 stages at 256 seeds, 45 at 512. One
// group, ranks / sort (us, check and statistics launches): 129 seeds 7.8 / 10.5, 192: 9.3 / 10.5, 256: 10.8 / 10.6,
// 300: 20.2 / 13.4; 512 groups of 192: 14.5 / 16.0, of 300: 28.3 / 21.8.
constexpr int SORT_MIN = 256;

// check_count > 0: this launch also checks all rewards (every workgroup for itself) and workgroup 0
// writes the status; otherwise status, when given, is what the check pass left.
__global__ void __launch_bounds__(256) reward_stats_kernel(const float* rw, int n, float adv_eps, int k, float* mean,
                                                           float* stdv, float* adv, int32_t* order, int32_t* sel,
                                                           int32_t* status, int64_t check_count, int32_t bad_code) {
  extern __shared__ __attribute__((aligned(16))) char rsm[];
  __shared__ double red[4];
  if (check_count > 0) {
    const bool bad = any_bad<256>(rw, check_count);
    if (blockIdx.x == 0 && threadIdx.x == 0) status[0] = bad ? bad_code : 0;
    if (bad) return;                            // non-finite input: nothing else is written
  } else if (status && status[0] != 0) {
    return;
  }
  float* sr = (float*)rsm;                      // n rewards
  int32_t* so = (int32_t*)(rsm + (((size_t)n * 4 + 15) & ~(size_t)15));   // order, or the sort keys
  int g = blockIdx.x;
  const float* r = rw + (int64_t)g * n;
  double part = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    float x = r[i];
    sr[i] = x;
    part += (double)x;
  }
  double mu = block_sum_f64(part, red) / (double)n;   // block_sum syncs after the LDS fill
  part = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    double d = (double)sr[i] - mu;
    part += d * d;
  }
  double sd = sqrt(block_sum_f64(part, red) / (double)n);
  if (threadIdx.x == 0) {
    if (mean) mean[g] = (float)mu;
    if (stdv) stdv[g] = (float)sd;
  }
  if (adv)
    for (int i = threadIdx.x; i < n; i += 256)
      adv[(int64_t)g * n + i] = sd > 0.0 ? (float)(((double)sr[i] - mu) / (sd + (double)adv_eps)) : 0.0f;
  const int top = (k + 1) / 2;
  if (n <= SORT_MIN) {
    for (int i = threadIdx.x; i < n; i += 256) {
      float ri = sr[i];
      int rank = 0;
      for (int j = 0; j < n; j++) {
        float rj = sr[j];
        rank += (rj > ri) || (rj == ri && j < i);
      }
      so[rank] = i;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256)
      if (order) order[(int64_t)g * n + i] = so[i];
    for (int q = threadIdx.x; q < k; q += 256)
      if (sel) sel[(int64_t)g * k + q] = so[q < top ? q : n - k + q];
    return;
  }
  uint64_t* key = (uint64_t*)so;
  int np = 2;
  while (np < n) np *= 2;
  for (int i = threadIdx.x; i < np; i += 256) {
    uint64_t kk = ~(uint64_t)0;                 // padding sorts last
    if (i < n) {
      const uint32_t u = __float_as_uint(sr[i] + 0.0f);            // -0 equals +0
      const uint32_t asc = u & 0x80000000u ? ~u : u | 0x80000000u;   // ascending as the float is
      kk = (uint64_t)~asc << 32 | (uint32_t)i;
    }
    key[i] = kk;
  }
  for (int len = 2; len <= np; len *= 2)
    for (int st = len / 2; st > 0; st /= 2) {
      __syncthreads();
      for (int p = threadIdx.x; p < np / 2; p += 256) {
        const int i = 2 * p - (p & (st - 1)), j = i + st;   // pair p of this stage
        const uint64_t a = key[i], b = key[j];
        if ((a > b) == ((i & len) == 0)) {
          key[i] = b;
          key[j] = a;
        }
      }
    }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 256)
    if (order) order[(int64_t)g * n + i] = (int32_t)(uint32_t)key[i];
  for (int q = threadIdx.x; q < k; q += 256)
    if (sel) sel[(int64_t)g * k + q] = (int32_t)(uint32_t)key[q < top ? q : n - k + q];
}

// do [a, a + na) and [b, b + nb) share a byte
static bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  return a && b && (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

// Whether the statistics launch also checks the rewards, every workgroup all of them, against a second launch (1.4
// us). A look costs a workgroup 5e-5 us per reward, and all of them together 7e-8 us per group and reward from L2:
// 1024 groups of 16, apart / in the launch: 6.9 / 6.7 us; 512 of 32: 6.5 / 6.0; 4096 of 4: 10.5 / 14.7; 8192 of
// 2: 15.8 / 25.0; 256 of 128: 9.4 / 9.7.
bool reward_check_in_launch(int G, int n) {
  const int64_t count = (int64_t)G * n;
  return count <= 16384 && G * count <= (int64_t)1 << 24;
}

hipError_t reward_stats(const float* r, int G, int n, float adv_eps, int k, float* mean, float* stdv, float* adv,
                        int32_t* order, int32_t* sel, int32_t* status, int32_t bad_code, hipStream_t s) {
  if (G == 0) return hipSuccess;
  const int64_t count = (int64_t)G * n;
  const size_t in = (size_t)count * 4;
  // One launch where that is the faster one and no output lies over the rewards, which a workgroup may still be
  // checking while another writes.
  const bool shared = overlap(mean, (size_t)G * 4, r, in) || overlap(stdv, (size_t)G * 4, r, in) || overlap(adv, in, r, in) ||
                      overlap(order, in, r, in) || overlap(sel, (size_t)G * k * 4, r, in) || overlap(status, 4, r, in);
  const bool fused = status && !shared && reward_check_in_launch(G, n);
  if (status && !fused) {
    reward_check_kernel<<<1, 1024, 0, s>>>(r, count, bad_code, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  size_t np = 2;
  while (np < (size_t)n) np *= 2;
  const size_t lds = (((size_t)n * 4 + 15) & ~(size_t)15) + (n <= SORT_MIN ? (size_t)n * 4 : np * 8);
  reward_stats_kernel<<<G, 256, lds, s>>>(r, n, adv_eps, k, mean, stdv, adv, order, sel, status, fused ? count : 0,
                                          bad_code);
  return hipGetLastError();
}

}  // namespace dit
