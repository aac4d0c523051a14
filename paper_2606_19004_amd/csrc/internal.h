// Internal interfaces between the C ABI layer (api.hip) and the gfx950 kernels.
// Nothing here crosses the library boundary.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace dit {

typedef unsigned short u16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// element access: bf16 storage (as u16 bits) or fp32, math always in fp32
// ---------------------------------------------------------------------------
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(u16 x) { return __uint_as_float(((uint32_t)x) << 16); }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ u16 from_f32<u16>(float x) {
  return __builtin_bit_cast(u16, (__bf16)x);  // round to nearest even (v_cvt_pk_bf16_f32)
}

// four consecutive elements as fp32 (16-byte aligned for fp32, 8-byte for bf16), and back
template <typename T> __device__ __forceinline__ void load4(const T* p, float* f);
template <> __device__ __forceinline__ void load4<u16>(const u16* p, float* f) {
  uint2 u = *(const uint2*)p;
  f[0] = __uint_as_float(u.x << 16);
  f[1] = __uint_as_float(u.x & 0xffff0000u);
  f[2] = __uint_as_float(u.y << 16);
  f[3] = __uint_as_float(u.y & 0xffff0000u);
}
template <> __device__ __forceinline__ void load4<float>(const float* p, float* f) {
  float4 a = *(const float4*)p;
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
}
// two fp32 values as packed bf16 (a in the low half), one v_cvt_pk_bf16_f32 (round to nearest even)
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
}
template <typename T> __device__ __forceinline__ void store4(T* p, const float* f);
template <> __device__ __forceinline__ void store4<u16>(u16* p, const float* f) {
  *(uint2*)p = make_uint2(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]));
}
template <> __device__ __forceinline__ void store4<float>(float* p, const float* f) {
  *(float4*)p = make_float4(f[0], f[1], f[2], f[3]);
}

// ---------------------------------------------------------------------------
// row addressing: logical row m of a [rows][cols] operand lives at element
//   (m / rows_per_batch) * batch_stride + (m % rows_per_batch) * row_stride + offset
// which lets one stream's tokens be a strided slice of a joint [B][S][...] buffer.
// ---------------------------------------------------------------------------
struct RowMap {
  int64_t rows_per_batch;
  int64_t batch_stride;
  int64_t row_stride;
  int64_t offset;
};
__host__ __device__ __forceinline__ int64_t row_offset(const RowMap& r, int64_t m) {
  int64_t b = m / r.rows_per_batch;
  return b * r.batch_stride + (m - b * r.rows_per_batch) * r.row_stride + r.offset;
}
inline RowMap contiguous_rows(int64_t cols) { return RowMap{1, cols, 0, 0}; }

__host__ __device__ __forceinline__ int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ---------------------------------------------------------------------------
// GEMM: C[m][n] = epilogue( sum_k A[m][k] W[n][k] + bias[n] ), W stored [N][K]
// ---------------------------------------------------------------------------
// (EPI_STORE_F32: fp32 output of a bf16 problem)
enum Epi { EPI_STORE = 0, EPI_GELU = 1, EPI_RESID = 2, EPI_QKV = 3, EPI_STORE_F32 = 4 };

struct GemmProblem {
  const void* A;  RowMap amap;   // rows of A (K contiguous)
  const void* W;                 // [N][K] contiguous
  const void* bias;              // [N] (weight dtype) or null
  void* C;        RowMap cmap;   // output rows (N contiguous)
  int M, N, K;
  // EPI_RESID: C = C + gate[b][n] * y with b = m / cmap.rows_per_batch
  const float* gate; int64_t gate_bstride;
  // EPI_QKV: 2D RoPE on columns [0, 2*hidden) (q and k) of image rows
  const float* rope_tab;         // [npos][head_dim/4] pairs (cos, sin), null = no RoPE
  int grid_w, head_dim, hidden, rope_npos;
};

struct GemmPair {              // up to two problems (image stream, text stream) in one launch
  GemmProblem p[2];
  int nprob;
};

enum Dtype { DT_F32 = 0, DT_BF16 = 1 };

// Scratch for a bf16 GEMM whose k range is shared out between workgroups (EPI_RESID): room for fp32 partial
// tiles and counters that are zero when the launch starts, 4 per tile. bytes = 0: none.
struct GemmSplitWs {
  float* partials;
  size_t bytes;   // (in the kernel, where tiles are not stored whole: of one part's rows)
  int* counters;
  int max_tiles;
};
constexpr int GEMM_SPLIT_TILES = 128;   // more tiles than this fill the chip without a split
hipError_t gemm(const GemmPair& pr, int epi, int dtype, const GemmSplitWs& split, hipStream_t s);
// how gemm() runs a bf16 pair: the tile, the tile width of a launch of its own for the second problem (0: one
// launch), the number of workgroups that share a tile's K, and the LDS stages of both operands (0: other kernels)
struct GemmPlan {
  int tile_m, tile_n, second_n, splits, ring;
};
GemmPlan gemm_plan(const GemmPair& pr, int epi, const GemmSplitWs& split);

// ---------------------------------------------------------------------------
// attention
// ---------------------------------------------------------------------------
struct AttnArgs {
  const void* q; const void* k; const void* v; void* o;
  int B, H, S, d;
  int64_t qs_b, qs_s, qs_h;
  int64_t os_b, os_s, os_h;
  float scale;
};
hipError_t attention(const AttnArgs& a, int dtype, hipStream_t s);

// ---------------------------------------------------------------------------
// memory-bound kernels
// ---------------------------------------------------------------------------
// LayerNorm (no affine) + modulate over the rows of up to two streams.
// out = LN(x)(1 + scale[b]) + shift[b]; shift at mod[s] + b*mod_bstride + shift_off.
struct LnArgs {
  const void* x[2]; RowMap xmap[2];
  void* out;        RowMap omap[2];
  const float* mod[2]; int64_t mod_bstride; int shift_off, scale_off;
  int64_t rows[2];     // rows per stream (B * N_s)
  int D; float eps;
  int* zero; int nzero;   // ints cleared by the way (counters of a later GEMM), or null
};
hipError_t ln_modulate(const LnArgs& a, int dtype, hipStream_t s);

// out[s][b][n] = sum_k W[s][n][k] in[b][k] + bias[s][n]  (fp32 in/out, W in weight dtype)
// up to GEMV_SLOTS independent weight matrices (same N, K, input) in one launch: the two streams of a
// block, or the modulation of several blocks at once
constexpr int GEMV_SLOTS = 16;
struct GemvArgs {
  const void* W[GEMV_SLOTS]; const void* bias[GEMV_SLOTS]; float* out[GEMV_SLOTS];
  int64_t out_bstride;
  const float* in; int64_t in_bstride;
  int N, K, B, nstreams;
  u16* xs_out;   // bf16, B <= 16, one slot: also write SiLU(out) as the next GEMV's split input (or null)
};
// RoPE (cos, sin) table: tab[pos][i], pos < npos, i < head_dim / 4
struct RopeArgs {
  float* tab;
  int npos, head_dim;
  float theta;
};
hipError_t gemv_f32(const GemvArgs& a, bool silu_in, hipStream_t s);   // VALU, fp32 weights; SiLU(in) when silu_in
bool gemv_f32_folds_silu(const GemvArgs& a);   // whether silu_in beats a silu_f32 pass of its own
hipError_t silu_f32(const float* in, float* out, int64_t n, hipStream_t s);
// bf16 weights through MFMA on the input's two bf16 parts, xs [2][16][K], which are made here from a.in
// (GEMV_RAW) or SiLU(a.in) (GEMV_SILU), or are there already (GEMV_SPLIT, B <= 16). The launch that makes
// them also fills rope (tab null: none). K must be a multiple of 32
enum GemvInput { GEMV_RAW = 0, GEMV_SILU = 1, GEMV_SPLIT = 2 };
hipError_t gemv_bf16(const GemvArgs& a, u16* xs, int input, const RopeArgs& rope, hipStream_t s);
// xs [2][16][256] = the split timestep sinusoid of t_dev[b] (or t_scalar), b < B <= 16, and lat16 = bf16
// of n latent elements (n a multiple of 8, 16-byte aligned; may be 0), in one launch
hipError_t step_prep(const float* t_dev, float t_scalar, int B, u16* xs, const float* latent, u16* lat16, int64_t n,
                     hipStream_t s);

hipError_t cast_f32_to_bf16(const float* in, u16* out, int64_t n, hipStream_t s);
hipError_t timestep_sinusoid(const float* t_dev, float t_scalar, float* e, int B, hipStream_t s);
hipError_t rope_table(const RopeArgs& r, hipStream_t s);
// per-sample Gaussian log-density of an SDE step: logp[b] = -sum (xn - mean)^2 * inv2var + cst,
// mean = x + h (v + k1 (x + omt v))
hipError_t flow_logprob_launch(const float* x, const float* v, const float* xn, int batch, int64_t n, double h,
                               double k1, double omt, double inv2var, double cst, double* logp, hipStream_t s);
// TeaCache: h = LN(x)(1 + scale) + shift over the image rows (stream 0 of a), rounded to dtype and
// compared with h_prev ([rows][D]): partials[2 p], [2 p + 1] = sum |h - h_prev|, sum |h_prev| over part p of
// teacache_parts(rows) (zeros when !measure); h_prev is then overwritten with h.
int teacache_parts(int64_t rows);
hipError_t teacache_ln_distance(const LnArgs& a, void* h_prev, bool measure, double* partials, int dtype, hipStream_t s);
// velocity head, bf16: v[m][c] = sum_k W[c][k] h[m][k] + bias[c], h = LN(x + resid)(1 + scale) + shift with
// (shift, scale) = mod[b][0..D), mod[b][D..2D), b = m / rows_per_batch; resid (fp32) may be null. D a
// multiple of 64 and at most 4096, C a multiple of 64.
struct FinalArgs {
  const void* x; const float* resid; const float* mod; const void* W; const void* bias; float* v;
  int64_t M, rows_per_batch;
  int D, C;
  float eps;
};
hipError_t final_head(const FinalArgs& a, hipStream_t s);
bool final_head_in_one_pass(const FinalArgs& a);   // whether it beats LayerNorm + modulate and a GEMM
// residual r (fp32) of the activation x (n elements): mode 0 r = x, 1 r = x - r, 2 x = x + r
hipError_t teacache_residual(void* x, float* r, int64_t n, int mode, int dtype, hipStream_t s);
constexpr int TEACACHE_PARTS = 512;
hipError_t flow_update(float* x, const float* v, const float* noise, int64_t n,
                       float cx, float cv, float ce, hipStream_t s);
// status (device, nullable): 0 or bad_code (any reward non-finite) is written there, by a check pass or by the
// statistics kernel itself (reward_check_in_launch), which writes nothing else when it is non-zero
bool reward_check_in_launch(int G, int n);
hipError_t reward_stats(const float* r, int G, int n, float adv_eps, int k,
                        float* mean, float* stdv, float* adv, int32_t* order, int32_t* sel,
                        int32_t* status, int32_t bad_code, hipStream_t s);

}  // namespace dit
