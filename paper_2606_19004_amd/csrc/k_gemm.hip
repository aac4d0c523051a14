// GEMMs of the MMDiT block on gfx950: C = epilogue(A W^T + bias), W stored [N][K].
//
// bf16 path: LDS-staged MFMA kernel with fp32 accumulation.
//   * Computed as C^T = W A^T: MFMA operand "A" = rows of W, operand "B" = rows
//     of A; both are K-contiguous, so every lane reads one 16-byte chunk per
//     fragment (ds_read_b128). The accumulator gives each lane one token row m
//     and runs of 4 consecutive output features n, which is what the epilogues
//     need (RoPE pairs (2i, 2i+1) sit in one lane).
//   * Tiles of A and W move HBM -> LDS with buffer_load ... lds (no VGPR
//     staging). Out-of-range rows use an offset past the buffer's num_records,
//     which the hardware turns into zeros. In the large tile a wave's refill of
//     one operand is a single burst of up to four such loads under one M0 value
//     (the instruction offset steps the LDS destination by 1 KB): a load issued
//     between MFMAs holds the wave's issue for ~17 cycles, and the M0 save and
//     restore around each load for ~13 more, while back-to-back loads share it.
//   * LDS rows are 64 bf16 = 8 chunks of 16 bytes; chunk c of row r is stored
//     at slot c ^ ((r >> 1) & 7), so every lane group that a ds_read_b128 of a
//     fragment is served in hits 16 different bank groups of the 64-bank LDS.
//   * The large tile (256 x 256 x 64, v_mfma_f32_16x16x32_bf16) runs 8 waves
//     (2 per SIMD), each 64 rows x 128 features, and keeps three LDS stages of
//     A and two of W (160 KB), so the activation rows are requested two k-tiles
//     before use. Fragments of the next 32-deep k step load while the current
//     step's MFMAs run; the k-tile barrier sits at the last step, whose
//     fragments are already in registers. The refill is split between the two
//     steps of a k-tile (W after the barrier, A in the other step), and each
//     wave lowers its issue priority as it advances between barriers, so the
//     two waves of a SIMD share the matrix pipe instead of one running ahead
//     and idling at the barrier. Smaller problems use 128 x 128 tiles with
//     a ring of five stages, or 64 x 64 and 32 x 32 tiles whose waves split K
//     (pick_tile below).
//   * Epilogue: bias, gate vectors and the RoPE table are staged in LDS per
//     tile; the gated residual reads of a wave's whole sub-tile are issued at
//     once.
//   * Workgroups are dispatched round-robin over the 8 XCDs; tile t is given
//     to workgroup ids so that each XCD owns one contiguous range of tiles,
//     ordered in groups of 8 M-tiles so concurrently running tiles share A and
//     W panels in that XCD's L2.
// fp32 path: fp32 MFMA tiles (64 x 64, or 32 x 32 with K split over the waves) with the same epilogue.
#include <atomic>
#include <type_traits>

#include "internal.h"

namespace dit {

// ---------------------------------------------------------------------------
// epilogue on 4 consecutive output features n..n+3 of row m
// ---------------------------------------------------------------------------
__device__ __forceinline__ float gelu_tanh_f(float z) {
  // 0.5 z (1 + tanh(u)) = z * sigmoid(2u), u = sqrt(2/pi) (z + 0.044715 z^3), and
  // sigmoid(2u) = 1 / (1 + 2^(-2u log2 e)) with -2u log2 e = z (K1 + K2 z^2)
  constexpr float K1 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
  constexpr float K2 = K1 * 0.044715f;
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z * fmaf(K2, z * z, K1)));
}


// Per-row epilogue state, computed once per output row m.
struct RowEpi {
  int64_t off;   // element offset of row m in C
  int64_t gate;  // element offset of the row's gate vector (EPI_RESID)
  int rpos, cpos;  // grid row / column of an image token (EPI_QKV with RoPE)
};

__device__ __forceinline__ RowEpi row_epi(const GemmProblem& P, int m) {
  RowEpi r;
  int rpb = (int)P.cmap.rows_per_batch;
  int b = m / rpb, i = m - b * rpb;
  r.off = (int64_t)b * P.cmap.batch_stride + (int64_t)i * P.cmap.row_stride + P.cmap.offset;
  r.gate = (int64_t)b * P.gate_bstride;
  r.rpos = P.grid_w > 0 ? i / P.grid_w : 0;
  r.cpos = P.grid_w > 0 ? i - r.rpos * P.grid_w : 0;
  return r;
}

template <int EPI, typename TW, typename TC>
__device__ __forceinline__ void epilogue4(const GemmProblem& P, const RowEpi& R, int n, float* v) {
  if (P.bias) {
    float b[4];
    const TW* bias = (const TW*)P.bias + n;
    // the biases outside a block are accepted at any element alignment
    if (sizeof(TW) == 4 || ((uintptr_t)P.bias & 7) == 0) {
      load4<TW>(bias, b);
    } else {
#pragma unroll
      for (int q = 0; q < 4; q++) b[q] = to_f32(bias[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; q++) v[q] += b[q];
  }
  if (EPI == EPI_GELU) {
#pragma unroll
    for (int q = 0; q < 4; q++) v[q] = gelu_tanh_f(v[q]);
  }
  TC* out = (TC*)P.C + R.off + n;
  if (EPI == EPI_RESID) {
    float4 g = *(const float4*)(P.gate + R.gate + n);
    float x[4];
    load4<TC>(out, x);
    v[0] = fmaf(g.x, v[0], x[0]);
    v[1] = fmaf(g.y, v[1], x[1]);
    v[2] = fmaf(g.z, v[2], x[2]);
    v[3] = fmaf(g.w, v[3], x[3]);
  }
  if (EPI == EPI_QKV) {
    if (P.rope_tab && n < 2 * P.hidden) {
      // head dims [0, d/2) rotate by the token's grid row, [d/2, d) by its column;
      // n..n+3 hold the pairs (pr, pr+1) of one half (head_dim is a power of two)
      int dd = n & (P.head_dim - 1);
      int hh = P.head_dim >> 1;
      int pos = dd < hh ? R.rpos : R.cpos;
      int pr = (dd & (hh - 1)) >> 1;
      float4 t = *(const float4*)(P.rope_tab + ((int64_t)pos * (P.head_dim >> 2) + pr) * 2);
      float a0 = v[0], b0 = v[1], a1 = v[2], b1 = v[3];
      v[0] = a0 * t.x - b0 * t.y;
      v[1] = a0 * t.y + b0 * t.x;
      v[2] = a1 * t.z - b1 * t.w;
      v[3] = a1 * t.w + b1 * t.z;
    }
  }
  store4<TC>(out, v);
}

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

// Direct-to-LDS 16-byte-per-lane buffer load (M0 = LDS destination of lane 0), written as inline
// assembly so that the compiler does not track it: with LDS addresses chosen at run time it cannot
// prove that a later LDS read does not alias the load, and would wait for all loads in flight. The
// caller's explicit s_waitcnt vmcnt is the only synchronisation for these loads. M0 is reserved by
// the compiler, so the sequence saves it in a scratch SGPR and restores it after issuing the load
// (the destination is taken from M0 when the load issues). rsrc is a raw buffer descriptor (base,
// stride 0, num_records, flags).
__device__ __forceinline__ void dma_b128(u32x4_t rsrc, uint32_t m0v, uint32_t voff, uint32_t soff) {
  uint32_t saved;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(saved) : "s"(m0v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// N (3 or 4) direct-to-LDS loads sharing one M0: destination M0 + 1024 i + 16 lane, global offset
// v[i] + 1024 i (the instruction offset moves both addresses)
template <int N>
__device__ __forceinline__ void dma_burst(u32x4_t rsrc, uint32_t m0v, const uint32_t* v, uint32_t soff) {
  uint32_t saved;
  if constexpr (N == 4)
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %2, %6, %7 offen lds\n\t"
                 "buffer_load_dwordx4 %3, %6, %7 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %4, %6, %7 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %5, %6, %7 offen offset:3072 lds\n\t"
                 "s_mov_b32 m0, %0"
                 : "=&s"(saved) : "s"(m0v), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(rsrc), "s"(soff) : "memory");
  else
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %2, %5, %6 offen lds\n\t"
                 "buffer_load_dwordx4 %3, %5, %6 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %4, %5, %6 offen offset:2048 lds\n\t"
                 "s_mov_b32 m0, %0"
                 : "=&s"(saved) : "s"(m0v), "v"(v[0]), "v"(v[1]), "v"(v[2]), "s"(rsrc), "s"(soff) : "memory");
}

// Exchange lanes 16-31 of x with lanes 0-15 of y and lanes 48-63 of x with lanes 32-47 of y.
__device__ __forceinline__ void swap16(uint32_t& x, uint32_t& y) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
  x = r[0];
  y = r[1];
}

__device__ __forceinline__ void tile_coords(int tl, int mt, int nt, int& tm, int& tn) {
  constexpr int GROUP_M = 8;
  int per_group = GROUP_M * nt;
  int group = tl / per_group;
  int first_m = group * GROUP_M;
  int gm = min(mt - first_m, GROUP_M);
  int in_group = tl - group * per_group;
  tm = first_m + in_group % gm;
  tn = in_group / gm;
}

// LDS swizzle key of tile row r (rows of 128 bytes = 64 bf16 of k): chunk c of row r lives in
// 16-byte slot c ^ f(r). Measured service rule of ds_read_b128 on this chip: the 64 lanes are
// served as four groups of 16, a group being the lanes that agree in lane bit 5 and in the
// parity of lane bits 2..4; a group takes as many cycles as the largest number of its lanes
// that hit one 16-byte bank group ((address / 16) mod 16) at different addresses. With
// f(r) = (r / 2) mod 8 every group of a 16x16x32 or a 32x32x16 fragment read hits 16 distinct
// bank groups, so a wave's read takes the minimum four cycles.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Instructions of one kind placed after MFMA q when n of them are spread evenly over the first
// `span` MFMAs of a k step.
__host__ __device__ constexpr int spread(int q, int n, int span) {
  return span <= 0 ? (q == 0 ? n : 0) : ((q + 1 < span ? q + 1 : span) * n) / span - ((q < span ? q : span) * n) / span;
}

// Scheduling hints for one k step of NM MFMAs: NV direct-to-LDS loads spread over the first half
// of the MFMAs, ND fragment reads over the first three quarters.
template <int NM, int NV, int ND, int Q = 0>
__device__ __forceinline__ void sched_step() {
  if constexpr (Q < NM) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
    constexpr int v = spread(Q, NV, NM / 2), d = spread(Q, ND, 3 * NM / 4);
    if constexpr (v > 0) __builtin_amdgcn_sched_group_barrier(0x020, v, 0);   // VMEM loads
    if constexpr (d > 0) __builtin_amdgcn_sched_group_barrier(0x100, d, 0);   // LDS reads
    sched_step<NM, NV, ND, Q + 1>();
  }
}

// One MFMA on a 16 x 16 block, 32 deep: one 8-element bf16 fragment per lane for each operand.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The 16x16x32 MFMA form delivers more throughput per watt than 32x32x16 under sustained load with
// random operands on this chip.
// RING = 0 (256-row tiles): three LDS stages for A and two for W (160 KB), so the activation
// operand is loaded two k-tiles ahead. RING > 0 (128 x 128 and, for short K, 64 x 64 tiles): a ring of RING
// LDS stages of both operands.
// SPLIT (EPI_RESID): `splits` workgroups (2 or 3) share a tile, each over its part of K. All but the last one
// to finish leave their accumulators in `split.partials`; the last adds them in the order of the parts
// (so the result does not depend on which was last) and runs the epilogue. It waits only for workgroups
// that have taken their ticket, that is, are storing, and wait for nothing themselves.
template <int BM, int BN, int WM, int WN, int EPI, int RING = 0, bool SPLIT = false, bool DENSE = false>
__global__ void __launch_bounds__(WM * WN * 64) gemm_bf16_kernel(GemmPair pr, int tiles0, int total_tiles, int splits,
                                                                 GemmSplitWs split) {
  constexpr int MS = 16, KS = 32;                      // MFMA block and k depth
  constexpr bool TRI = RING == 0;
  constexpr int NW = WM * WN;
  constexpr int BK = 64;
  constexpr int WTM = BM / WM, WTN = BN / WN;          // wave tile (m, n)
  constexpr int TJ = WTM / MS, TI = WTN / MS;          // MFMA blocks per wave along m and n
  constexpr int A_LOADS = BM / 8 / NW, W_LOADS = BN / 8 / NW;  // 8-row groups each wave loads per k-tile
  constexpr int A_BYTES = BM * BK * 2, W_BYTES = BN * BK * 2;
  static_assert(A_LOADS >= 1 && W_LOADS >= 1, "every wave loads at least one row group");
  static_assert(!TRI || (BM == 256 && (BN == 256 || BN == 192)), "three A stages only for 256-row tiles");
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist only in the device pass
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  // XCD-aware tile index
  int per = gridDim.x >> 3;
  int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (t >= (SPLIT ? total_tiles * splits : total_tiles)) return;
  // parts are the slow index: an XCD's workgroups then share the panels of one part of K
  const int part = SPLIT ? t / total_tiles : 0;
  if constexpr (SPLIT) t -= part * total_tiles;
  int pi = t < tiles0 ? 0 : 1;
  const GemmProblem P = pr.p[pi];   // a copy: its fields stay in registers instead of being reloaded per use
  int tl = pi == 0 ? t : t - tiles0;
  int mt = cdiv(P.M, BM), nt = cdiv(P.N, BN);
  int tm, tn;
  tile_coords(tl, mt, nt, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int K = P.K;

  // buffer resources; rows outside the matrix get an offset beyond num_records -> zeros
  const uint32_t OOB = 0x80000000u;
  // a wave-load writes 8 rows x 8 slots (lane -> row lane/8, slot lane%8) and fetches chunk slot ^ f(row)
  const int lrow = lane >> 3;
  uint32_t aoff[A_LOADS], woff[W_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; i++) {
    int g = wave * A_LOADS + i;
    int chunk = (lane & 7) ^ swz(8 * g + lrow);
    int m = m0 + 8 * g + lrow;
    aoff[i] = m < P.M ? (uint32_t)(row_offset(P.amap, m) * 2 + chunk * 16) : OOB;
  }
#pragma unroll
  for (int i = 0; i < W_LOADS; i++) {
    int g = wave * W_LOADS + i;
    int chunk = (lane & 7) ^ swz(8 * g + lrow);
    int n = n0 + 8 * g + lrow;
    woff[i] = n < P.N ? (uint32_t)((int64_t)n * K * 2 + chunk * 16) : OOB;
  }
  // RING = 0: [W0][W1][A0][A1][A2], tile kt uses W stage kt % 2 and A stage kt % 3; else tile kt uses
  // stage kt % RING of [W][A] pairs
  auto stage_w = [&](int kt) -> char* { return smem + (TRI ? (kt & 1) * W_BYTES : (kt % (RING + TRI)) * (A_BYTES + W_BYTES)); };
  auto stage_a = [&](int kt) -> char* {
    return smem + (TRI ? 2 * W_BYTES + (kt % 3) * A_BYTES : (kt % (RING + TRI)) * (A_BYTES + W_BYTES) + W_BYTES);
  };
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int kt_all = K / BK, kt0 = SPLIT ? part * kt_all / splits : 0;   // this workgroup's k-tiles start at kt0
  const uint64_t pa64 = (uint64_t)P.A + (SPLIT ? kt0 * BK * 2 : 0), pw64 = (uint64_t)P.W + (SPLIT ? kt0 * BK * 2 : 0);
  // refills as one burst per operand: offsets carry -1024 i plus a 4 KB bias taken back from the base
  constexpr bool BA = TRI && (A_LOADS == 3 || A_LOADS == 4), BW = TRI && (W_LOADS == 3 || W_LOADS == 4);
  const uint64_t pa64b = pa64 - (BA ? 4096u : 0u), pw64b = pw64 - (BW ? 4096u : 0u);
  // (with the bias every in-range offset stays below 2^31 + 4 KB, the records bound; rows outside the
  // matrix move to 3 GiB, past it, and still read zeros)
  const u32x4_t ra4 = {(uint32_t)pa64b, (uint32_t)(pa64b >> 32) & 0xffffu, BA ? 0x80001000u : 0x7fffffffu, 0x00020000u};
  const u32x4_t rw4 = {(uint32_t)pw64b, (uint32_t)(pw64b >> 32) & 0xffffu, BW ? 0x80001000u : 0x7fffffffu, 0x00020000u};
  uint32_t aoffb[A_LOADS], woffb[W_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; i++) aoffb[i] = BA ? (aoff[i] == OOB ? 0xC0000000u : aoff[i]) + 4096u - 1024u * i : aoff[i];
#pragma unroll
  for (int i = 0; i < W_LOADS; i++) woffb[i] = BW ? (woff[i] == OOB ? 0xC0000000u : woff[i]) + 4096u - 1024u * i : woff[i];
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  auto issue_a = [&](int kt) {
    const uint32_t sa = smem_lds + (uint32_t)(stage_a(kt) - smem);
    const uint32_t soff = kt * BK * 2;
#pragma unroll
    for (int i = 0; i < (BA ? 0 : A_LOADS); i++) dma_b128(ra4, sa + (wave_s * A_LOADS + i) * 1024, aoffb[i], soff);
    if constexpr (BA) dma_burst<A_LOADS>(ra4, sa + wave_s * A_LOADS * 1024, aoffb, soff);
  };
  auto issue_w = [&](int kt) {
    const uint32_t sw = smem_lds + (uint32_t)(stage_w(kt) - smem);
    const uint32_t soff = kt * BK * 2;
#pragma unroll
    for (int i = 0; i < (BW ? 0 : W_LOADS); i++) dma_b128(rw4, sw + (wave_s * W_LOADS + i) * 1024, woffb[i], soff);
    if constexpr (BW) dma_burst<W_LOADS>(rw4, sw + wave_s * W_LOADS * 1024, woffb, soff);
  };
  f32x4 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; i++)
#pragma unroll
    for (int j = 0; j < TJ; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int wm = wave / WN, wn = wave % WN;
  // lane -> (fragment row inside an MS-row block, 8-element k chunk inside a KS step)
  const int frow = lane % MS, lkc = lane / MS;
  const int nk = SPLIT ? (part + 1) * kt_all / splits - kt0 : kt_all;
  int fwk[TI], fak[TJ];
#pragma unroll
  for (int i = 0; i < TI; i++) fwk[i] = swz(wn * WTN + MS * i + frow);
#pragma unroll
  for (int j = 0; j < TJ; j++) fak[j] = swz(wm * WTM + MS * j + frow);
  const int wrow0 = (wn * WTN + frow) * 128, arow0 = (wm * WTM + frow) * 128;
  // fragments of k step s, register-double-buffered so step s+1 loads while step s multiplies
  bf16x8 fw[2][TI], fa[2][TJ];
  auto frags = [&](int kt, int s, int rb) {
    const char* sa = stage_a(kt);
    const char* sw = stage_w(kt);
    const int c = (KS / 8) * s + lkc;
#pragma unroll
    for (int i = 0; i < TI; i++) fw[rb][i] = *(const bf16x8*)(sw + wrow0 + MS * i * 128 + ((c ^ fwk[i]) << 4));
#pragma unroll
    for (int j = 0; j < TJ; j++) fa[rb][j] = *(const bf16x8*)(sa + arow0 + MS * j * 128 + ((c ^ fak[j]) << 4));
  };

  // The reads and loads of a k step are spread over its MFMAs: loads over the first half, fragment
  // reads over the first three quarters, leaving the tail of the step to cover their latency.
  constexpr int NM = TI * TJ;
  // Epilogue inputs (bias, gate vectors, RoPE table) are requested into registers before the last
  // k-tile, so their memory latency is covered by its MFMAs; after the loop they are written to LDS.
  // Tiles whose inputs exceed the register budget (more than one gate row per thread or four table
  // entries per thread) load them after the loop instead.
  constexpr int NT = NW * 64;
  constexpr int LDS_BYTES = TRI ? 2 * (A_BYTES + W_BYTES) : RING * (A_BYTES + W_BYTES);
  const int rpb = (int)P.cmap.rows_per_batch;
  const int bfirst = m0 / rpb;
  const int nbt = (min(m0 + BM, P.M) - 1) / rpb - bfirst + 1;
  const bool gate_lds = EPI == EPI_RESID && (size_t)(BN + nbt * BN) * 4 <= (size_t)LDS_BYTES;
  const int rope_n = (EPI == EPI_QKV && P.rope_tab) ? P.rope_npos * (P.head_dim >> 1) : 0;
  const bool rope_lds = rope_n > 0 && (size_t)(BN + rope_n) * 4 <= (size_t)LDS_BYTES;
  const bool pre = (!gate_lds || nbt * BN <= NT) && (!rope_lds || rope_n <= 4 * NT);
  // branch-free buffer loads: a lane with nothing to fetch uses an offset past num_records and reads 0
  u16 pre_b = 0;
  float pre_g = 0.f, pre_r[4] = {0.f, 0.f, 0.f, 0.f};
  auto prefetch_epi = [&]() {
    if (!pre) return;
    const uint32_t OOB = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        P.bias ? (void*)P.bias : (void*)P.W, (short)0, P.bias ? P.N * 2 : 0, 0x00020000);
    pre_b = __builtin_amdgcn_raw_buffer_load_b16(rb, tid < BN ? (uint32_t)(n0 + tid) * 2u : OOB, 0, 0);
    if (gate_lds) {
      const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void*)P.gate, (short)0, 0x7fffffff, 0x00020000);
      const int bb = tid / BN, nn = tid - bb * BN;
      const bool ok = bb < nbt && n0 + nn < P.N;
      pre_g = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
          rg, ok ? (uint32_t)(((int64_t)(bfirst + bb) * P.gate_bstride + n0 + nn) * 4) : OOB, 0, 0));
    }
    if (rope_lds) {
      const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)P.rope_tab, (short)0, rope_n * 4, 0x00020000);
#pragma unroll
      for (int r = 0; r < 4; r++)
        pre_r[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rr, (uint32_t)(tid + r * NT) * 4u, 0, 0));
    }
  };

  if constexpr (TRI) {
    // k-tile kt. First step: refill A stage (kt+2) % 3 with tile kt+2 (that stage last held tile
    // kt-1, whose reads ended before the previous barrier). Last step: wait for tile kt+1 (the A
    // loads of tile kt+2, issued last, may still be in flight: vmcnt(A_LOADS)), barrier, then
    // refill W stage kt % 2 with tile kt+2 and read tile kt+1's first fragments.
    // Issue priority between two barriers runs 3, 2 (halves of the last step), 1, 0 (halves of
    // the next tile's first step): a wave that has run ahead yields the matrix pipe to the other
    // wave of its SIMD, so both reach the barrier together.
    auto ktile3 = [&](int kt, auto ph_c) {
      constexpr int PH = decltype(ph_c)::value;   // 0, 1: refill tile kt+2; 2: none; 3: last tile
#pragma unroll
      for (int s = 0; s < BK / KS; s++) {
        const int rb = s & 1;
        const bool seam = s == BK / KS - 1;
        if (!seam) {
          __builtin_amdgcn_s_setprio(1);
          frags(kt, s + 1, rb ^ 1);
          if (PH <= 1) issue_a(kt + 2);
        } else if (PH < 3) {
          if (PH < 2) __builtin_amdgcn_s_waitcnt(0x0070 | A_LOADS);   // vmcnt(A_LOADS) lgkmcnt(0)
          else __builtin_amdgcn_s_waitcnt(0);
          __syncthreads();
          __builtin_amdgcn_s_setprio(3);
          if (PH <= 1) issue_w(kt + 2);
          frags(kt + 1, 0, rb ^ 1);
        }
        // the step's MFMAs in two halves; the priority drops between them (a scheduling boundary,
        // so the step's reads and loads are placed among the first half's MFMAs)
#pragma unroll
        for (int i = 0; i < TI / 2; i++)
#pragma unroll
          for (int j = 0; j < TJ; j++)
            acc[i][j] = mfma16(fw[rb][i], fa[rb][j], acc[i][j]);
        if (!seam) sched_step<NM / 2, PH <= 1 ? A_LOADS : 0, TI + TJ>();
        else sched_step<NM / 2, PH <= 1 ? W_LOADS : 0, PH < 3 ? TI + TJ : 0>();
        if (seam) __builtin_amdgcn_s_setprio(2);
        else __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int i = TI / 2; i < TI; i++)
#pragma unroll
          for (int j = 0; j < TJ; j++)
            acc[i][j] = mfma16(fw[rb][i], fa[rb][j], acc[i][j]);
      }
    };
    issue_a(0);
    issue_w(0);
    if (nk > 1) issue_a(1);
    if (nk > 1) __builtin_amdgcn_s_waitcnt(0x0070 | A_LOADS);
    else __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (nk > 1) issue_w(1);
    frags(0, 0, 0);
    for (int kt = 0; kt + 3 < nk; kt++) ktile3(kt, std::integral_constant<int, 0>());
    if (nk >= 3) ktile3(nk - 3, std::integral_constant<int, 1>());
    if (nk >= 2) ktile3(nk - 2, std::integral_constant<int, 2>());
    prefetch_epi();
    ktile3(nk - 1, std::integral_constant<int, 3>());
    __builtin_amdgcn_s_setprio(0);
  } else {
    // All RING stages are filled up front; the hand-over from tile kt to kt + 1 sits before the last
    // step's MFMAs, whose fragments are in registers: wait until tile kt + 1 has landed (the loads of
    // the RING - 2 tiles after it stay in flight), barrier, then stage kt % RING, which every wave has
    // read, takes tile kt + RING. With five stages three to four k-tiles (96-128 KB) are on their way at any
    // time, which is what covers the memory latency when a CU holds this one workgroup; with two stages
    // the other workgroups of the CU do.
    constexpr int L = A_LOADS + W_LOADS;
    static_assert(RING <= 1 || (RING - 2) * L <= 15, "the waits below use the low four bits of vmcnt");
    auto wait_tiles = [&](int n) {   // at most the loads of n tiles in flight, LDS reads done
      if (n >= RING - 2) __builtin_amdgcn_s_waitcnt(0x0070 | ((RING - 2) * L & 15));
      else if (n == 2) __builtin_amdgcn_s_waitcnt(0x0070 | (2 * L & 15));
      else if (n == 1) __builtin_amdgcn_s_waitcnt(0x0070 | L);
      else __builtin_amdgcn_s_waitcnt(0x0070);
    };
    auto step = [&](int kt, auto ph_c) {
      constexpr int PH = decltype(ph_c)::value;   // 0: refill tile kt + RING; 1: none; 2: last tile
#pragma unroll
      for (int s = 0; s < BK / KS; s++) {
        const int rb = s & 1;
        const bool seam = s == BK / KS - 1;
        if (!seam) {
          frags(kt, s + 1, rb ^ 1);
        } else if (PH < 2) {
          wait_tiles(PH == 0 ? RING - 2 : nk - 2 - kt);
          __syncthreads();
          if (PH == 0) {
            issue_a(kt + RING);
            issue_w(kt + RING);
          }
          frags(kt + 1, 0, rb ^ 1);
        }
#pragma unroll
        for (int i = 0; i < TI; i++)
#pragma unroll
          for (int j = 0; j < TJ; j++) acc[i][j] = mfma16(fw[rb][i], fa[rb][j], acc[i][j]);
      }
    };
    for (int kt = 0; kt < RING && kt < nk; kt++) {
      issue_a(kt);
      issue_w(kt);
    }
    if (nk >= RING) __builtin_amdgcn_s_waitcnt(0x0070 | ((RING - 1) * L & 15) | (((RING - 1) * L >> 4) << 14));
    else wait_tiles(nk - 1);
    __syncthreads();
    frags(0, 0, 0);
    int kt = 0;
    for (; kt + RING < nk; kt++) step(kt, std::integral_constant<int, 0>());
    for (; kt + 1 < nk; kt++) step(kt, std::integral_constant<int, 1>());
    prefetch_epi();
    step(nk - 1, std::integral_constant<int, 2>());
  }

  if constexpr (SPLIT) {
    // The exchange uses stores and loads of system scope (past this XCD's L2, the caches of different XCDs
    // not being coherent), each completed before the count that announces it. Ordinary accesses with
    // fences cost far more: a fence writes back, or drops, the whole L2 under every other workgroup
    // (one-seed MLP down 177 us with them).
    constexpr int SYSTEM = 17;           // cache policy bits sc0 | sc1
    int* cnt = split.counters + 4 * t;   // tickets taken, partial tiles stored, parts in slots 0 and 1
    __syncthreads();                     // every wave is done with the operand tiles
    int* bc = (int*)smem;
    if (tid == 0) bc[0] = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(bc[0]);
    // A tile's slots lie one after the other, each as [i][j][wave] blocks of 1 KB. Where the scratch has no room for
    // that, every slot holds, for all tiles, the rows that exist and no others (DENSE), so that two partial sums of any
    // number of rows fit in 8 bytes per row and column: a ragged tile as [i][j][wm][wn] blocks of 16 columns and up to
    // 16 rows.
    const int vr = DENSE ? min(P.M - m0, BM) : BM;
    const size_t first = DENSE ? (size_t)(pi == 0 ? 0 : pr.p[0].M) * cdiv(pr.p[0].N, BN) + (size_t)m0 * nt + (size_t)tn * vr
                               : (size_t)t * (splits - 1) * BM;   // row of BN sums that this tile starts at
    const uint32_t slot_bytes = DENSE ? (uint32_t)split.bytes : BM * BN * 4;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (char*)split.partials + first * BN * 4, (short)0, (int)((splits - 2) * slot_bytes + vr * BN * 4), 0x00020000);
    // Block (i, j) of this wave: a scalar offset in the slot, and this lane's place there (past the buffer where the
    // block has no such row), which are constants in a whole tile.
    struct Whole {
      uint32_t v;
      __device__ __forceinline__ uint32_t soff(int i, int j) const { return (uint32_t)(i * TJ + j) * (NW * 1024u); }
      __device__ __forceinline__ uint32_t voff(int) const { return v; }
      __device__ __forceinline__ bool has(int) const { return true; }
    };
    struct Ragged {
      uint32_t istep, b[TJ], v[TJ];
      __device__ __forceinline__ uint32_t soff(int i, int j) const { return i * istep + b[j]; }
      __device__ __forceinline__ uint32_t voff(int j) const { return v[j]; }
      __device__ __forceinline__ bool has(int j) const { return v[j] != 0x80000000u; }
    };
    auto ragged = [&]() {
      const int wm_s = wave_s / WN, wn_s = wave_s % WN;
      Ragged r;
      r.istep = (uint32_t)vr * WN * 64u;
      int before = 0;   // rows in blocks (0, j') of j' < j
#pragma unroll
      for (int j = 0; j < TJ; j++) {
        int rows = 0, mine = 0, lower = before;
#pragma unroll
        for (int w = 0; w < WM; w++) {
          const int q = min(max(vr - w * WTM - MS * j, 0), MS);
          if (w < wm_s) lower += q;
          if (w == wm_s) mine = q;
          rows += q;
        }
        r.b[j] = mine > 0 ? (uint32_t)(lower * WN + mine * wn_s) * 64u : 0u;
        r.v[j] = frow < mine ? (uint32_t)(lkc * mine + frow) * 16u : OOB;
        before += rows;
      }
      return r;
    };
    auto store = [&](const auto& at) {
#pragma unroll
      for (int i = 0; i < TI; i++)
#pragma unroll
        for (int j = 0; j < TJ; j++)
          if (at.has(j))
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[i][j]), rs, at.voff(j),
                                                   ticket * slot_bytes + at.soff(i, j), SYSTEM);
    };
    auto add = [&](const auto& at, uint32_t lo) {
      auto load = [&](uint32_t slot, int i, int j) {   // (zeros for rows past the end)
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, at.voff(j), slot * slot_bytes + at.soff(i, j), SYSTEM));
      };
      if (splits == 2) {
#pragma unroll
        for (int i = 0; i < TI; i++) {
#pragma unroll
          for (int j = 0; j < TJ; j++) acc[i][j] += load(0, i, j);
          __builtin_amdgcn_sched_barrier(0);   // a row of blocks in flight: more would not fit the registers
        }
      } else {   // (p0 + p1) + p2, whichever of them this one is
#pragma unroll
        for (int i = 0; i < TI; i++) {
#pragma unroll
          for (int j = 0; j < TJ; j++) {
            const f32x4 l = load(lo, i, j), h = load(lo ^ 1, i, j);
            acc[i][j] = part == 2 ? (l + h) + acc[i][j] : (l + acc[i][j]) + h;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    const bool whole = !DENSE || vr == BM;
    if (ticket < splits - 1) {
      if (whole) store(Whole{tid * 16u});
      else store(ragged());
      if (tid == 0) __hip_atomic_store(cnt + 2 + ticket, part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) __hip_atomic_fetch_add(cnt + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    if (tid == 0) {
      while (__hip_atomic_load(cnt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < splits - 1) __builtin_amdgcn_s_sleep(2);
      // which of the two slots holds the lower part
      bc[1] = splits > 2 && __hip_atomic_load(cnt + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >
                                __hip_atomic_load(cnt + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const uint32_t lo = __builtin_amdgcn_readfirstlane(bc[1]);
    if (whole) add(Whole{tid * 16u}, lo);
    else add(ragged(), lo);
  }

  // ---- epilogue: bias, gate vectors and the RoPE table are staged in LDS once per tile ----
  // accumulator (i, j), register q: n = 16 i + 4 (lane / 16) + q, m = 16 j + lane % 16
  // Blocks i and i + 1 of a row group (32 adjacent columns) are finished
  // together and regrouped with v_permlane16_swap, which exchanges lanes 16-31 of one register with
  // lanes 0-15 of another (and 48-63 with 32-47). Lane group g = lane / 16 then holds the 8 adjacent
  // columns 32 p + 16 (g & 1) + 8 (g >> 1) of pair p, stored with one 16-byte store. A CU issues a
  // store of 16 rows x 32 B (the accumulator layout) in ~74 cycles and one of 16 rows x 64 B in ~20,
  // and with 256 stores per tile that issue time, not HBM, bounded the epilogue. The paired layout
  // needs 16-byte aligned output rows; otherwise the accumulator layout is stored as it is.
  static_assert(TI % 2 == 0, "the paired store joins blocks 2p and 2p + 1");
  constexpr bool OUTF32 = EPI == EPI_STORE_F32;   // 16 bytes per block as it is
  const bool pairs = !OUTF32 && (P.N & 7) == 0 && ((uintptr_t)P.C & 15) == 0 &&
                     ((P.cmap.batch_stride | P.cmap.row_stride | P.cmap.offset) & 7) == 0;
  const int pair_col = 16 * (lkc & 1) + 8 * (lkc >> 1);
  // The residual values of this wave's whole sub-tile (64 registers, free now that the
  // fragment registers are dead) are requested at once, before the staging barriers, so their memory
  // latency is paid once per tile and overlaps the staging. xq[j][p] holds blocks (2p, j) and
  // (2p + 1, j): in the paired layout as loaded (one 16-byte load), else as two 8-byte loads in the
  // accumulator layout.
  constexpr bool XALL = EPI == EPI_RESID;
  uint4 xq[XALL ? TJ : 1][XALL ? TI / 2 : 1];
  if constexpr (XALL) {
    // buffer loads, so that no load sits in a branch: a conditional load leaves the compiler unable to
    // count the loads in flight, and it then waits for every earlier memory operation (stores
    // included) before each use
    const uint32_t OOB = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(P.C, (short)0, 0x7fffffff, 0x00020000);
    if (pairs) {
#pragma unroll
      for (int j = 0; j < TJ; j++) {
        const int m = m0 + wm * WTM + MS * j + frow;
        const uint32_t roff = m < P.M ? (uint32_t)(row_epi(P, m).off * 2) : OOB;
#pragma unroll
        for (int p = 0; p < TI / 2; p++) {
          const int c = n0 + wn * WTN + 32 * p + pair_col;
          const uint32_t off = (m < P.M && c < P.N) ? roff + (uint32_t)c * 2u : OOB;
          xq[j][p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rc, off, 0, 0));
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < TJ; j++) {
        const int m = m0 + wm * WTM + MS * j + frow;
        const uint32_t roff = m < P.M ? (uint32_t)(row_epi(P, m).off * 2) : OOB;
#pragma unroll
        for (int p = 0; p < TI / 2; p++) {
          uint2 h[2];
#pragma unroll
          for (int e = 0; e < 2; e++) {
            const int n = n0 + wn * WTN + MS * (2 * p + e) + 4 * lkc;
            const uint32_t off = (m < P.M && n < P.N) ? roff + (uint32_t)n * 2u : OOB;
            h[e] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rc, off, 0, 0));
          }
          xq[j][p] = make_uint4(h[0].x, h[0].y, h[1].x, h[1].y);
        }
      }
    }
  }
  __syncthreads();   // every wave is done with the operand tiles
  float* s_bias = (float*)smem;                       // [BN]
  float* s_gate = s_bias + BN;                        // [nbt][BN]
  float* s_rope = s_bias + BN;                        // [npos][head_dim/4][2] (QKV only)
  if (pre) {
    if (tid < BN) s_bias[tid] = to_f32(pre_b);
    if (gate_lds && tid < nbt * BN) s_gate[tid] = pre_g;
    if (rope_lds) {
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (tid + r * NT < rope_n) s_rope[tid + r * NT] = pre_r[r];
    }
  } else {
    for (int q = tid; q < BN; q += NT)
      s_bias[q] = (P.bias && n0 + q < P.N) ? to_f32(((const u16*)P.bias)[n0 + q]) : 0.f;
    if (gate_lds)
      for (int q = tid; q < nbt * BN; q += NT) {
        int bb = q / BN, nn = q - bb * BN;
        s_gate[q] = n0 + nn < P.N ? P.gate[(int64_t)(bfirst + bb) * P.gate_bstride + n0 + nn] : 0.f;
      }
    if (rope_lds)
      for (int q = tid; q < rope_n; q += NT) s_rope[q] = P.rope_tab[q];
  }
  __syncthreads();

  // The store loop reads the gate vectors and the RoPE table either from LDS (STAGED) or, for tiles
  // whose inputs did not fit the staging area, from global memory. The two are separate instances:
  // a pointer that may point to either is a flat address, and a flat load makes the compiler wait
  // for every store issued before it.
  const bool rope_on = EPI == EPI_QKV && P.rope_tab != nullptr;
  const int rope_cols = 2 * P.hidden, head_dim = P.head_dim;
  auto store_tile = [&](auto staged_c) {
    constexpr bool STAGED = decltype(staged_c)::value;
#pragma unroll
    for (int j = 0; j < TJ; j++) {
      int m = m0 + wm * WTM + MS * j + frow;
      if (m >= P.M) continue;
      const RowEpi R = row_epi(P, m);
      const int bt = m / rpb - bfirst;
#pragma unroll
      for (int i = 0; i < TI; i++) {
        int nl = wn * WTN + MS * i + 4 * lkc;   // column inside the tile
        int n = n0 + nl;
        if (n >= P.N) continue;
        float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
        float4 bv = *(const float4*)(s_bias + nl);
        v[0] += bv.x; v[1] += bv.y; v[2] += bv.z; v[3] += bv.w;
        if (EPI == EPI_GELU) {
#pragma unroll
          for (int q = 0; q < 4; q++) v[q] = gelu_tanh_f(v[q]);
        }
        if (EPI == EPI_RESID) {
          float4 gv = STAGED ? *(const float4*)(s_gate + bt * BN + nl) : *(const float4*)(P.gate + R.gate + n);
          const uint4 xx = xq[j][i >> 1];
          const uint2 u = (i & 1) ? make_uint2(xx.z, xx.w) : make_uint2(xx.x, xx.y);
          v[0] = fmaf(gv.x, v[0], __uint_as_float(u.x << 16));
          v[1] = fmaf(gv.y, v[1], __uint_as_float(u.x & 0xffff0000u));
          v[2] = fmaf(gv.z, v[2], __uint_as_float(u.y << 16));
          v[3] = fmaf(gv.w, v[3], __uint_as_float(u.y & 0xffff0000u));
        }
        if (EPI == EPI_QKV && rope_on && n < rope_cols) {
          int dd = n & (head_dim - 1);
          int hh = head_dim >> 1;
          int pos = dd < hh ? R.rpos : R.cpos;
          int pr = (dd & (hh - 1)) >> 1;
          int ti = (pos * (head_dim >> 2) + pr) * 2;
          float4 t = STAGED ? *(const float4*)(s_rope + ti) : *(const float4*)(P.rope_tab + ti);
          float a0 = v[0], b0 = v[1], a1 = v[2], b1 = v[3];
          v[0] = a0 * t.x - b0 * t.y;
          v[1] = a0 * t.y + b0 * t.x;
          v[2] = a1 * t.z - b1 * t.w;
          v[3] = a1 * t.w + b1 * t.z;
        }
        if constexpr (OUTF32) store4<float>((float*)P.C + R.off + n, v);
        else store4<u16>((u16*)P.C + R.off + n, v);
      }
    }
  };
  // The paired store: the same arithmetic per accumulator block as store_tile, then the regrouping
  // swap on the packed bf16 pairs and one 16-byte store per pair of blocks. The residual values arrive
  // in the paired layout and go through the same swap (it is its own inverse) before use.
  auto store_pairs = [&](auto staged_c) {
    constexpr bool STAGED = decltype(staged_c)::value;
#pragma unroll
    for (int j = 0; j < TJ; j++) {
      const int m = m0 + wm * WTM + MS * j + frow;
      if (m >= P.M) continue;   // the swap partners (lanes l and l ^ 16) share the row m
      const RowEpi R = row_epi(P, m);
      const int bt = m / rpb - bfirst;
#pragma unroll
      for (int p = 0; p < TI / 2; p++) {
        uint4 xr = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (XALL) {
          xr = xq[j][p];
          swap16(xr.x, xr.z);
          swap16(xr.y, xr.w);
        }
        uint32_t w[2][2];
#pragma unroll
        for (int e = 0; e < 2; e++) {
          const int i = 2 * p + e;
          const int nl = wn * WTN + MS * i + 4 * lkc;   // column inside the tile
          const int n = n0 + nl;
          float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
          float4 bv = *(const float4*)(s_bias + nl);
          v[0] += bv.x; v[1] += bv.y; v[2] += bv.z; v[3] += bv.w;
          if (EPI == EPI_GELU) {
#pragma unroll
            for (int q = 0; q < 4; q++) v[q] = gelu_tanh_f(v[q]);
          }
          if (EPI == EPI_RESID) {
            float4 gv = make_float4(0.f, 0.f, 0.f, 0.f);
            if (STAGED) gv = *(const float4*)(s_gate + bt * BN + nl);
            else if (n < P.N) gv = *(const float4*)(P.gate + R.gate + n);
            const uint32_t u0 = e ? xr.z : xr.x, u1 = e ? xr.w : xr.y;
            v[0] = fmaf(gv.x, v[0], __uint_as_float(u0 << 16));
            v[1] = fmaf(gv.y, v[1], __uint_as_float(u0 & 0xffff0000u));
            v[2] = fmaf(gv.z, v[2], __uint_as_float(u1 << 16));
            v[3] = fmaf(gv.w, v[3], __uint_as_float(u1 & 0xffff0000u));
          }
          if (EPI == EPI_QKV && rope_on && n < rope_cols) {
            int dd = n & (head_dim - 1);
            int hh = head_dim >> 1;
            int pos = dd < hh ? R.rpos : R.cpos;
            int pr = (dd & (hh - 1)) >> 1;
            int ti = (pos * (head_dim >> 2) + pr) * 2;
            float4 t = STAGED ? *(const float4*)(s_rope + ti) : *(const float4*)(P.rope_tab + ti);
            float a0 = v[0], b0 = v[1], a1 = v[2], b1 = v[3];
            v[0] = a0 * t.x - b0 * t.y;
            v[1] = a0 * t.y + b0 * t.x;
            v[2] = a1 * t.z - b1 * t.w;
            v[3] = a1 * t.w + b1 * t.z;
          }
          w[e][0] = pack_bf16x2(v[0], v[1]);
          w[e][1] = pack_bf16x2(v[2], v[3]);
        }
        swap16(w[0][0], w[1][0]);
        swap16(w[0][1], w[1][1]);
        const int c = n0 + wn * WTN + 32 * p + pair_col;
        if (c < P.N) *(uint4*)((u16*)P.C + R.off + c) = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
      }
    }
  };
  const bool staged = (EPI != EPI_RESID || gate_lds) && (!rope_on || rope_lds);
  // XALL: every residual load has landed before the first store. The compiler cannot order stores
  // against loads on this counter, so inside the loop it would instead wait for earlier stores.
  if constexpr (XALL) __builtin_amdgcn_s_waitcnt(0);
  if (pairs) {   // (never with fp32 output)
    if (staged) store_pairs(std::true_type());
    else store_pairs(std::false_type());
  } else {
    if (staged) store_tile(std::true_type());
    else store_tile(std::false_type());
  }
#endif
}

// buffer descriptor of a tile's operand rows, starting at the tile's first row
__device__ __forceinline__ u32x4_t tile_rsrc(const void* p) {
  const uint64_t u = (uint64_t)p;
  return u32x4_t{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(u >> 32) & 0xffffu)), 0x7fffffffu, 0x00020000u};
}

// T x T tile (T = 32 or 64) for problems with few tiles: each of a workgroup's 4 waves takes every 4th
// 64-deep k slice of the whole tile, with two LDS stages of its own (2 x T x 256 bytes), so no barrier
// stands in the k loop and two slices per wave are in flight; the four partial tiles meet in LDS and
// are summed in a fixed order, each wave finishing the 16 features x T rows (T = 64) or the 16 x 16
// block (T = 32) of its index. Small problems are bound by the latency of the chain of k-tiles, which
// this divides by four. Offsets are relative to the tile's first row; rows past the end repeat the last.
template <int T, int EPI>
__global__ void __launch_bounds__(256) gemm_bf16_ksplit_kernel(GemmPair pr, int tiles0, int total_tiles) {
  constexpr int NB = T / 16, LD = T / 8, STAGE = 2 * T * 128;
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int per = gridDim.x >> 3;
  const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (t >= total_tiles) return;
  const int pi = t < tiles0 ? 0 : 1;
  const GemmProblem P = pr.p[pi];
  int tm, tn;
  tile_coords(pi == 0 ? t : t - tiles0, cdiv(P.M, T), cdiv(P.N, T), tm, tn);
  const int m0 = tm * T, n0 = tn * T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t a0 = row_offset(P.amap, m0);
  const u32x4_t ra = tile_rsrc((const u16*)P.A + a0);
  const u32x4_t rw = tile_rsrc((const u16*)P.W + (int64_t)n0 * P.K);
  uint32_t aoff[LD], woff[LD];
#pragma unroll
  for (int i = 0; i < LD; i++) {
    const int r = 8 * i + (lane >> 3);
    const uint32_t chunk = ((lane & 7) ^ swz(r)) * 16;
    aoff[i] = (uint32_t)((row_offset(P.amap, min(m0 + r, P.M - 1)) - a0) * 2) + chunk;
    woff[i] = (uint32_t)(min(n0 + r, P.N - 1) - n0) * (uint32_t)P.K * 2u + chunk;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem + wave * 2 * STAGE;
  auto issue = [&](int slice, int st) {
    const uint32_t base = lds0 + st * STAGE;
#pragma unroll
    for (int i = 0; i < LD; i++) {
      dma_b128(ra, base + i * 1024, aoff[i], slice * 128);
      dma_b128(rw, base + T * 128 + i * 1024, woff[i], slice * 128);
    }
  };
  const int r16 = lane & 15, kq = lane >> 4;
  f32x4 acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int j = 0; j < NB; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = P.K / 64;
  if (wave < nk) issue(wave, 0);
  if (wave + 4 < nk) issue(wave + 4, 1);
  int st = 0;
  for (int kt = wave; kt < nk; kt += 4) {
    // this wave's slice kt has landed (the 2 LD loads of its next slice may be in flight)
    if (kt + 4 >= nk) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (LD == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    const char* sa = smem + wave * 2 * STAGE + st * STAGE;
    const char* sw = sa + T * 128;
    bf16x8 fw[2][NB], fa[2][NB];
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int i = 0; i < NB; i++) {
        const int r = 16 * i + r16;
        fw[s][i] = *(const bf16x8*)(sw + r * 128 + (((4 * s + kq) ^ swz(r)) << 4));
        fa[s][i] = *(const bf16x8*)(sa + r * 128 + (((4 * s + kq) ^ swz(r)) << 4));
      }
    if (kt + 8 < nk) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the fragments are in registers: the stage is free
      issue(kt + 8, st);
    }
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < NB; j++) acc[i][j] = mfma16(fw[s][i], fa[s][j], acc[i][j]);
    st ^= 1;
  }
  __syncthreads();   // every wave's loads have landed and been read
  f32x4* part = (f32x4*)smem;   // [block][wave][lane]
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int j = 0; j < NB; j++) part[((NB * i + j) * 4 + wave) * 64 + lane] = acc[i][j];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NB * NB / 4; q++) {
    const int blk = wave * (NB * NB / 4) + q, i = blk / NB, j = blk % NB;
    f32x4 c = part[(blk * 4) * 64 + lane];
#pragma unroll
    for (int g = 1; g < 4; g++) {
      const f32x4 p = part[(blk * 4 + g) * 64 + lane];
#pragma unroll
      for (int r = 0; r < 4; r++) c[r] += p[r];
    }
    const int m = m0 + 16 * j + r16, n = n0 + 16 * i + 4 * kq;
    if (m < P.M && n < P.N) {
      float v[4] = {c[0], c[1], c[2], c[3]};
      epilogue4<EPI, u16, std::conditional_t<EPI == EPI_STORE_F32, float, u16>>(P, row_epi(P, m), n, v);
    }
  }
#endif
}

// Raises a kernel's dynamic-LDS limit once per device and kernel instance (the flags belong to it).
// Two host threads may reach this at once; setting the attribute twice is harmless, and the flags are
// atomics so the check itself is race-free.
static hipError_t allow_lds(const void* kernel, size_t lds, std::atomic<bool>* attr_set) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = 0;
  if (lds > 65536 && (dev < 0 || dev >= 64 || !attr_set[dev].load(std::memory_order_acquire))) {
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) attr_set[dev].store(true, std::memory_order_release);
  }
  return hipSuccess;
}

// tiles of each problem of a pair
static int count_tiles(const GemmPair& pr, int bm, int bn, int* tiles) {
  int total = 0;
  for (int i = 0; i < 2; i++) {
    tiles[i] = i < pr.nprob && pr.p[i].M > 0 && pr.p[i].N > 0 ? cdiv(pr.p[i].M, bm) * cdiv(pr.p[i].N, bn) : 0;
    total += tiles[i];
  }
  return total;
}

// bytes of one part's partial sums in tiles of bn columns, for the rows that exist
static size_t split_slot_bytes(const GemmPair& pr, int bn) {
  size_t b = 0;
  for (int i = 0; i < pr.nprob; i++)
    if (pr.p[i].M > 0 && pr.p[i].N > 0) b += (size_t)pr.p[i].M * cdiv(pr.p[i].N, bn) * bn * 4;
  return b;
}

template <int T, int EPI>
static hipError_t launch_ksplit(const GemmPair& pr, hipStream_t s) {
  int tiles[2];
  const int total = count_tiles(pr, T, T, tiles);
  if (total == 0) return hipSuccess;
  constexpr size_t lds = (size_t)16 * T * 128;
  static std::atomic<bool> attr_set[64] = {};
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&gemm_bf16_ksplit_kernel<T, EPI>), lds, attr_set);
  if (e != hipSuccess) return e;
  gemm_bf16_ksplit_kernel<T, EPI><<<8 * cdiv(total, 8), 256, lds, s>>>(pr, tiles[0], total);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int EPI, int RING = 0, bool SPLIT = false, bool DENSE = false>
static hipError_t launch_bf16(const GemmPair& pr, hipStream_t s, int splits = 1, const GemmSplitWs& split = GemmSplitWs{}) {
  int tiles[2];
  const int total = count_tiles(pr, BM, BN, tiles);
  if (total == 0) return hipSuccess;
  GemmSplitWs ws = split;
  if constexpr (SPLIT && !DENSE)
    if ((size_t)total * (splits - 1) * BM * BN * 4 > split.bytes)
      return launch_bf16<BM, BN, WM, WN, EPI, RING, true, true>(pr, s, splits, split);
  if constexpr (DENSE) ws.bytes = split_slot_bytes(pr, BN);
  constexpr size_t lds = RING == 0 ? (size_t)(2 * BN + 3 * BM) * 64 * 2 : RING * (size_t)(BM + BN) * 64 * 2;
  static std::atomic<bool> attr_set[64] = {};
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&gemm_bf16_kernel<BM, BN, WM, WN, EPI, RING, SPLIT, DENSE>), lds, attr_set);
  if (e != hipSuccess) return e;
  gemm_bf16_kernel<BM, BN, WM, WN, EPI, RING, SPLIT, DENSE><<<8 * cdiv((int64_t)total * splits, 8), WM * WN * 64, lds, s>>>(
      pr, tiles[0], total, splits, ws);
  return hipGetLastError();
}

// Compute units of the current device (one 256 x 256 workgroup fills a CU: 160 KB of LDS and the
// whole register file), read once per device.
static int cu_count() {
  static std::atomic<int> cus[64] = {};   // 0 = not read yet; concurrent first reads store the same value
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Which tile a problem pair takes, from the estimated time (us) of its rounds of workgroups. A CU takes
// operand tiles in at about 54 KB/us whatever the tile, so a k-tile costs in proportion to its bytes
// (1.2 us for 256 x 256, 0.59 for 128 x 128, 0.30 for 64 x 64; 32 x 32 runs two workgroups per CU), on
// top of a fixed cost per tile (prologue, epilogue). Measured at hidden 3072, one seed at 512x512
// (1024 + 256 rows; us for 32 / 64 / 128 / 256 tiles): out-projection 93 / 77 / 39 / 71, MLP down
// 331 / 218 / 124 / 230, QKV 258 / 197 / 104 / 74; at 256 + 64 rows: out-projection 32 / 25 / 36 / 70;
// at hidden 320, 286 + 74 rows: 6.7 / 9.7 / 10 / 18. 256 x 192 tiles for all rows take 0.85-0.88
// of a 256 x 256 round (17% more operand bytes per flop) and win where they fill a round that 256 x 256
// tiles leave part empty (QKV of one seed, 240 tiles against 180: 65 against 74 us); a text problem's own
// launch of them, after the image rows' whole rounds, takes 0.83.
enum Tile { TILE_32, TILE_64, TILE_64_RING, TILE_128, TILE_192, TILE_256, TILE_256_192 };
static Tile pick_tile(const GemmPair& pr, bool plain, const GemmSplitWs& split, int* splits) {
  int t[2];
  const int64_t cus = cu_count();
  *splits = 1;
  // Plain stores of short K (the patch embedding) are bound by what a tile costs besides its k loop, which the
  // estimates below, made for long K, do not tell apart. 64 x 64 tiles in a ring of two stages (32 KB, up to
  // five workgroups per CU: one's stores overlap another's loads) win where they give every second CU one and
  // no CU more than six, and at one or two k-tiles also below that. With the rounding of the latent, this / the
  // tile picked below / the former 64 x 64 and 128 x 128 tiles of two stages (us): 9000 x 64, K 64: 6.4 / 8.5 /
  // 6.5; 1000 x 640, K 128: 6.2 / 8.0 / 8.6; 4096 x 1280, K 64: 9.5 / 11.5 / 11.8, K 512: 19.7 / 22.8 / 20.6;
  // outside, 360 x 640, K 512: 9.1 / 6.8 / 12.2; 16384 x 1280, K 512: 51.4 / 44.8 / 48.8.
  if (plain && pr.p[0].K <= 512) {
    const int64_t n = count_tiles(pr, 64, 64, t);
    if (n <= 6 * cus && (2 * n >= cus || pr.p[0].K <= 128)) return TILE_64_RING;
  }
  const double kt = pr.p[0].K / 64;
  auto rounds = [&](int64_t tiles, int64_t slots) { return (double)((tiles + slots - 1) / slots); };
  const double r256 = 1.2 * kt + 14.0;
  double best = rounds(count_tiles(pr, 256, 256, t), cus) * r256;
  Tile pick = TILE_256;
  // image and text rows as two launches, the text rows on 256 x 192 tiles: with 4096 text rows and 3072 or
  // 9216 output features those divide into whole rounds
  if (t[0] > 0 && t[1] > 0) {
    const int64_t t0 = t[0];
    count_tiles(pr, 256, 192, t);
    const double c = (rounds(t0, cus) + 0.83 * rounds(t[1], cus)) * r256;
    if (c < best) best = c, pick = TILE_256_192;
  }
  auto consider = [&](Tile tile, double cost) {
    if (cost < best) best = cost, pick = tile;
  };
  consider(TILE_192, rounds(count_tiles(pr, 256, 192, t), cus) * 0.87 * r256);
  consider(TILE_128, rounds(count_tiles(pr, 128, 128, t), cus) * (0.59 * kt + 7.0));
  consider(TILE_64, rounds(count_tiles(pr, 64, 64, t), cus) * (0.30 * kt + 7.0));
  consider(TILE_32, rounds(count_tiles(pr, 32, 32, t), 2 * cus) * (0.22 * kt + 3.0));
  // 256-row tiles with K shared out, where the partial tiles fit the scratch: storing and adding those takes 5 us and
  // 0.6 us per MB, with 256 x 256 tiles, whose registers hold fewer loads in flight, 10 us in two parts and 18 in
  // three. Measured with every form forced in turn (us, unsplit / two parts on 256 x 192 / three / two on 256 x 256 /
  // three; - where it does not fit): hidden 3072, 1024 + 256 rows: 128 / 119 / 101 / 140 / 116, 1024 + 250: 129 / 122 /
  // 104 / 143 / 121, 2046 + 500: 207 / - / - / 166 / -; hidden 576, 4784 + 2004 rows: 41 / 38 / 43 / 49 / 41; hidden 832,
  // 6708 + 4: 62 / 63 / - / 69 / -. Within 3% the unsplit form stays: its estimate is high where 128 x 128 tiles leave
  // half of the CUs idle (hidden 1152, 1130 + 64 rows: 42 / - / 45 / - / -).
  if (split.bytes > 0) {
    best *= 0.97;
    for (int sp = 2; sp <= 3; sp++)
      for (int bn = 192; bn <= 256; bn += 64) {
        const int64_t n = count_tiles(pr, 256, bn, t);
        const size_t partials = (sp - 1) * split_slot_bytes(pr, bn);
        if (n > split.max_tiles || kt < 8 * sp || partials > split.bytes) continue;
        const double c = rounds(n * sp, cus) * (bn == 192 ? 0.87 : 1.0) * (1.2 * kt / sp + 14.0) + 0.6e-6 * partials +
                         (bn == 192 ? 5.0 : sp == 2 ? 10.0 : 18.0);
        if (c < best) best = c, pick = bn == 192 ? TILE_192 : TILE_256, *splits = sp;
      }
  }
  return pick;
}

GemmPlan gemm_plan(const GemmPair& pr, int epi, const GemmSplitWs& split) {
  GemmPlan p{0, 0, 0, 1, 0};
  const Tile t = pick_tile(pr, epi == EPI_STORE || epi == EPI_STORE_F32, epi == EPI_RESID ? split : GemmSplitWs{}, &p.splits);
  p.tile_m = t == TILE_32 ? 32 : t == TILE_64 || t == TILE_64_RING ? 64 : t == TILE_128 ? 128 : 256;
  p.tile_n = t == TILE_192 ? 192 : p.tile_m;
  p.second_n = t == TILE_256_192 ? 192 : 0;
  p.ring = t == TILE_64_RING ? 2 : t == TILE_128 ? 5 : 0;
  return p;
}

template <int EPI>
static hipError_t dispatch_bf16(const GemmPair& pr, const GemmSplitWs& split, hipStream_t s) {
  int splits = 1;
  constexpr bool PLAIN = EPI == EPI_STORE || EPI == EPI_STORE_F32;
  const Tile tile = pick_tile(pr, PLAIN, split, &splits);
  if constexpr (EPI == EPI_RESID) {
    if (splits > 1 && tile == TILE_192) return launch_bf16<256, 192, 4, 2, EPI, 0, true>(pr, s, splits, split);
    if (splits > 1) return launch_bf16<256, 256, 4, 2, EPI, 0, true>(pr, s, splits, split);
  }
  switch (tile) {
    case TILE_32: return launch_ksplit<32, EPI>(pr, s);
    case TILE_64: return launch_ksplit<64, EPI>(pr, s);
    case TILE_64_RING:
      if constexpr (PLAIN) return launch_bf16<64, 64, 2, 2, EPI, 2>(pr, s);
      break;
    case TILE_128: return launch_bf16<128, 128, 2, 4, EPI, 5>(pr, s);
    case TILE_192: return launch_bf16<256, 192, 4, 2, EPI>(pr, s);
    case TILE_256: return launch_bf16<256, 256, 4, 2, EPI>(pr, s);
    case TILE_256_192: {
      GemmPair a = pr, b = pr;
      a.nprob = 1;
      b.nprob = 1;
      b.p[0] = pr.p[1];
      hipError_t e = launch_bf16<256, 256, 4, 2, EPI>(a, s);
      return e != hipSuccess ? e : launch_bf16<256, 192, 4, 2, EPI>(b, s);
    }
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// fp32 GEMM on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums).
// As in the bf16 path, MFMA operand "A" = rows of W, "B" = rows of A, so a lane owns one output row m
// and runs of 4 consecutive features n. A lane reads 4 consecutive k of its row with one ds_read_b128
// and gives element j to the j-th of four MFMAs; lane group g = lane / 16 then supplies k = 4 g + j of
// both operands, which is a permutation of the 16 k the four instructions sum over. LDS rows are 32
// floats = 8 chunks of 16 bytes, swizzled like the bf16 tiles (the reads have the same pattern).
// Operands go straight to LDS (buffer loads with the LDS bit) from a 64-bit base per tile with the
// offsets relative to the tile's first row; rows past the end repeat the last row and are not stored.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mfma_k16(float4 w, float4 a, f32x4& c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, a.x, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, a.y, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, a.z, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, a.w, c, 0, 0, 0);
}

// 64 x 64 tile, 4 waves of 32 x 32, 32-deep k-tiles in a ring of three LDS stages (48 KB, three
// workgroups per CU), one barrier per k-tile, which takes 1024 cycles of the fp32 matrix rate (256 flop per clock and
// CU) and moves 16 KB. 83-101 TFLOP/s in a block of hidden 768 and 2176 rows (a large library product: 137), whose
// 408 tiles of the output projection and MLP down fill the second round of 256 CUs by 60%.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmPair pr, int tiles0, int total_tiles) {
  constexpr int BM = 64, BN = 64, ST = 3, STAGE = (BM + BN) * 128;
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) char smem[ST * STAGE];
  const int per = gridDim.x >> 3;
  const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);   // XCD-aware, as in the bf16 kernel
  if (t >= total_tiles) return;
  const int pi = t < tiles0 ? 0 : 1;
  const GemmProblem P = pr.p[pi];
  int tm, tn;
  tile_coords(pi == 0 ? t : t - tiles0, cdiv(P.M, BM), cdiv(P.N, BN), tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t a0 = row_offset(P.amap, m0);
  const u32x4_t ra = tile_rsrc((const float*)P.A + a0);
  const u32x4_t rw = tile_rsrc((const float*)P.W + (int64_t)n0 * P.K);
  // a wave load fills 8 rows: lane -> row lane / 8, slot lane % 8, which holds chunk slot ^ swz(row)
  uint32_t aoff[2], woff[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int r = 8 * (wave * 2 + i) + (lane >> 3);
    const uint32_t chunk = ((lane & 7) ^ swz(r)) * 16;
    aoff[i] = (uint32_t)((row_offset(P.amap, min(m0 + r, P.M - 1)) - a0) * 4) + chunk;
    woff[i] = (uint32_t)(min(n0 + r, P.N - 1) - n0) * (uint32_t)P.K * 4u + chunk;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  auto issue = [&](int kt, int st) {
    const uint32_t base = lds0 + st * STAGE + wave_s * 2048;
#pragma unroll
    for (int i = 0; i < 2; i++) {
      dma_b128(ra, base + i * 1024, aoff[i], kt * 128);
      dma_b128(rw, base + BM * 128 + i * 1024, woff[i], kt * 128);
    }
  };
  const int wm = wave >> 1, wn = wave & 1, r16 = lane & 15, kq = lane >> 4;
  f32x4 acc[2][2] = {};
  const int nk = P.K / 32;
  issue(0, 0);
  if (nk > 1) issue(1, 1);
  int st = 0;
  for (int kt = 0; kt < nk; kt++) {
    // tile kt has landed (the 4 loads of tile kt + 1 may be in flight) in every wave, and every wave is
    // done reading tile kt - 1, whose stage takes tile kt + 2
    if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0f74);
    else __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    if (kt + 2 < nk) issue(kt + 2, st == 0 ? 2 : st - 1);
    const char* sa = smem + st * STAGE;
    const char* sw = sa + BM * 128;
#pragma unroll
    for (int s = 0; s < 2; s++) {
      float4 fw[2], fa[2];
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const int rw_ = 32 * wn + 16 * i + r16, ra_ = 32 * wm + 16 * i + r16;
        fw[i] = *(const float4*)(sw + rw_ * 128 + (((4 * s + kq) ^ swz(rw_)) << 4));
        fa[i] = *(const float4*)(sa + ra_ * 128 + (((4 * s + kq) ^ swz(ra_)) << 4));
      }
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) mfma_k16(fw[i], fa[j], acc[i][j]);
    }
    st = st == 2 ? 0 : st + 1;
  }
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const int m = m0 + 32 * wm + 16 * j + r16;
    if (m >= P.M) continue;
    const RowEpi R = row_epi(P, m);
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int n = n0 + 32 * wn + 16 * i + 4 * kq;
      float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      if (n < P.N) epilogue4<EPI, float, float>(P, R, n, v);
    }
  }
#endif
}

// 32 x 32 tile for problems with too few 64 x 64 tiles: the 4 waves of a workgroup take every 4th
// 32-deep k slice of the same tile, each with two LDS stages of its own (64 KB in all), so no barrier
// stands in the k loop and two slices of every wave are in flight; the four partial tiles meet in LDS
// and are summed in a fixed order. A quarter of the serial chain of the 64 x 64 kernel per tile, at
// twice its operand bytes per flop.
// WIDE: for rows so long that a tile's rows span more than a buffer descriptor addresses (2 GiB). The same
// slices come through registers from 64-bit addresses.
template <int EPI, bool WIDE>
__global__ void __launch_bounds__(256) gemm_f32_ksplit_kernel(GemmPair pr, int tiles0, int total_tiles) {
  constexpr int BM = 32, BN = 32, STAGE = (BM + BN) * 128;
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) char smem[4 * 2 * STAGE];
  const int per = gridDim.x >> 3;
  const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (t >= total_tiles) return;
  const int pi = t < tiles0 ? 0 : 1;
  const GemmProblem P = pr.p[pi];
  int tm, tn;
  tile_coords(pi == 0 ? t : t - tiles0, cdiv(P.M, BM), cdiv(P.N, BN), tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t a0 = row_offset(P.amap, m0);
  const u32x4_t ra = tile_rsrc((const float*)P.A + a0);
  const u32x4_t rw = tile_rsrc((const float*)P.W + (int64_t)n0 * P.K);
  uint32_t aoff[4], woff[4];
  const char *ap[4], *wp[4];   // WIDE: the same addresses in full
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = 8 * i + (lane >> 3);
    const uint32_t chunk = ((lane & 7) ^ swz(r)) * 16;
    const int64_t arow = row_offset(P.amap, min(m0 + r, P.M - 1)), wrow = min(n0 + r, P.N - 1);
    aoff[i] = (uint32_t)((arow - a0) * 4) + chunk;
    woff[i] = (uint32_t)(wrow - n0) * (uint32_t)P.K * 4u + chunk;
    if constexpr (WIDE) {
      ap[i] = (const char*)((const float*)P.A + arow) + chunk;
      wp[i] = (const char*)((const float*)P.W + wrow * P.K) + chunk;
    }
  }
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem + wave_s * 2 * STAGE;
  auto issue = [&](int slice, int st) {
    const uint32_t base = lds0 + st * STAGE;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if constexpr (WIDE) {
        char* dst = smem + (wave_s * 2 + st) * STAGE + i * 1024 + lane * 16;
        *(f32x4*)dst = *(const f32x4*)(ap[i] + (int64_t)slice * 128);
        *(f32x4*)(dst + BM * 128) = *(const f32x4*)(wp[i] + (int64_t)slice * 128);
      } else {
        dma_b128(ra, base + i * 1024, aoff[i], slice * 128);
        dma_b128(rw, base + BM * 128 + i * 1024, woff[i], slice * 128);
      }
    }
  };
  const int r16 = lane & 15, kq = lane >> 4;
  f32x4 acc[2][2] = {};
  const int nk = P.K / 32;
  if (wave_s < nk) issue(wave_s, 0);
  if (wave_s + 4 < nk) issue(wave_s + 4, 1);
  int st = 0;
  for (int kt = wave_s; kt < nk; kt += 4) {
    // this wave's slice kt has landed (the 8 loads of its next slice may be in flight)
    if (kt + 4 < nk) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* sa = smem + wave_s * 2 * STAGE + st * STAGE;
    const char* sw = sa + BM * 128;
    float4 fw[2][2], fa[2][2];
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const int r = 16 * i + r16;
        fw[s][i] = *(const float4*)(sw + r * 128 + (((4 * s + kq) ^ swz(r)) << 4));
        fa[s][i] = *(const float4*)(sa + r * 128 + (((4 * s + kq) ^ swz(r)) << 4));
      }
    if (kt + 8 < nk) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the fragments are in registers: the stage is free
      issue(kt + 8, st);
    }
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) mfma_k16(fw[s][i], fa[s][j], acc[i][j]);
    st ^= 1;
  }
  __syncthreads();   // every wave's loads have landed and been read
  f32x4* part = (f32x4*)smem;   // [block][wave][lane]
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) part[((2 * i + j) * 4 + wave) * 64 + lane] = acc[i][j];
  __syncthreads();
  // wave q finishes block (q / 2, q % 2)
  f32x4 c = part[(wave * 4) * 64 + lane];
#pragma unroll
  for (int g = 1; g < 4; g++) {
    const f32x4 p = part[(wave * 4 + g) * 64 + lane];
#pragma unroll
    for (int r = 0; r < 4; r++) c[r] += p[r];
  }
  const int m = m0 + 16 * (wave & 1) + r16, n = n0 + 16 * (wave >> 1) + 4 * kq;
  if (m < P.M && n < P.N) {
    float v[4] = {c[0], c[1], c[2], c[3]};
    epilogue4<EPI, float, float>(P, row_epi(P, m), n, v);
  }
#endif
}

template <int EPI>
static hipError_t launch_f32(const GemmPair& pr, hipStream_t s) {
  int tiles[2] = {0, 0}, small[2] = {0, 0};
  for (int i = 0; i < pr.nprob; i++)
    if (pr.p[i].M > 0 && pr.p[i].N > 0) {
      tiles[i] = cdiv(pr.p[i].M, 64) * cdiv(pr.p[i].N, 64);
      small[i] = cdiv(pr.p[i].M, 32) * cdiv(pr.p[i].N, 32);
    }
  const int total = tiles[0] + tiles[1], total_small = small[0] + small[1];
  if (total == 0) return hipSuccess;
  // matrix cycles of the fullest CU: a 64 x 64 tile takes 32 per k, a 32 x 32 one 8, and the small
  // tiles' doubled operand traffic costs them about a quarter
  const int cus = cu_count();
  const double big = 32.0 * cdiv(total, cus), little = 1.25 * 8.0 * cdiv(total_small, cus);
  // and a tile's rows must lie within what its buffer descriptor addresses
  const int64_t row = (int64_t)pr.p[0].K * 4, span = 0x7fffffff;
  if (32 * row > span)
    gemm_f32_ksplit_kernel<EPI, true><<<8 * cdiv(total_small, 8), 256, 0, s>>>(pr, small[0], total_small);
  else if (little < big || 64 * row > span)
    gemm_f32_ksplit_kernel<EPI, false><<<8 * cdiv(total_small, 8), 256, 0, s>>>(pr, small[0], total_small);
  else
    gemm_f32_kernel<EPI><<<8 * cdiv(total, 8), 256, 0, s>>>(pr, tiles[0], total);
  return hipGetLastError();
}

hipError_t gemm(const GemmPair& pr, int epi, int dtype, const GemmSplitWs& split, hipStream_t s) {
  if (dtype == DT_F32) {
    switch (epi) {
      case EPI_STORE: return launch_f32<EPI_STORE>(pr, s);
      case EPI_GELU: return launch_f32<EPI_GELU>(pr, s);
      case EPI_RESID: return launch_f32<EPI_RESID>(pr, s);
      case EPI_QKV: return launch_f32<EPI_QKV>(pr, s);
    }
    return hipErrorInvalidValue;
  }
  switch (epi) {
    case EPI_STORE: return dispatch_bf16<EPI_STORE>(pr, GemmSplitWs{}, s);
    case EPI_GELU: return dispatch_bf16<EPI_GELU>(pr, GemmSplitWs{}, s);
    case EPI_RESID: return dispatch_bf16<EPI_RESID>(pr, split, s);
    case EPI_QKV: return dispatch_bf16<EPI_QKV>(pr, GemmSplitWs{}, s);
    case EPI_STORE_F32: return dispatch_bf16<EPI_STORE_F32>(pr, GemmSplitWs{}, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace dit
