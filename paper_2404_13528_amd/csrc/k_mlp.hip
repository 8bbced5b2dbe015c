// Fused MLP: Y = residual + W2 . gelu(W1 . norm(x) + b1) + b2 per token, the hidden activation never leaving the
// compute unit.  Not an operator pair of the paper's tables (two ILD & Variable operators are kept apart there):
// it is the deeper fusion next to the layout path, where the hidden tensor is the largest intermediate of a block.
//
// Shape of the work: a workgroup owns 32 tokens and has one wave per 32 output features (T = C / 32 waves).  The
// token tile (normalised in place when the norm is folded) stays in LDS.  The hidden dimension is processed in rounds
// of T slices of 32 units.  In a round, wave w first forms its slice
//   H^T[32 hidden, 32 tokens] = W1[slice, :] . X^T        (C / 16 MFMAs, X fragments from LDS)
// applies bias + GELU in registers and writes the bf16 result into the round's hidden tile in LDS; after one barrier it
// accumulates its own output block over the whole round,
//   Y^T[32 features, 32 tokens] += W2[block, round's hidden] . H        (2 T MFMAs, H fragments from LDS)
// so no partial sums are exchanged and a wave needs 16 accumulator registers per product.  The hidden tile is
// double-buffered: one barrier per round.  No weight element is used twice inside a workgroup, so the weights go
// straight from L2 into MFMA operand registers (no LDS staging): one set of C / 16 fragment registers carries the
// wave's whole weight stream, each register refilled, right after the MFMA that read it, with the fragment the next
// product needs at the same position, so every load has a full product (C / 16 MFMAs) to arrive.
//
// Weight layout (the paper's principle that a producer writes the layout its consumer reads best, Sec. 3.2.2, applied
// to constants: done once by mlp_pack_kernel): an MFMA operand fragment is 64 lanes x 16 bytes taken from 32 rows, 32
// bytes per row; read from the row-major matrix every such load touches 32 cache lines for a quarter of their
// bytes (measured on an earlier form of this kernel: 76 us against 33 us for M = 6272, C = 384, hidden 1536).
// Packed, a fragment is 1 KiB contiguous in lane order, and each wave's fragments follow each other in the order it
// uses them:
//   W1 fragment (slice sc, step kk) at index sc * C/16 + kk:            lane (l32, hf) = W1[32 sc + l32][16 kk + 8 hf ..+7]
//   W2 fragment (block t, slice sc, step s) at (t * hidden/32 + sc) * 2 + s: lane (l32, hf) = W2[32 t + l32][32 sc + 16 s + 8 hf ..+7]
#include <atomic>
#include <type_traits>
#include "device_common.h"
#include "kernels.h"

namespace sm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 mlp_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float mlp_f32x16;
typedef unsigned int mlp_u32x4 __attribute__((ext_vector_type(4)));
typedef float mlp_f32x4 __attribute__((ext_vector_type(4)));
typedef float mlp_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 mlp_bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned mlp_pack2(float a, float b) {
  const mlp_f32x2 p = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(p, mlp_bf16x2));
}
__device__ __forceinline__ void mlp_unpack8(mlp_u32x4 v, float* f) {
#pragma unroll
  for (int e = 0; e < 4; ++e) { f[2 * e] = __uint_as_float(v[e] << 16); f[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u); }
}

// eight elements times rstd plus sh (the normalised value), times gamma plus beta, rounded to bf16
__device__ __forceinline__ mlp_u32x4 mlp_scale8(const mlp_u32x4& v, float rstd, float sh, const mlp_u32x4& gam, const mlp_u32x4& bet) {
  float f[8], g[8], b[8];
  mlp_unpack8(v, f);
  mlp_unpack8(gam, g);
  mlp_unpack8(bet, b);
  mlp_u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    o[e] = mlp_pack2(fmaf(fmaf(f[2 * e], rstd, sh), g[2 * e], b[2 * e]), fmaf(fmaf(f[2 * e + 1], rstd, sh), g[2 * e + 1], b[2 * e + 1]));
  return o;
}

// one thread per 16-byte chunk of the packed buffer: [W1 fragments | W2 fragments]
__global__ void mlp_pack_kernel(const bf16_t* W1, const bf16_t* W2, mlp_u32x4* packed, int C, int Hd) {
  const int KK = C / 16, nsub = Hd / 32;
  const int64_t n1 = (int64_t)Hd * C / 8;
  const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= 2 * n1) return;
  const int64_t q = o < n1 ? o : o - n1;
  const int lane = (int)(q & 63), l32 = lane & 31, hf = lane >> 5;
  const int64_t frag = q >> 6;
  const bf16_t* src;
  if (o < n1) {
    const int sc = (int)(frag / KK), kk = (int)(frag - (int64_t)sc * KK);
    src = W1 + (int64_t)(32 * sc + l32) * C + 16 * kk + 8 * hf;
  } else {
    const int s = (int)(frag & 1);
    const int64_t ft = frag >> 1;
    const int t = (int)(ft / nsub), sc = (int)(ft - (int64_t)t * nsub);
    src = W2 + (int64_t)(32 * t + l32) * Hd + 32 * sc + 16 * s + 8 * hf;
  }
  packed[o] = *(const mlp_u32x4*)src;
}

// ROWS token rows -> LDS, rows at an odd pitch of 16-byte slots (rows past M as zeros), in steps: rows() puts every row-offset
// lookup in flight, load() the loads, store() waits for them.  What a kernel requests in between (a second tile, the weight
// stream) travels at the same time.
template <int C, int NTHR, int ROWS>
struct MlpTile {
  static constexpr int XS = C / 8, XP = XS + 1, NIT = (ROWS * XS + NTHR - 1) / NTHR;
  mlp_u32x4 v[NIT];
  int64_t off[NIT];
  __device__ __forceinline__ void rows(int64_t row0, int64_t M, int ident, int64_t ld, const SM_KARG RowProg* prog) {
    int64_t row[NIT];
#pragma unroll
    for (int i = 0; i < NIT; ++i) row[i] = min(row0 + min((int)(threadIdx.x + i * NTHR) / XS, ROWS - 1), M - 1);
    if (ident) {
#pragma unroll
      for (int i = 0; i < NIT; ++i) off[i] = row[i] * ld;
    } else if (const int32_t* tab = prog->table) {
      int32_t t[NIT];
#pragma unroll
      for (int i = 0; i < NIT; ++i) t[i] = tab[row[i]];
#pragma unroll
      for (int i = 0; i < NIT; ++i) off[i] = t[i];
    } else {
#pragma unroll
      for (int i = 0; i < NIT; ++i) off[i] = eval_rows_k(prog, row[i]);
    }
  }
  __device__ __forceinline__ void load(const bf16_t* X) {
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int s = threadIdx.x + i * NTHR, c = s - s / XS * XS;
      v[i] = *(const mlp_u32x4*)(X + off[i] + (s < ROWS * XS ? c : 0) * 8);
    }
  }
  __device__ __forceinline__ void request(const bf16_t* X, int64_t row0, int64_t M, int ident, int64_t ld, const SM_KARG RowProg* prog) {
    rows(row0, M, ident, ld, prog);
    load(X);
  }
  __device__ __forceinline__ void store(mlp_u32x4* x_l, int64_t row0, int64_t M) const {
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int s = threadIdx.x + i * NTHR, r = s / XS, c = s - r * XS;
      if (s < ROWS * XS) x_l[r * XP + c] = row0 + r < M ? v[i] : mlp_u32x4{0u, 0u, 0u, 0u};
    }
  }
};

// LayerNorm of the tile's rows in place (the norm that precedes the product, folded): TPT adjacent lanes per token, each
// holding its chunks of the row in registers; two-pass fp32 statistics, the result rounded to bf16 as a separate norm
// kernel would have stored it.  No barrier inside.
template <int C, int NTHR, int NTOK>
__device__ __forceinline__ void mlp_norm_x_tile(mlp_u32x4* x_l, float eps, const mlp_u32x4* gam, const mlp_u32x4* bet) {
  constexpr int XS = C / 8, XP = XS + 1, Q = NTHR / NTOK, TPT = Q >= 16 ? 16 : Q >= 8 ? 8 : 4, NCH = (XS + TPT - 1) / TPT;
  static_assert(Q >= 4, "at least four lanes per token");
  const int r = threadIdx.x / TPT, p = threadIdx.x & (TPT - 1);
  if (r >= NTOK) return;                        // (whole groups of TPT lanes)
  mlp_u32x4* xr = x_l + r * XP;
  mlp_u32x4 x[NCH], gv[NCH], bv[NCH];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = min(p + TPT * i, XS - 1);
    x[i] = xr[c]; gv[i] = gam[c]; bv[i] = bet[c];
  }
  float sum = 0.f, var = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    float f[8];
    mlp_unpack8(x[i], f);
    if (XS % TPT == 0 || p + TPT * i < XS)
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += f[e];
  }
#pragma unroll
  for (int o = 1; o < TPT; o <<= 1) sum += __shfl_xor(sum, o, 64);
  const float mean = sum / (float)C;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    float f[8];
    mlp_unpack8(x[i], f);
    if (XS % TPT == 0 || p + TPT * i < XS)
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float d = f[e] - mean; var += d * d; }
  }
#pragma unroll
  for (int o = 1; o < TPT; o <<= 1) var += __shfl_xor(var, o, 64);
  const float rstd = rsqrtf(var / (float)C + eps), sh = -mean * rstd;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (XS % TPT == 0 || p + TPT * i < XS) xr[p + TPT * i] = mlp_scale8(x[i], rstd, sh, gv[i], bv[i]);
}

// Statistics of rows whose features lie in the registers of NW waves, NB blocks of 32 each (lane (token, hf): 16 features of a
// block): every wave leaves its own mean and sum of squared deviations, and after one barrier a lane joins them,
//   C var = sum over waves of [squares + 32 NB (mean of the wave - mean)^2],
// which loses no more than a second pass over the row would.
template <int NB>
__device__ __forceinline__ void mlp_stats_put(const mlp_u32x4 (&v)[NB][2], int hf, float2* st) {
  float f[NB][16];
  float sum = 0.f, sq = 0.f;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    mlp_unpack8(v[b][0], f[b]);
    mlp_unpack8(v[b][1], f[b] + 8);
#pragma unroll
    for (int e = 0; e < 16; ++e) sum += f[b][e];
  }
  sum += __shfl_xor(sum, 32, 64);
  const float m = sum * (1.f / (32 * NB));
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) { const float d = f[b][e] - m; sq += d * d; }
  sq += __shfl_xor(sq, 32, 64);
  if (hf == 0) *st = make_float2(m, sq);
}
// st: the token's word of wave 0, the next wave's `pitch` further on
template <int NB, int NW>
__device__ __forceinline__ void mlp_stats_get(const float2* st, int pitch, float eps, float* rstd, float* sh) {
  float mean = 0.f, sq = 0.f;
#pragma unroll
  for (int i = 0; i < NW; ++i) mean += st[i * pitch].x;
  mean *= 1.f / NW;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const float2 s = st[i * pitch];
    const float d = s.x - mean;
    sq += s.y + (float)(32 * NB) * d * d;
  }
  *rstd = rsqrtf(sq * (1.f / (32 * NB * NW)) + eps);
  *sh = -mean * *rstd;
}

// the lane's number computed afresh (a register that is live over all rounds for the epilogue's sake would be spilled)
__device__ __forceinline__ int mlp_lane() {
  unsigned z = 0;
  asm volatile("" : "+s"(z));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, z));
}
// A 32 x 32 block of results that a wave holds as 16-byte runs (lane (token, hf): runs 2 gp + hf of the token's four) goes to
// memory in whole 64-byte pieces, a piece in four adjacent lanes, by way of 2 KiB of LDS that only this wave uses.  Stored from
// where they are, an instruction touches 32 rows for 32 bytes each, and the Linears that write more than they read wait for the
// store path (packed Linear with LayerNorm, us: 200704 x 384 x 128 74.9 -> 62.2, 50176 x 768 x 256 51.0 -> 45.0, 12544 x 768 x 256
// 17.0 -> 13.3).  mlp_stage_get(i): token 16 i + lane / 4, run lane % 4.
__device__ __forceinline__ void mlp_stage_put(mlp_u32x4* st, int l32, int hf, const mlp_u32x4& v0, const mlp_u32x4& v1) {
  const int k = (l32 >> 2) & 3;                 // (16 lanes of a write, and of a read, in 16 different bank groups)
  st[l32 * 4 + (hf ^ k)] = v0;
  st[l32 * 4 + ((2 + hf) ^ k)] = v1;
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ mlp_u32x4 mlp_stage_get(const mlp_u32x4* st, int lane, int i) {
  const int t = 16 * i + (lane >> 2);
  return st[t * 4 + ((lane & 3) ^ ((t >> 2) & 3))];
}
// Stores are written as assembly so that the compiler's wait-count bookkeeping sees loads only: with stores pending next to
// loads it stops counting and waits for everything (vmcnt 0) at the next use of a load, which exposes the latency of the whole
// weight prefetch.  Its counts stay safe: it may wait for more operations than needed, never fewer (loads return in issue
// order among themselves).
__device__ __forceinline__ void mlp_store16(bf16_t* p, const mlp_u32x4& v) {
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
}

// bias, optional GELU, optional residual of one 32 x 32 accumulator: register 4b + i of lane (token, hf) is row
// 8b + 4 hf + i of the block; one v_permlane32_swap per value pair gives the lane eight consecutive rows (run
// 2 gp + hf of the block's four), packed to bf16 in outv[gp]
__device__ __forceinline__ mlp_u32x4 mlp_finish_half(const mlp_f32x16& h, int gp, const mlp_u32x4& bias, const mlp_u32x4& res, bool gelu_on) {
  float v[8], bb[8], rr[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(h[8 * gp + q]), __float_as_uint(h[8 * gp + 4 + q]), false, false);
    v[q] = __uint_as_float(sw[0]);
    v[4 + q] = __uint_as_float(sw[1]);
  }
  mlp_unpack8(bias, bb);
  mlp_unpack8(res, rr);
  mlp_u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = v[2 * e] + bb[2 * e], b = v[2 * e + 1] + bb[2 * e + 1];
    const float ga = gelu_poly(a), gb = gelu_poly(b);
    a = gelu_on ? ga : a;
    b = gelu_on ? gb : b;
    o[e] = mlp_pack2(a + rr[2 * e], b + rr[2 * e + 1]);
  }
  return o;
}
// ... and back: an accumulator that starts from the block's values instead of zeros (the residual of a sum of products needs
// no registers of its own then)
__device__ __forceinline__ void mlp_start_from(mlp_f32x16& h, const mlp_u32x4 (&v)[2]) {
#pragma unroll
  for (int gp = 0; gp < 2; ++gp) {
    float f[8];
    mlp_unpack8(v[gp], f);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(f[q]), __float_as_uint(f[4 + q]), false, false);
      h[8 * gp + q] = __uint_as_float(sw[0]);
      h[8 * gp + 4 + q] = __uint_as_float(sw[1]);
    }
  }
}
__device__ __forceinline__ void mlp_finish(const mlp_f32x16& h, const mlp_u32x4& bias_v, const mlp_u32x4& bias_w, const mlp_u32x4* res,
                                           bool gelu_on, mlp_u32x4* outv) {
#pragma unroll
  for (int gp = 0; gp < 2; ++gp) outv[gp] = mlp_finish_half(h, gp, gp ? bias_w : bias_v, res[gp], gelu_on);
}

// an accumulator that starts from the biases of its 32 rows (four slots of eight, bf16, LDS)
__device__ __forceinline__ void mlp_start_bias(mlp_f32x16& h, const mlp_u32x4* bias, int hf) {
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint2 v = ((const uint2*)(bias + b))[hf];
    h[4 * b] = __uint_as_float(v.x << 16); h[4 * b + 1] = __uint_as_float(v.x & 0xffff0000u);
    h[4 * b + 2] = __uint_as_float(v.y << 16); h[4 * b + 3] = __uint_as_float(v.y & 0xffff0000u);
  }
}
// four pairs of packed values (rows 8 b + 4 hf .. + 3 of b = 2 gp, 2 gp + 1) -> the lane's run of eight rows, 2 gp + hf
__device__ __forceinline__ mlp_u32x4 mlp_run8(const unsigned (&pk)[4]) {
  const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
  return mlp_u32x4{s0[0], s1[0], s0[1], s1[1]};
}
template <typename Act> __device__ __forceinline__ mlp_u32x4 mlp_run(const mlp_f32x16& h, int gp, Act act) {
  unsigned pk[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) pk[i] = mlp_pack2(act(h[8 * gp + 2 * i]), act(h[8 * gp + 2 * i + 1]));
  return mlp_run8(pk);
}
// acc += the wave's fragments wf x a 32-token tile in LDS (slot `at`: the lane's first of its row).  The order of issue is pinned
// (a fence behind every step): the MFMA, the refill of its weight register with what refill(kk) asks for, and the tile's
// fragment three steps ahead
template <int KK, typename Refill>
__device__ __forceinline__ void mlp32_product(const mlp_u32x4* tile, int at, mlp_u32x4 (&wf)[KK], mlp_f32x16& acc, Refill refill) {
  asm volatile("" : "+v"(at));                          // opaque per call: the tile's fragments are re-read from LDS instead of being
  mlp_u32x4 fb[3] = {tile[at], tile[at + 2], tile[at + 4]};      // hoisted into (and spilled from) registers
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(mlp_bf16x8, wf[kk]), __builtin_bit_cast(mlp_bf16x8, fb[kk % 3]), acc, 0, 0, 0);
    wf[kk] = refill(kk);
    if (kk + 3 < KK) fb[kk % 3] = tile[at + 2 * (kk + 3)];
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// vectors of C elements beside b1 in the kernel's LDS: b2; bproj, gamma, beta; gamma, beta of the second output; bq (three)
constexpr int mlp_vectors(bool proj, int lnout) { return 1 + (proj ? 3 : 0) + (lnout ? 2 : 0) + (lnout == 2 ? 3 : 0); }

// PROJ: the Linear that precedes the MLP's residual stream is computed here as well (a transformer block's attention
// output projection): x1 = A . Wp^T + bp + x0 for the tile's 32 tokens, x0 read (and Y written) through y_rows, then
// Y = x1 + MLP(LayerNorm(x1)).  x1 never reaches memory: a normalised copy feeds the first product from LDS, and the
// accumulators of the final sum start from x1 itself.
// LNOUT = 1: a second output, LayerNorm(Y) with its own gamma / beta, stored through its own row map: the norm that opens
// the next block, computed while the rows are still in registers (statistics over the C / 32 waves through LDS).
// LNOUT = 2 (with PROJ): that norm stays in LDS and the Linear that follows it (the next block's QKV, N = 3 C, packed
// like lin_pack_kernel's) runs here too, three slices of 32 outputs per wave, stored through the same row map.
template <int C, bool PROJ, int LNOUT>
__global__ __launch_bounds__(64 * (C / 32), C <= 256 ? 4 : 3) void mlp_fused_kernel(MlpArgs g) {
  constexpr int KK = C / 16;            // 16-wide steps of the first product
  constexpr int T = C / 32;             // 32-row blocks of Y^T = waves of the workgroup
  constexpr int NTHR = 64 * T;
  constexpr int XS = C / 8;             // 16-byte slots per token row
  constexpr int XP = XS + 1;            // odd pitch: the fragment reads of 16 tokens hit 16 different bank groups
  constexpr int HP = 4 * T + 1;         // the same for a round's hidden tile (T slices of 32 = 4 slots each)
  constexpr size_t TILE = (size_t)32 * XP * 16, HTILE = (size_t)32 * HP * 16;
  const SM_KARG MlpArgs* gk = kernarg_ptr<MlpArgs>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // [A tile (PROJ) | X tile | H x 2 | b1 | b2 | bproj, gamma, beta (PROJ) | gamma, beta of the second output | bq | row offsets | statistics]
  mlp_u32x4* a_l = (mlp_u32x4*)smem_raw;
  mlp_u32x4* x_l = (mlp_u32x4*)(smem_raw + (PROJ ? TILE : 0));            // [32][XP]; PROJ: x0, then x1 normalised
  mlp_u32x4* h_l = (mlp_u32x4*)(smem_raw + (PROJ ? 2 : 1) * TILE);        // [2][32][HP]
  mlp_u32x4* b1_l = (mlp_u32x4*)(smem_raw + (PROJ ? 2 : 1) * TILE + 2 * HTILE);   // [Hd / 8]
  mlp_u32x4* vec_l = b1_l + g.Hd / 8;                                     // [NV][XS]
  constexpr int V_BP = 1, V_G1 = 2, V_E1 = 3, V_G2 = PROJ ? 4 : 1, V_E2 = V_G2 + 1, V_BQ = V_E2 + 1;   // (b2 first)
  constexpr int NV = mlp_vectors(PROJ, LNOUT);
  int64_t* ro_l = (int64_t*)(vec_l + NV * XS);                            // [2][32]: of Y and of the second output; -1 past M
  float2* st_l = (float2*)(ro_l + 64);                                    // [T][32] row statistics

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave index as a scalar: fragment bases become scalar addresses
  const int64_t row0 = (int64_t)blockIdx.x * 32;
  const int Hd = g.Hd;
  const int nsub = Hd >> 5;
  const int rounds = (nsub + T - 1) / T;
  // Weight fragments (1 KiB each, see the file header) are fetched with buffer loads: the descriptor and the fragment's
  // offset are scalar, the only vector operand is the lane's 16 bytes within the fragment, so no address arithmetic
  // touches the vector registers (and a fragment index past the end would read zeros instead of faulting).
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wp), 0, 4 * Hd * C, 0x00020000);
  const int W2o = 2 * Hd * C + w * nsub * 2048;                           // byte offset of this wave's W2 row block: (slice, step) in order
  const int lo = lane * 16;
  auto wload = [&](const __amdgpu_buffer_rsrc_t& r, int soff) __attribute__((always_inline)) { return __builtin_amdgcn_raw_buffer_load_b128(r, lo, soff, 0); };

  // One set of C / 16 fragment registers carries the whole weight stream of the wave: a product of C / 16 MFMAs
  // consumes them in order, and each is refilled, right after the MFMA that read it, with the fragment the NEXT
  // product needs at the same position (first product -> this round's W2 fragments -> next round's W1 slice -> ...):
  // every load has a full product to arrive and the compiler's wait is one constant count.
  mlp_u32x4 wf[KK];
  const int sc0 = w < nsub ? w : nsub - 1;      // (a wave past the last slice works on a copy of it and contributes zeros)
  __amdgpu_buffer_rsrc_t rp = rw, rq = rw;
  if constexpr (PROJ) rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wproj_p), 0, 2 * C * C, 0x00020000);
  if constexpr (LNOUT == 2) rq = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wq_p), 0, 6 * C * C, 0x00020000);

  // Everything the tile needs from memory is requested before anything is waited for, in the order of its use (loads return in the
  // order they were asked for): the tile, the row offsets and vectors, the weight stream, and behind its first fragments PROJ's
  // residual x0 (through y_rows), which has the projection to arrive in
  MlpTile<C, NTHR, 32> xt, rt;
  if constexpr (PROJ) rt.rows(row0, g.M, g.y_rows.identity, g.y_rows.ld, &gk->y_rows);
  xt.request((const bf16_t*)g.X, row0, g.M, g.x_rows.identity, g.x_rows.ld, &gk->x_rows);
  if (tid < 32 || (LNOUT != 0 && tid < 64)) {
    const int64_t row = row0 + (tid & 31), prow = row < g.M ? row : g.M - 1;
    int64_t o;
    if (LNOUT == 0 || tid < 32) o = g.y_rows.identity ? prow * g.y_rows.ld : eval_rows_k(&gk->y_rows, prow);
    else o = g.y2_rows.identity ? prow * g.y2_rows.ld : eval_rows_k(&gk->y2_rows, prow);
    ro_l[tid] = row < g.M ? o : -1;
  }
  for (int s = tid; s < Hd / 8; s += NTHR) b1_l[s] = ((const mlp_u32x4*)g.b1)[s];
  if (tid < XS) {
    mlp_u32x4 v[6];
    v[0] = ((const mlp_u32x4*)g.b2)[tid];
    if constexpr (PROJ) {
      v[V_BP] = ((const mlp_u32x4*)g.bproj)[tid];
      v[V_G1] = v[V_E1] = mlp_u32x4{0u, 0u, 0u, 0u};
      if (g.norm) { v[V_G1] = ((const mlp_u32x4*)g.norm_gamma)[tid]; v[V_E1] = ((const mlp_u32x4*)g.norm_beta)[tid]; }
    }
    if constexpr (LNOUT != 0) { v[V_G2] = ((const mlp_u32x4*)g.ln2_gamma)[tid]; v[V_E2] = ((const mlp_u32x4*)g.ln2_beta)[tid]; }
#pragma unroll
    for (int i = 0; i < (LNOUT == 2 ? V_BQ : NV); ++i) vec_l[i * XS + tid] = v[i];
  }
  if constexpr (LNOUT == 2) for (int s = tid; s < 3 * XS; s += NTHR) vec_l[V_BQ * XS + s] = ((const mlp_u32x4*)g.bq)[s];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) wf[kk] = PROJ ? wload(rp, (w * KK + kk) * 1024) : wload(rw, (sc0 * KK + kk) * 1024);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (PROJ) rt.load((const bf16_t*)g.resid0);
  __builtin_amdgcn_sched_barrier(0);
  xt.store(PROJ ? a_l : x_l, row0, g.M);
  __syncthreads();

  const mlp_u32x4 zero4[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
  const int fs = w * 4 + hf;                                              // first of the lane's two feature slots (the other: fs + 2)
  const int xs = l32 * XP + fs;

  mlp_f32x16 out;
#pragma unroll
  for (int e = 0; e < 16; ++e) out[e] = 0.f;
  if constexpr (PROJ) {
    // wave w forms features 32 w ..+31 of x1
    mlp_f32x16 h;
#pragma unroll
    for (int e = 0; e < 16; ++e) h[e] = 0.f;
    mlp32_product(a_l, l32 * XP + hf, wf, h, [&](int kk) __attribute__((always_inline)) { return wload(rw, (sc0 * KK + kk) * 1024); });
    rt.store(x_l, row0, g.M);
    __syncthreads();
    const mlp_u32x4 res[2] = {x_l[xs], x_l[xs + 2]};           // x0, of which every lane reads the slots that it overwrites below
    mlp_u32x4 x1[1][2];
    mlp_finish(h, vec_l[V_BP * XS + fs], vec_l[V_BP * XS + fs + 2], res, false, x1[0]);          // x1 rounded to bf16, as the separate Linear stores it
    mlp_start_from(out, x1[0]);
    if (g.norm) {
      mlp_stats_put<1>(x1, hf, st_l + w * 32 + l32);
      __syncthreads();
      float rstd, sh;
      mlp_stats_get<1, T>(st_l + l32, 32, g.norm_eps, &rstd, &sh);
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) x_l[xs + 2 * gp] = mlp_scale8(x1[0][gp], rstd, sh, vec_l[V_G1 * XS + fs + 2 * gp], vec_l[V_E1 * XS + fs + 2 * gp]);
    } else {
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) x_l[xs + 2 * gp] = x1[0][gp];
    }
    __syncthreads();
  } else if (g.norm) {
    mlp_norm_x_tile<C, NTHR, 32>(x_l, g.norm_eps, (const mlp_u32x4*)g.norm_gamma, (const mlp_u32x4*)g.norm_beta);
    __syncthreads();
  }

  {
  const int lane = mlp_lane(), l32 = lane & 31, hf = lane >> 5;
  for (int r = 0; r < rounds; ++r) {
    // ---- first product: this wave's slice of the round -> H (bias, GELU, bf16) into LDS
    const int sc = r * T + w;
    const bool sc_ok = sc < nsub;
    const int scc = sc_ok ? sc : nsub - 1;
    const int nsc = sc + T < nsub ? sc + T : scc;
    const int s0 = r * T;                                // first slice of the round
    const int rem = nsub - s0;                           // slices of W2 from this round's first to the end (>= 1)
    const int cur2 = W2o + s0 * 2048;                    // scalar: this round's W2 fragments of this wave, (slice, step) in order
    mlp_f32x16 h;
    mlp_start_bias(h, b1_l + scc * 4, hf);
    // refills: the second product's fragments of this round; past the end of W2 the last valid pair again (its H is zero)
    mlp32_product(x_l, l32 * XP + hf, wf, h, [&](int kk) __attribute__((always_inline)) { return wload(rw, cur2 + (kk < 2 * rem ? kk : (kk & 1) + 2 * (rem - 1)) * 1024); });
    mlp_u32x4* hb = h_l + (r & 1) * (32 * HP);
#pragma unroll
    for (int gp = 0; gp < 2; ++gp) {
      const mlp_u32x4 hv = mlp_run(h, gp, gelu_poly);
      hb[l32 * HP + w * 4 + 2 * gp + hf] = sc_ok ? hv : zero4[0];     // past the last slice: zeros
    }
    __syncthreads();
    // ---- second product: this wave's 32 output features over the round's T slices.  One barrier per round: the
    // other H buffer is written next, and nobody writes this one again before the barrier after that
    // what follows in the stream: the wave's slice of the next round; after the last the Linear that follows, or nothing (a descriptor
    // of no bytes: zeros, without a look at memory)
    const bool last = r + 1 == rounds;
    const __amdgpu_buffer_rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(LNOUT == 2 && last ? g.Wq_p : g.Wp), 0,
                                                                        last ? (LNOUT == 2 ? 6 * C * C : 0) : 4 * Hd * C, 0x00020000);
    const int next = (LNOUT == 2 && last ? w : nsc) * KK * 1024;
    mlp32_product(hb, l32 * HP + hf, wf, out, [&](int i) __attribute__((always_inline)) { return wload(rn, next + i * 1024); });
  }
  }

  {
  // every wave holds its 32 features of Y^T complete: bias, residual, and out in 64-byte pieces through the wave's 2 KiB of
  // the X tile (nobody has read that since the last barrier)
  const int lane = mlp_lane(), l32 = lane & 31, hf = lane >> 5, fs = w * 4 + hf, xs = l32 * XP + fs;
  mlp_u32x4* stage = x_l + w * 128;
  auto emit = [&](bf16_t* base, int scale, const int64_t* ro, int col, const mlp_u32x4& v0, const mlp_u32x4& v1) __attribute__((always_inline)) {
    mlp_stage_put(stage, l32, hf, v0, v1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const mlp_u32x4 v = mlp_stage_get(stage, lane, i);
      const int64_t o = ro[16 * i + (lane >> 2)];
      if (o >= 0) mlp_store16(base + o * scale + col + (lane & 3) * 8, v);
    }
  };
  mlp_u32x4 resid[2] = {zero4[0], zero4[0]};              // (PROJ: x1, which the sum started from)
  if constexpr (!PROJ) {
    if (g.residual) {          // (asked for here, not before the rounds: eight more live registers there mean spills)
      const int64_t o = ro_l[l32];
      const bf16_t* R = (const bf16_t*)g.residual + (o < 0 ? ro_l[0] : o);      // (lanes past M: the tile's first row)
      resid[0] = *(const mlp_u32x4*)(R + fs * 8);
      resid[1] = *(const mlp_u32x4*)(R + fs * 8 + 16);
    }
  }
  mlp_u32x4 yv[1][2];
  mlp_finish(out, vec_l[fs], vec_l[fs + 2], resid, false, yv[0]);
  if constexpr (LNOUT != 0) mlp_stats_put<1>(yv, hf, st_l + w * 32 + l32);
  emit((bf16_t*)g.Y, 1, ro_l, w * 32, yv[0][0], yv[0][1]);
  if constexpr (LNOUT != 0) {
    // LayerNorm of the bf16 row, as the norm kernel would compute it from the stored Y
    __syncthreads();
    float rstd, sh;
    mlp_stats_get<1, T>(st_l + l32, 32, g.ln2_eps, &rstd, &sh);
    mlp_u32x4 nv[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) nv[q] = mlp_scale8(yv[0][q], rstd, sh, vec_l[V_G2 * XS + fs + 2 * q], vec_l[V_E2 * XS + fs + 2 * q]);
    if constexpr (LNOUT == 1) {
      emit((bf16_t*)g.Y2, 1, ro_l + 32, w * 32, nv[0], nv[1]);
    } else {
      static_assert(LNOUT != 2 || PROJ, "the fused following Linear needs the projection variant's spare LDS tile");
      // the normalised tile (bf16, as a norm kernel would have stored it) into the A tile's LDS, dead since the projection; then
      // wave w forms outputs 32 (w + T j) ..+31, j < 3
      mlp_u32x4* n_l = a_l;
      n_l[xs] = nv[0];
      n_l[xs + 2] = nv[1];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int sc = w + T * j;
        mlp_f32x16 h;
        mlp_start_bias(h, vec_l + V_BQ * XS + sc * 4, hf);
        mlp32_product(n_l, l32 * XP + hf, wf, h, [&](int kk) __attribute__((always_inline)) { return j < 2 ? wload(rq, ((sc + T) * KK + kk) * 1024) : wf[kk]; });
        const auto same = [](float a) __attribute__((always_inline)) { return a; };
        const mlp_u32x4 qv[2] = {mlp_run(h, 0, same), mlp_run(h, 1, same)};
        emit((bf16_t*)g.Y2, 3, ro_l + 32, sc * 32, qv[0], qv[1]);        // same row map, rows three times as long
      }
    }
  }
  }
}

// What the 64-token kernels have in common.  The order in which a step's instructions are issued is pinned (a fence behind every
// step, groups inside): an MFMA keeps the matrix pipe for eight issue slots, the vector work (`piece`, a step's share of it) goes
// into the slots behind each, a weight register is asked for again right behind its last MFMA, and the tile's fragments are read
// two steps ahead.  Left alone the compiler gathers the refills at the end of a phase, reads each fragment right before its MFMA
// and puts the vector work of a phase in one piece, in which the matrix pipe idles (mlp64p_kernel<512, 2>, 196 workgroups, weights
// in the caches: rounds 86 -> 71 thousand clocks, of which the MFMAs take 57, QKV 32 -> 25, of 24; 88 -> 80 us).
template <int VALU> __device__ __forceinline__ void mlp64_mfma_order() {
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
  if constexpr (VALU > 0) __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
}
// out[bt][tb] += W(step i, feature block bt) x tile(token block tb, step i) for STEPS steps: the wave's 64 features against a
// 64-token tile in LDS (row pitch `pitch` slots); refill(t) loads the fragment at position t of the call's stream (t >= 2 STEPS:
// what follows it).
template <int STEPS, int VALU, int RING, typename Refill, typename Piece>
__device__ __forceinline__ void mlp64_pair(const mlp_u32x4* tile, int pitch, int l32, int hf, mlp_u32x4 (&wf)[RING], mlp_f32x16 (&out)[2][2],
                                           Refill refill, Piece piece) {
  int to = l32 * pitch + hf;
  asm volatile("" : "+v"(to));                          // opaque per call: the tile's fragments are re-read, not hoisted
  const int hi = 32 * pitch;
  mlp_u32x4 ga[2][2] = {{tile[to], tile[to + hi]}, {tile[to + 2], tile[to + 2 + hi]}};
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < STEPS; ++i) {
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) {
      const int t = 2 * i + bt;
      const mlp_bf16x8 wv = __builtin_bit_cast(mlp_bf16x8, wf[t % RING]);
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) out[bt][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, __builtin_bit_cast(mlp_bf16x8, ga[i & 1][tb]), out[bt][tb], 0, 0, 0);
      wf[t % RING] = refill(t + RING);
    }
    if (i + 2 < STEPS) { ga[i & 1][0] = tile[to + 2 * (i + 2)]; ga[i & 1][1] = tile[to + 2 * (i + 2) + hi]; }
    piece(i);
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) {
      mlp64_mfma_order<VALU>();
      mlp64_mfma_order<0>();
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      if (bt) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      if constexpr (VALU > 0) __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}
// h[tb] = bias + W(the wave's slice) x tile(token block tb): 32 features of a slice for the 64 tokens.  bias: the slice's four
// slots of eight (bf16, LDS)
template <int KK, int VALU, int RING, typename Refill, typename Piece>
__device__ __forceinline__ void mlp64_slice(const mlp_u32x4* tile, int pitch, int l32, int hf, const mlp_u32x4* bias, mlp_u32x4 (&wf)[RING],
                                            mlp_f32x16 (&h)[2], Refill refill, Piece piece) {
  int xo = l32 * pitch + hf;
  asm volatile("" : "+v"(xo));
  const int hi = 32 * pitch;
  mlp_start_bias(h[0], bias, hf);
  h[1] = h[0];
  mlp_u32x4 fa[2][2] = {{tile[xo], tile[xo + hi]}, {tile[xo + 2], tile[xo + 2 + hi]}};
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const mlp_bf16x8 wv = __builtin_bit_cast(mlp_bf16x8, wf[kk % RING]);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) h[tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, __builtin_bit_cast(mlp_bf16x8, fa[kk & 1][tb]), h[tb], 0, 0, 0);
    wf[kk % RING] = refill(kk + RING);
    if (kk + 2 < KK) { fa[kk & 1][0] = tile[xo + 2 * (kk + 2)]; fa[kk & 1][1] = tile[xo + 2 * (kk + 2) + hi]; }
    piece(kk);
    mlp64_mfma_order<VALU>();
    mlp64_mfma_order<0>();
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    if constexpr (VALU > 0) __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}
// Piece i of n of a slice's way out of its accumulators: the 16 pairs of values are dealt to the pieces, act(a), packed to bf16,
// and every four pairs make one run of eight features (run 2 gp + hf of token 32 tb + l32) by two v_permlane32_swap: put(tb, gp, run)
template <typename Act, typename Put>
__device__ __forceinline__ void mlp64_out_piece(int i, int n, const mlp_f32x16 (&h)[2], unsigned (&pk)[4], Act act, Put put) {
#pragma unroll
  for (int d = 16 * i / n; d < 16 * (i + 1) / n; ++d) {
    const int tb = d >> 3, e = 2 * (d & 7);
    pk[d & 3] = mlp_pack2(act(h[tb][e]), act(h[tb][e + 1]));
    if ((d & 3) == 3) put(tb, (d >> 2) & 1, mlp_run8(pk));
  }
}

// ---------------------------------------------------------------------------------------------------------------
// The fused MLP for wide rows (C = 512): Y = residual + W2 . gelu(W1 . LayerNorm(x) + b1) + b2 with a tile of 64 tokens
// per workgroup and eight waves, each owning 64 output features.  With 32 tokens every weight fragment feeds one MFMA
// and the stream of fragments from L2 sets the pace; here a fragment of W1 feeds two MFMAs (the two token blocks) and
// in the second product two weight fragments and two hidden fragments feed four, so per MFMA half a KiB comes from L2
// and half a KiB from LDS.  Rounds of 256 hidden units: wave w forms slice 8 r + w of the round (32 hidden units x 64
// tokens: bias, GELU, bf16 into the round's hidden tile in LDS, double-buffered, one barrier per round), then adds
// the round to its 64 x 64 block of Y^T.  Same packed weight layout as the kernel above (mlp_pack_kernel).  The weight
// stream of a wave (blocks of 32 fragments: a W1 slice, or a round's W2 fragments in (step, feature block) order) runs
// through a ring of 16 fragment registers: each is refilled, right after the MFMAs that read it, with the fragment 16
// places on.
template <int C>
__global__ __launch_bounds__(C, (C >= 384 ? 1 : 2)) void mlp64_kernel(MlpArgs g) {
  constexpr int KK = C / 16, XS = C / 8, XP = XS + 1, NW = C / 64, NTHR = 64 * NW, RING = KK % 16 == 0 ? 16 : 8;
  constexpr int GV = 48 / NW;                           // vector instructions behind an MFMA of the second product (bias + GELU)
  constexpr int HP = 4 * NW + 1;                        // slots of a token's row of the round's hidden tile (+1: odd pitch)
  constexpr size_t TILE = (size_t)64 * XP * 16, HTILE = (size_t)64 * HP * 16;
  static_assert(C % 64 == 0 && KK % RING == 0 && 4 * NW == KK && NW % 2 == 0, "the ring position of a fragment must be a compile-time constant");
  const SM_KARG MlpArgs* gk = kernarg_ptr<MlpArgs>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  mlp_u32x4* x_l = (mlp_u32x4*)smem_raw;                               // [64][XP] token tile, normalised in place
  mlp_u32x4* h_l = (mlp_u32x4*)(smem_raw + TILE);                      // [2][64][HP]
  mlp_u32x4* b1_l = (mlp_u32x4*)(smem_raw + TILE + 2 * HTILE);         // [Hd / 8]
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  const int Hd = g.Hd, nsub = Hd >> 5, rounds = nsub / NW;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wp), 0, 4 * Hd * C, 0x00020000);
  const int lo = lane * 16;
  auto wload = [&](int soff) __attribute__((always_inline)) { return __builtin_amdgcn_raw_buffer_load_b128(rw, lo, soff, 0); };
  // The wave's weight stream in blocks of 32 fragments: W1 slice of round 0; then, for every further round r, the W1
  // slice of round r followed by the W2 fragments of round r - 1 (step, feature block); last the W2 fragments of the last
  // round.  Byte offset of fragment s of block b (s may run into the next block; past the last block that one again).
  const int last_blk = 2 * rounds - 1;
  auto foff = [&](int b, int s) __attribute__((always_inline)) -> int {
    if (s >= KK) { b += 1; s -= KK; }
    b = b < last_blk ? b : last_blk;
    const bool w2 = b == last_blk || (b != 0 && !(b & 1));
    const int rr = b == last_blk ? rounds - 1 : (b & 1 ? (b + 1) >> 1 : (b ? (b >> 1) - 1 : 0));
    return w2 ? 2 * Hd * C + (((2 * w + (s & 1)) * nsub + NW * rr) * 2 + (s >> 1)) * 1024 : ((NW * rr + w) * KK + s) * 1024;
  };
  mlp_u32x4 wf[RING];
#pragma unroll
  for (int s = 0; s < RING; ++s) wf[s] = wload(foff(0, s));

  // the lane's two token rows (one per token block): offsets for the residual and the store
  int64_t ro[2]; bool row_ok[2];
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    const int64_t row = row0 + 32 * tb + l32;
    row_ok[tb] = row < g.M;
    const int64_t prow = row_ok[tb] ? row : g.M - 1;
    ro[tb] = g.y_rows.identity ? prow * g.y_rows.ld : eval_rows_k(&gk->y_rows, prow);
  }
  MlpTile<C, NTHR, 64> xt;
  xt.request((const bf16_t*)g.X, row0, g.M, g.x_rows.identity, g.x_rows.ld, &gk->x_rows);
  xt.store(x_l, row0, g.M);
  for (int s = tid; s < Hd / 8; s += NTHR) b1_l[s] = ((const mlp_u32x4*)g.b1)[s];
  __syncthreads();
  if (g.norm) {
    mlp_norm_x_tile<C, NTHR, 64>(x_l, g.norm_eps, (const mlp_u32x4*)g.norm_gamma, (const mlp_u32x4*)g.norm_beta);
    __syncthreads();
  }

  mlp_f32x16 out[2][2];                                 // [feature block][token block]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) out[i >> 1][i & 1][e] = 0.f;

  // bias + GELU of the slice just formed, bf16, into the round's hidden tile, a piece per step of the second product of the round
  // before: both depend on the last barrier only
  unsigned pk[4];
  auto gelu_piece = [&](int i, int n, const mlp_f32x16 (&h)[2], mlp_u32x4* hb) __attribute__((always_inline)) {
    mlp64_out_piece(i, n, h, pk, gelu_poly, [&](int tb, int gp, const mlp_u32x4& v) __attribute__((always_inline)) {
      hb[(32 * tb + l32) * HP + w * 4 + 2 * gp + hf] = v;
    });
  };
  auto nothing = [&](int) __attribute__((always_inline)) {};
  {
    mlp_f32x16 h[2];
    mlp64_slice<KK, 0>(x_l, XP, l32, hf, b1_l + w * 4, wf, h, [&](int s) __attribute__((always_inline)) { return wload(foff(0, s)); }, nothing);
    gelu_piece(0, 1, h, h_l);
    __syncthreads();
    for (int r = 1; r < rounds; ++r) {
      mlp64_slice<KK, 0>(x_l, XP, l32, hf, b1_l + (NW * r + w) * 4, wf, h, [&](int s) __attribute__((always_inline)) { return wload(foff(2 * r - 1, s)); }, nothing);
      mlp_u32x4* hb = h_l + (r & 1) * (64 * HP);
      mlp64_pair<2 * NW, GV>(h_l + ((r - 1) & 1) * (64 * HP), HP, l32, hf, wf, out, [&](int s) __attribute__((always_inline)) { return wload(foff(2 * r, s)); },
                             [&](int i) __attribute__((always_inline)) { gelu_piece(i, 2 * NW, h, hb); });
      __syncthreads();
    }
    mlp64_pair<2 * NW, 0>(h_l + ((rounds - 1) & 1) * (64 * HP), HP, l32, hf, wf, out, [&](int s) __attribute__((always_inline)) { return wload(foff(last_blk, s)); }, nothing);
  }

  // every wave holds its 64 features of Y^T for the 64 tokens: bias, residual, two 16-byte stores per block and lane
  bf16_t* Y = (bf16_t*)g.Y;
  const bf16_t* R = (const bf16_t*)g.residual;
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) {
    const int fo = (2 * w + bt) * 32 + hf * 8;
    const mlp_u32x4 b2v = *(const mlp_u32x4*)((const bf16_t*)g.b2 + fo), b2w = *(const mlp_u32x4*)((const bf16_t*)g.b2 + fo + 16);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      mlp_u32x4 resid[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
      if (R) { resid[0] = *(const mlp_u32x4*)(R + ro[tb] + fo); resid[1] = *(const mlp_u32x4*)(R + ro[tb] + fo + 16); }
      mlp_u32x4 yv[2];
      mlp_finish(out[bt][tb], b2v, b2w, resid, false, yv);
      if (row_ok[tb]) {
        *(mlp_u32x4*)(Y + ro[tb] + fo) = yv[0];
        *(mlp_u32x4*)(Y + ro[tb] + fo + 16) = yv[1];
      }
    }
  }
}

// mlp64_kernel with the attention output projection in front and, optionally, the next block's LayerNorm-1 (LNOUT = 1)
// or LayerNorm-1 + QKV Linear (LNOUT = 2) behind it: the C = 512 form of mlp_fused_kernel<C, true, LNOUT>, 64-token
// tiles.  x1 = A . Wproj^T + bproj + x0 (x0 read and Y written through y_rows).  The accumulators of the final sum start from x1
// (rounded to bf16); normalised it goes to LDS for the first product.  LDS: [x0, then x1 normalised, then the waves' stages of
// mlp_stage_put | A tile, then the two hidden tiles, then the normalised Y for the QKV Linear | b1, then bq | row offsets |
// row statistics | vectors, where there is room].
// One weight stream per wave through the ring of 16 fragment registers, in blocks of 32 fragments: two blocks of Wproj
// ((step, feature block) order, the wave's two slices of lin_pack_kernel's layout), the blocks of mlp64_kernel, then
// the wave's six QKV slices.
template <int C, int LNOUT>
__global__ __launch_bounds__(C, (C >= 384 ? 1 : 2)) void mlp64p_kernel(MlpArgs g, int vec_lds) {
  constexpr int KK = C / 16, XS = C / 8, XP = XS + 1, NW = C / 64, NTHR = 64 * NW, RING = KK % 16 == 0 ? 16 : 8, HP = 4 * NW + 1, NQ = 3 * C / 32 / NW;
  constexpr int GV = 48 / NW;                           // vector instructions behind an MFMA of the second product (bias + GELU)
  constexpr size_t TILE = (size_t)64 * XP * 16, HTILE = (size_t)64 * HP * 16;
  static_assert(C % 64 == 0 && KK % RING == 0 && 4 * NW == KK && NW % 2 == 0 && 2 * HTILE >= TILE, "block and alias assumptions");
  const SM_KARG MlpArgs* gk = kernarg_ptr<MlpArgs>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  mlp_u32x4* x_l = (mlp_u32x4*)smem_raw;                               // [64][XP] x1, normalised in place
  mlp_u32x4* a_l = (mlp_u32x4*)(smem_raw + TILE);                      // [64][XP] attention output; dead after the projection
  mlp_u32x4* h_l = a_l;                                                // [2][64][HP] hidden tiles
  mlp_u32x4* n_l = a_l;                                                // [64][XP] normalised Y (LNOUT = 2), after the last round
  mlp_u32x4* b1_l = (mlp_u32x4*)(smem_raw + TILE + 2 * HTILE);         // [Hd / 8], later bq [3 C / 8]
  int64_t* ro_l = (int64_t*)(b1_l + g.Hd / 8);                         // [2][64]: of Y and of the second output; -1 past M
  float2* st_l = (float2*)(ro_l + 128);                                // [NW][64] row statistics
  mlp_u32x4* vec_l = (mlp_u32x4*)(st_l + NW * 64);                     // vec_lds: [NV][C / 8], else read from memory where they are used
  constexpr int NV = LNOUT != 0 ? 6 : 4;                               // bproj, gamma, beta, b2, gamma and beta of the second output
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  const int Hd = g.Hd, nsub = Hd >> 5, rounds = nsub / NW;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wp), 0, 4 * Hd * C, 0x00020000);
  const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wproj_p), 0, 2 * C * C, 0x00020000);
  const __amdgpu_buffer_rsrc_t rq = LNOUT == 2 ? __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wq_p), 0, 6 * C * C, 0x00020000) : rw;
  const int lo = lane * 16;
  // In a net the weights of a block have left the caches when it runs, and all workgroups ask for the same ones at the same time:
  // the ring (about 2000 clocks ahead) does not cover memory.  So the workgroups of an XCD bring every chunk of the stream (Wproj;
  // a round of W1 and W2; a third of the QKV weight: 2 C^2 bytes each) into its L2 two to three rounds ahead, a word of every
  // 128-byte line, two lines a lane.  Workgroups behind the first 256 find what those have brought (C = 256: all of it fits).
  // 12544 tokens of C = 512 in a net of 24 blocks, mean of its 17 launches: 110.7 -> 93.9 us, every MFMA phase in as many clocks as with
  // warm caches.
  constexpr int CHUNK_LOADS = C * C * 2 / 8192;         // of 64 lines
  const int pf_waves = ((min((int)gridDim.x, 256) + 7) >> 3) * NW, pf_wave = blockIdx.x < 256 ? (int)(blockIdx.x >> 3) * NW + w : CHUNK_LOADS;
  unsigned pf[2] = {0u, 0u};
  auto prefetch = [&](int chunk) __attribute__((always_inline)) {
    if (chunk >= 1 + rounds + (LNOUT == 2 ? 3 : 0)) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      asm volatile("" ::"v"(pf[i]));                    // (the last one has long arrived)
      if (pf_wave + i * pf_waves >= CHUNK_LOADS) continue;
      const int at = (pf_wave + i * pf_waves) * 8192 + lane * 128;
      if (chunk == 0) pf[i] = __builtin_amdgcn_raw_buffer_load_b32(rp, at, 0, 0);
      else if (chunk <= rounds) {
        constexpr int HALF = C * C, ROW = 2 * NW * 1024;      // bytes of a round of W1 (in one run), of one feature block's part of a round of W2
        const int q = at - HALF, rr = chunk - 1;
        pf[i] = __builtin_amdgcn_raw_buffer_load_b32(rw, q < 0 ? rr * HALF + at : 2 * Hd * C + q / ROW * (nsub * 2048) + rr * ROW + q % ROW, 0, 0);
      } else pf[i] = __builtin_amdgcn_raw_buffer_load_b32(rq, at, (chunk - 1 - rounds) * (2 * C * C), 0);
    }
  };
  prefetch(0); prefetch(1); prefetch(2);
  // The wave's stream: 64 fragments of Wproj ((step, feature block) order), the MLP's blocks of 32 (see mlp64_kernel),
  // then NQ blocks of the QKV weight.  Which weight a refill reads is known where it is written, so each kind has its
  // own loader (descriptor and offset scalar) and the MFMA loops stay straight-line code.
  const int lastm = 2 * rounds - 1;
  auto frag_p = [&](int t) __attribute__((always_inline)) {          // t < 64: step t / 2, feature block t % 2
    return __builtin_amdgcn_raw_buffer_load_b128(rp, lo, ((2 * w + (t & 1)) * KK + (t >> 1)) * 1024, 0);
  };
  auto frag_m = [&](int m, int s) __attribute__((always_inline)) {   // fragment s of MLP block m (s >= KK: of block m + 1)
    if (s >= KK) { m += 1; s -= KK; }
    m = m < lastm ? m : lastm;
    const bool w2 = m == lastm || (m != 0 && !(m & 1));
    const int rr = m == lastm ? rounds - 1 : (m & 1 ? (m + 1) >> 1 : (m ? (m >> 1) - 1 : 0));
    return __builtin_amdgcn_raw_buffer_load_b128(rw, lo, w2 ? 2 * Hd * C + (((2 * w + (s & 1)) * nsub + NW * rr) * 2 + (s >> 1)) * 1024
                                                            : ((NW * rr + w) * KK + s) * 1024, 0);
  };
  auto frag_q = [&](int j, int s) __attribute__((always_inline)) {   // fragment s of the wave's j-th QKV slice
    if (s >= KK) { j += 1; s -= KK; }
    j = j < NQ ? j : NQ - 1;
    return __builtin_amdgcn_raw_buffer_load_b128(rq, lo, ((w + NW * j) * KK + s) * 1024, 0);
  };
  // The tile is requested first, then the weight stream, the residual x0 (through y_rows) behind its first fragments: loads return in
  // the order they were asked for, and x0 has the projection to arrive in.  One workgroup per CU has nothing to run beside its row phases, in which the matrix cores wait: tile,
  // projection's epilogue, both norms and Y took 23 of the 96 us of 12544 x 512 with the next QKV
  MlpTile<C, NTHR, 64> xt, rt;
  rt.rows(row0, g.M, g.y_rows.identity, g.y_rows.ld, &gk->y_rows);
  xt.request((const bf16_t*)g.X, row0, g.M, g.x_rows.identity, g.x_rows.ld, &gk->x_rows);
  if (tid < (LNOUT != 0 ? 128 : 64)) {
    const int64_t row = row0 + (tid & 63), prow = row < g.M ? row : g.M - 1;
    int64_t o;
    if (LNOUT == 0 || tid < 64) o = g.y_rows.identity ? prow * g.y_rows.ld : eval_rows_k(&gk->y_rows, prow);
    else o = g.y2_rows.identity ? prow * g.y2_rows.ld : eval_rows_k(&gk->y2_rows, prow);
    ro_l[tid] = row < g.M ? o : -1;
  }
  for (int s = tid; s < Hd / 8; s += NTHR) b1_l[s] = ((const mlp_u32x4*)g.b1)[s];
  mlp_u32x4 wf[RING];
#pragma unroll
  for (int s = 0; s < RING; ++s) wf[s] = frag_p(s);
  __builtin_amdgcn_sched_barrier(0);
  rt.load((const bf16_t*)g.resid0);
  __builtin_amdgcn_sched_barrier(0);
  // vector i of C elements: a lane's slots are those of blocks 2 w + bt, runs 2 gp + hf
  auto vec = [&](int i) __attribute__((always_inline)) -> const mlp_u32x4* {
    return (const mlp_u32x4*)(i == 0 ? g.bproj : i == 1 ? g.norm_gamma : i == 2 ? g.norm_beta : i == 3 ? g.b2 : i == 4 ? g.ln2_gamma : g.ln2_beta);
  };
  typedef mlp_u32x4 Slots[2][2];
  const int fs = w * 8 + hf;
  auto slots = [&](Slots& v, int i) __attribute__((always_inline)) {
    if (vec_lds) {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k >> 1][k & 1] = vec_l[i * XS + fs + 2 * k];
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k >> 1][k & 1] = vec(i)[fs + 2 * k];
    }
  };
  if (vec_lds && tid < XS) {
    mlp_u32x4 v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = vec(i)[tid];
#pragma unroll
    for (int i = 0; i < NV; ++i) vec_l[i * XS + tid] = v[i];
  }
  xt.store(a_l, row0, g.M);
  __syncthreads();

  mlp_f32x16 out[2][2];                                 // [feature block][token block]: the projection, then Y^T
  const mlp_u32x4 zero4[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
  auto nothing = [&](int) __attribute__((always_inline)) {};
  // ---- projection: x1 = A . Wproj^T + bproj + x0 for the wave's 64 features
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) out[i >> 1][i & 1][e] = 0.f;
  mlp64_pair<KK, 0>(a_l, XP, l32, hf, wf, out, [&](int t) __attribute__((always_inline)) { return t < 2 * KK ? frag_p(t) : frag_m(0, t - 2 * KK); }, nothing);
  rt.store(x_l, row0, g.M);
  __syncthreads();
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    mlp_u32x4 x1[2][2];
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) {
      mlp_u32x4* x0 = x_l + (32 * tb + l32) * XP + fs + 4 * bt;           // (a lane's own slots: x0, x1, x1 normalised)
      const mlp_u32x4 res[2] = {x0[0], x0[2]};
      mlp_u32x4 bp[2];
      if (vec_lds) { bp[0] = vec_l[fs + 4 * bt]; bp[1] = vec_l[fs + 4 * bt + 2]; } else { bp[0] = vec(0)[fs + 4 * bt]; bp[1] = vec(0)[fs + 4 * bt + 2]; }
      mlp_finish(out[bt][tb], bp[0], bp[1], res, false, x1[bt]);          // x1 rounded to bf16, as the separate Linear stores it
      mlp_start_from(out[bt][tb], x1[bt]);
      x0[0] = x1[bt][0]; x0[2] = x1[bt][1];
      __builtin_amdgcn_sched_barrier(0);                                  // (one block at a time: together they spill)
    }
    mlp_stats_put<2>(x1, hf, st_l + w * 64 + 32 * tb + l32);
    __builtin_amdgcn_sched_barrier(0);
  }
  // (rows of the norm: a lane's runs get(tb, bt) -> put(tb, bt, normalised runs); their statistics lie in st_l)
  auto normalised = [&](float eps, int vec0, auto get, auto put) __attribute__((always_inline)) {
    Slots gam, bet;
    slots(gam, vec0); slots(bet, vec0 + 1);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      float rstd, sh;
      mlp_stats_get<2, NW>(st_l + 32 * tb + l32, 64, eps, &rstd, &sh);
#pragma unroll
      for (int bt = 0; bt < 2; ++bt)
        put(tb, bt, mlp_scale8(get(tb, bt, 0), rstd, sh, gam[bt][0], bet[bt][0]), mlp_scale8(get(tb, bt, 1), rstd, sh, gam[bt][1], bet[bt][1]));
    }
  };
  auto into = [&](mlp_u32x4* tile) __attribute__((always_inline)) {
    return [=](int tb, int bt, const mlp_u32x4& n0, const mlp_u32x4& n1) __attribute__((always_inline)) {
      mlp_u32x4* t = tile + (32 * tb + l32) * XP + fs + 4 * bt;
      t[0] = n0; t[2] = n1;
    };
  };
  __syncthreads();
  normalised(g.norm_eps, 1, [&](int tb, int bt, int gp) __attribute__((always_inline)) { return x_l[(32 * tb + l32) * XP + fs + 4 * bt + 2 * gp]; }, into(x_l));
  __syncthreads();

  // ---- the MLP's rounds, as in mlp64_kernel (stream blocks 2 ..)
  unsigned pk[4];
  auto gelu_piece = [&](int i, int n, const mlp_f32x16 (&h)[2], mlp_u32x4* hb) __attribute__((always_inline)) {
    mlp64_out_piece(i, n, h, pk, gelu_poly, [&](int tb, int gp, const mlp_u32x4& v) __attribute__((always_inline)) {
      hb[(32 * tb + l32) * HP + w * 4 + 2 * gp + hf] = v;
    });
  };
  {
    mlp_f32x16 h[2];
    prefetch(3);
    mlp64_slice<KK, 0>(x_l, XP, l32, hf, b1_l + w * 4, wf, h, [&](int s) __attribute__((always_inline)) { return frag_m(0, s); }, nothing);
    gelu_piece(0, 1, h, h_l);
    __syncthreads();
    for (int r = 1; r < rounds; ++r) {
      prefetch(r + 3);
      mlp64_slice<KK, 0>(x_l, XP, l32, hf, b1_l + (NW * r + w) * 4, wf, h, [&](int s) __attribute__((always_inline)) { return frag_m(2 * r - 1, s); }, nothing);
      mlp_u32x4* hb = h_l + (r & 1) * (64 * HP);
      mlp64_pair<2 * NW, GV>(h_l + ((r - 1) & 1) * (64 * HP), HP, l32, hf, wf, out, [&](int s) __attribute__((always_inline)) { return frag_m(2 * r, s); },
                             [&](int i) __attribute__((always_inline)) { gelu_piece(i, 2 * NW, h, hb); });
      __syncthreads();
    }
    prefetch(rounds + 3);
    // the last block of the MLP: what follows it in the stream is the first QKV slice (or nothing)
    mlp64_pair<2 * NW, 0>(h_l + ((rounds - 1) & 1) * (64 * HP), HP, l32, hf, wf, out,
                          [&](int s) __attribute__((always_inline)) { return (LNOUT == 2 && s >= KK) ? frag_q(0, s - KK) : frag_m(lastm, s < KK ? s : KK - 1); }, nothing);
  }

  // ---- Y = x1 + MLP, out in 64-byte pieces through the wave's 2 KiB of the X tile (not read since the last round's barrier)
  Slots b2;
  slots(b2, 3);
  mlp_u32x4 bq[(3 * XS + NTHR - 1) / NTHR];
  if constexpr (LNOUT == 2)
#pragma unroll
    for (int i = 0; i < (3 * XS + NTHR - 1) / NTHR; ++i) bq[i] = ((const mlp_u32x4*)g.bq)[min(tid + i * NTHR, 3 * XS - 1)];
  mlp_u32x4* stage = x_l + w * 128;
  auto emit = [&](bf16_t* base, int scale, const int64_t* ro, int col, const mlp_u32x4& v0, const mlp_u32x4& v1) __attribute__((always_inline)) {
    mlp_stage_put(stage, l32, hf, v0, v1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const mlp_u32x4 v = mlp_stage_get(stage, lane, i);
      const int64_t o = ro[16 * i + (lane >> 2)];
      if (o >= 0) mlp_store16(base + o * scale + col + (lane & 3) * 8, v);
    }
  };
  mlp_u32x4 yv[2][2][2];
  auto yget = [&](int tb, int bt, int gp) __attribute__((always_inline)) { return yv[tb][bt][gp]; };
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) mlp_finish(out[bt][tb], b2[bt][0], b2[bt][1], zero4, false, yv[tb][bt]);
    if constexpr (LNOUT != 0) mlp_stats_put<2>(yv[tb], hf, st_l + w * 64 + 32 * tb + l32);
  }
#pragma unroll
  for (int tb = 0; tb < 2; ++tb)
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) emit((bf16_t*)g.Y, 1, ro_l + 32 * tb, (2 * w + bt) * 32, yv[tb][bt][0], yv[tb][bt][1]);
  if constexpr (LNOUT == 1) {
    __syncthreads();
    normalised(g.ln2_eps, 4, yget, [&](int tb, int bt, const mlp_u32x4& n0, const mlp_u32x4& n1) __attribute__((always_inline)) {
      emit((bf16_t*)g.Y2, 1, ro_l + 64 + 32 * tb, (2 * w + bt) * 32, n0, n1);
    });
  }
  if constexpr (LNOUT == 2) {
    // LayerNorm of the bf16 rows of Y into the hidden tiles' LDS (dead: every wave is past them at the barrier), bq over b1, then the
    // next block's QKV Linear: wave w forms outputs 32 (w + NW j) ..+31, j < NQ
#pragma unroll
    for (int i = 0; i < (3 * XS + NTHR - 1) / NTHR; ++i) if (tid + i * NTHR < 3 * XS) b1_l[tid + i * NTHR] = bq[i];
    __syncthreads();
    normalised(g.ln2_eps, 4, yget, into(n_l));
    __syncthreads();
    // slice j leaves while slice j + 1 is formed: its values in the first KK - 4 steps, a finished token block through the wave's
    // stage one step later
    mlp_u32x4 run[2];
    auto emit_q = [&](int j, int kk, const mlp_f32x16 (&h)[2]) __attribute__((always_inline)) {
      constexpr int S = KK - 4;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        if (kk == ((tb + 1) * S + 1) / 2) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const mlp_u32x4 v = mlp_stage_get(stage, lane, i);
            const int64_t o = ro_l[64 + 32 * tb + 16 * i + (lane >> 2)];         // same row map as the norm's, rows three times as long
            if (o >= 0) mlp_store16((bf16_t*)g.Y2 + o * 3 + (w + NW * j) * 32 + (lane & 3) * 8, v);
          }
        }
      }
      if (kk < S)
        mlp64_out_piece(kk, S, h, pk, [](float a) __attribute__((always_inline)) { return a; }, [&](int, int gp, const mlp_u32x4& v) __attribute__((always_inline)) {
          run[gp] = v;
          if (gp) mlp_stage_put(stage, l32, hf, run[0], run[1]);
        });
    };
    static_assert(NQ % 2 == 0, "slices are taken two at a time");
    mlp_f32x16 ha[2], hb2[2];
    mlp64_slice<KK, 0>(n_l, XP, l32, hf, b1_l + w * 4, wf, ha, [&](int s) __attribute__((always_inline)) { return frag_q(0, s); }, nothing);
#pragma unroll 1
    for (int j = 0; j < NQ; j += 2) {
      mlp64_slice<KK, 2>(n_l, XP, l32, hf, b1_l + (w + NW * (j + 1)) * 4, wf, hb2, [&](int s) __attribute__((always_inline)) { return frag_q(j + 1, s); },
                         [&](int kk) __attribute__((always_inline)) { emit_q(j, kk, ha); });
      if (j + 2 < NQ) {
        mlp64_slice<KK, 2>(n_l, XP, l32, hf, b1_l + (w + NW * (j + 2)) * 4, wf, ha, [&](int s) __attribute__((always_inline)) { return frag_q(j + 2, s); },
                           [&](int kk) __attribute__((always_inline)) { emit_q(j + 1, kk, hb2); });
      } else {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) emit_q(j + 1, kk, hb2);
      }
    }
  }
}

static size_t mlp64p_smem(int C, int Hd) {
  const int NW = C / 64;
  return (size_t)64 * (C / 8 + 1) * 16 + 2 * (size_t)64 * (4 * NW + 1) * 16 + (size_t)Hd * 2 + 2 * 64 * 8 + (size_t)NW * 64 * 8;
}

template <int C, int LNOUT>
static int mlp64p_launch(const MlpArgs& g, void* stream) {
  constexpr size_t vec = (size_t)(LNOUT ? 6 : 4) * C * 2;
  const int vec_lds = mlp64p_smem(C, g.Hd) + vec <= 160 * 1024;      // (a very wide hidden layer's bias takes their place)
  const size_t smem = mlp64p_smem(C, g.Hd) + (vec_lds ? vec : 0);
  static std::atomic<size_t> allowed{0};
  if (smem > allowed.load()) {
    const hipError_t e = hipFuncSetAttribute((const void*)mlp64p_kernel<C, LNOUT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return (int)e;
    allowed.store(smem);
  }
  mlp64p_kernel<C, LNOUT><<<dim3((unsigned)((g.M + 63) / 64)), dim3(C), smem, (hipStream_t)stream>>>(g, vec_lds);
  return (int)hipGetLastError();
}

static size_t mlp64_smem(int C, int Hd) { return (size_t)64 * (C / 8 + 1) * 16 + 2 * (size_t)64 * (4 * (C / 64) + 1) * 16 + (size_t)Hd * 2; }
// shapes the 64-token kernels take: whole rounds of C / 2 hidden units
static bool mlp64_shape(int C, int Hd) { return (C == 256 || C == 384 || C == 512) && Hd >= C / 2 && Hd % (C / 2) == 0 && Hd <= 16384; }
// ... and where they are used: always at C = 512 (the 32-token kernels stop at 384); at 256 and 384 on grids of at least
// one workgroup of 64 tokens per CU (on smaller ones the 32-token tile fills more CUs); not at 128, where the 32-token
// kernel is faster (measured at 32768 tokens, MLP alone: C = 128 21 us against 32; 256: 66 against 51; 384: 147 against 122)
static bool mlp64_use(const MlpArgs& g) {
  if (!mlp64_shape(g.C, g.Hd)) return false;
  if (g.C == 512) return true;
  if (g.C == 128 || g.M < 64 * 256) return false;
  if (g.Wproj_p) return g.norm && g.Hd >= 3 * g.C && mlp64p_smem(g.C, g.Hd) <= 160 * 1024;
  return !g.Y2 && !g.Wq_p && mlp64_smem(g.C, g.Hd) <= 160 * 1024;
}

template <int C>
static int mlp64_launch(const MlpArgs& g, void* stream) {
  if (g.Wproj_p) {      // projection in front (the folded LayerNorm is part of that form), optionally the next block's norm / QKV
    if (!g.norm || g.Hd < 3 * C) return (int)hipErrorInvalidValue;
    if (g.Y2 && g.Wq_p) return mlp64p_launch<C, 2>(g, stream);
    return g.Y2 ? mlp64p_launch<C, 1>(g, stream) : mlp64p_launch<C, 0>(g, stream);
  }
  if (g.Y2 || g.Wq_p) return (int)hipErrorInvalidValue;
  const size_t smem = mlp64_smem(C, g.Hd);
  static std::atomic<size_t> allowed{0};
  if (smem > allowed.load()) {
    const hipError_t e = hipFuncSetAttribute((const void*)mlp64_kernel<C>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return (int)e;
    allowed.store(smem);
  }
  mlp64_kernel<C><<<dim3((unsigned)((g.M + 63) / 64)), dim3(C), smem, (hipStream_t)stream>>>(g);
  return (int)hipGetLastError();
}

static size_t mlp_smem(int C, int Hd, bool proj, int lnout) {
  const size_t tile = (size_t)32 * (C / 8 + 1) * 16, htile = (size_t)32 * (C / 8 + 1) * 16;
  return (proj ? 2 : 1) * tile + 2 * htile + (size_t)Hd * 2 + (size_t)mlp_vectors(proj, lnout) * C * 2 + 2 * 32 * 8 + (size_t)(C / 32) * 32 * 8;
}

template <int C, bool PROJ, int LNOUT>
static int mlp_launch3(const MlpArgs& g, void* stream) {
  const size_t smem = mlp_smem(C, g.Hd, PROJ, LNOUT);
  static std::atomic<size_t> allowed{0};   // raised on demand: the attribute is per kernel, the hidden size varies
  if (smem > allowed.load()) {
    const hipError_t e = hipFuncSetAttribute((const void*)mlp_fused_kernel<C, PROJ, LNOUT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return (int)e;
    allowed.store(smem);
  }
  const int64_t n_wg = (g.M + 31) / 32;
  mlp_fused_kernel<C, PROJ, LNOUT><<<dim3((unsigned)n_wg), dim3(64 * (C / 32)), smem, (hipStream_t)stream>>>(g);
  return (int)hipGetLastError();
}
template <int C>
static int mlp_launch(const MlpArgs& g, void* stream) {
  if (g.Wproj_p) {
    if (g.Y2 && g.Wq_p) return g.Hd >= 3 * C ? mlp_launch3<C, true, 2>(g, stream) : (int)hipErrorInvalidValue;   // (the 64-token kernel's limit: its following bias reuses the first bias's LDS)
    return g.Y2 ? mlp_launch3<C, true, 1>(g, stream) : mlp_launch3<C, true, 0>(g, stream);
  }
  if (g.Wq_p) return (int)hipErrorInvalidValue;
  return g.Y2 ? mlp_launch3<C, false, 1>(g, stream) : mlp_launch3<C, false, 0>(g, stream);
}

// LDS capacity of the projection variant: the A tile beside the others
bool mlp_proj_supported(int C, int Hd, int dtype) {
  if (!mlp_fused_supported(C, Hd, dtype)) return false;
  if (C == 512) return mlp64_shape(C, Hd) && Hd >= 3 * C && mlp64p_smem(C, Hd) <= 160 * 1024;
  return mlp_smem(C, Hd, true, 2) <= 160 * 1024;
}

bool mlp_fused_supported(int C, int Hd, int dtype) {
  if (dtype != SM_BF16) return false;
  if (C == 512) return mlp64_shape(C, Hd) && mlp64_smem(C, Hd) <= 160 * 1024;      // wide rows: the 64-token kernels only
  return (C == 128 || C == 256 || C == 384) && Hd >= 32 && Hd % 32 == 0 && Hd <= 16384;
}

int launch_mlp_pack(const void* W1, const void* W2, int C, int Hd, void* packed, void* stream) {
  const int64_t n = 2 * ((int64_t)Hd * C / 8);
  mlp_pack_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>((const bf16_t*)W1, (const bf16_t*)W2, (mlp_u32x4*)packed, C, Hd);
  return (int)hipGetLastError();
}

int launch_mlp_fused(const MlpArgs& g, void* stream) {
  if (mlp64_use(g)) {
    switch (g.C) {
      case 256: return mlp64_launch<256>(g, stream);
      case 384: return mlp64_launch<384>(g, stream);
      case 512: return mlp64_launch<512>(g, stream);
    }
  }
  switch (g.C) {
    case 128: return mlp_launch<128>(g, stream);
    case 256: return mlp_launch<256>(g, stream);
    case 384: return mlp_launch<384>(g, stream);
  }
  return (int)hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------------------------------------
// Linear for a short reduction dimension (K = C in {128, 256, 384}), Y = act(norm(X) . W^T + b) (+ residual): the first
// product of the kernel above on its own, with four waves.  A workgroup owns 32 token rows, whose K elements stay in LDS for all N outputs;
// the N / 32 row slices of W are dealt round-robin to the four waves and stream from L2 straight into MFMA operand
// registers (packed by lin_pack_kernel: fragment (slice sc, step kk) at sc * K/16 + kk, lane (l32, hf) =
// W[32 sc + l32][16 kk + 8 hf ..+7]); every wave finishes its 32 x 32 outputs in registers and stores them: no
// barrier after the prologue.  Against the tiled kernel of k_gemm.hip this trades L2 -> CU traffic (W once per 32
// rows) for the absence of K-loop barriers and of a separate norm kernel.  Measured (with LayerNorm, against norm
// kernel + tiled kernel resp. the tiled kernel's own folded norm): 200704 x 384 x 128: 62 us against 89;
// 50176 x 768 x 256: 45 against 71; 6272 x 1152 x 384: 15 against 26.
// NW waves per workgroup: 4 (two workgroups per CU, X fragments in registers: large grids) or C / 32 (one workgroup
// per CU with three waves per SIMD at C = 384, X fragments re-read from LDS: grids of about one workgroup per CU)
template <int C, bool RES, int NW>
__global__ __launch_bounds__(64 * NW, 1) void lin32_kernel(Lin32Args g) {
  constexpr int KK = C / 16, XS = C / 8, XP = XS + 1, NTHR = 64 * NW;
  constexpr bool XREG = NW <= 4;
  const SM_KARG Lin32Args* gk = kernarg_ptr<Lin32Args>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  mlp_u32x4* x_l = (mlp_u32x4*)smem_raw;                                  // [32][XP]
  mlp_u32x4* st_l = x_l + 32 * XP;                                        // [NW][128]: the waves' stages of mlp_stage_put
  mlp_u32x4* b_l = st_l + NW * 128;                                       // [N / 8]
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave index as a scalar: slice bases become scalar addresses
  const int64_t row0 = (int64_t)blockIdx.x * 32;
  const int nsub = g.N >> 5;
  const char* Wp = (const char*)g.Wp;

  // weight fragments by buffer loads: descriptor and fragment offset scalar, the lane's 16 bytes the only vector operand
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wp), 0, 2 * g.N * C, 0x00020000);
  const int lo = lane * 16;
  (void)Wp;
  mlp_u32x4 w1[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) w1[kk] = __builtin_amdgcn_raw_buffer_load_b128(rw, lo, ((w < nsub ? w : 0) * KK + kk) * 1024, 0);
  MlpTile<C, NTHR, 32> xt;
  xt.request((const bf16_t*)g.X, row0, g.M, g.x_rows.identity, g.x_rows.ld, &gk->x_rows);
  xt.store(x_l, row0, g.M);
  for (int s = tid; s < g.N / 8; s += NTHR) b_l[s] = g.bias ? ((const mlp_u32x4*)g.bias)[s] : mlp_u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  if (g.norm) {
    mlp_norm_x_tile<C, NTHR, 32>(x_l, g.norm_eps, (const mlp_u32x4*)g.norm_gamma, (const mlp_u32x4*)g.norm_beta);
    __syncthreads();
  }

  // the lane's X fragments do not depend on the slice: with four waves they stay in registers (K / 4 of them)
  mlp_u32x4 xf[XREG ? KK : 1];
  if constexpr (XREG) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) xf[kk] = x_l[l32 * XP + hf + 2 * kk];
  }
  auto y_off = [&](int64_t row) __attribute__((always_inline)) { return g.y_rows.identity ? row * g.y_rows.ld : eval_rows_k(&gk->y_rows, row); };
  int64_t ro = 0;                                 // the residual's row: the lane's token (accumulator column); past M the last row's
  if constexpr (RES) ro = y_off(min(row0 + l32, g.M - 1));
  int64_t so[2];                                  // the rows that the lane stores a 16-byte run of (mlp_stage_get)
  bool s_ok[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t row = row0 + 16 * i + (lane >> 2);
    s_ok[i] = row < g.M;
    so[i] = y_off(s_ok[i] ? row : g.M - 1) + (lane & 3) * 8;
  }
  const bf16_t* R = (const bf16_t*)g.residual;
  bf16_t* Y = (bf16_t*)g.Y;
  const bool gelu_on = g.act == SM_ACT_GELU;
  // the slice loop is one basic block up to the final masked store, so that the issue order below holds; loads
  // that the epilogue needs are issued before the slice's weight prefetch (vector loads return in issue order)
  for (int sc = w; sc < nsub; sc += NW) {
    const int nx = sc + NW < nsub ? sc + NW : sc;
    int xo = l32 * XP + hf;
    if constexpr (!XREG) asm volatile("" : "+v"(xo));   // opaque per slice: fragments re-read from LDS, not kept in registers
    const mlp_u32x4 bias_v = b_l[sc * 4 + hf];          // features 8 hf ..+7 and 16 + 8 hf ..+7 of the slice: the two
    const mlp_u32x4 bias_w = b_l[sc * 4 + 2 + hf];      // runs this lane stores
    mlp_u32x4 res[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
    if constexpr (RES) {
      res[0] = *(const mlp_u32x4*)(R + ro + sc * 32 + hf * 8);
      res[1] = *(const mlp_u32x4*)(R + ro + sc * 32 + 16 + hf * 8);
    }
    mlp_f32x16 h;
#pragma unroll
    for (int e = 0; e < 16; ++e) h[e] = 0.f;
    mlp_u32x4 fb[3] = {x_l[xo], x_l[xo + 2], x_l[xo + 4]};      // (!XREG) LDS fragments three steps ahead of their MFMA
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const mlp_u32x4 xv = XREG ? xf[XREG ? kk : 0] : fb[kk % 3];
      h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(mlp_bf16x8, w1[kk]), __builtin_bit_cast(mlp_bf16x8, xv), h, 0, 0, 0);
      w1[kk] = __builtin_amdgcn_raw_buffer_load_b128(rw, lo, (nx * KK + kk) * 1024, 0);
      if (!XREG && kk + 3 < KK) fb[kk % 3] = x_l[xo + 2 * (kk + 3)];
    }
    __builtin_amdgcn_sched_group_barrier(0x100, XREG ? 2 : 5, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      if constexpr (!XREG) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    mlp_u32x4 outv[2];
    // (a literal flag in each branch: with a run-time flag the polynomial is evaluated for every value and thrown away)
    if (gelu_on) mlp_finish(h, bias_v, bias_w, res, true, outv); else mlp_finish(h, bias_v, bias_w, res, false, outv);
    mlp_stage_put(st_l + w * 128, l32, hf, outv[0], outv[1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const mlp_u32x4 v = mlp_stage_get(st_l + w * 128, lane, i);
      if (s_ok[i]) mlp_store16(Y + so[i] + sc * 32, v);
    }
  }
}

__global__ void lin_pack_kernel(const bf16_t* W, mlp_u32x4* packed, int N, int K) {
  const int KK = K / 16;
  const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= (int64_t)N * K / 8) return;
  const int lane = (int)(o & 63), l32 = lane & 31, hf = lane >> 5;
  const int64_t frag = o >> 6;
  const int sc = (int)(frag / KK), kk = (int)(frag - (int64_t)sc * KK);
  packed[o] = *(const mlp_u32x4*)(W + (int64_t)(32 * sc + l32) * K + 16 * kk + 8 * hf);
}

// The same Linear for wide rows (K = 512): 64 tokens per workgroup, eight waves, every weight fragment feeding two
// MFMAs (the two token blocks); the N / 32 slices of W are dealt round-robin to the waves and a wave's fragments run
// through a ring of 16 registers, as in mlp64_kernel.  LayerNorm folded as above.
template <int C, bool RES>
__global__ __launch_bounds__(512, 1) void lin64_kernel(Lin32Args g) {
  constexpr int KK = C / 16, XS = C / 8, XP = XS + 1, NW = 8, NTHR = 512, RING = 16;
  const SM_KARG Lin32Args* gk = kernarg_ptr<Lin32Args>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  mlp_u32x4* x_l = (mlp_u32x4*)smem_raw;                                  // [64][XP]
  mlp_u32x4* st_l = x_l + 64 * XP;                                        // [NW][128]: the waves' stages of mlp_stage_put
  mlp_u32x4* b_l = st_l + NW * 128;                                       // [N / 8]
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  const int nsub = g.N >> 5;
  const int njobs = (nsub - w + NW - 1) / NW;                             // slices of this wave: w, w + NW, ...
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.Wp), 0, 2 * g.N * C, 0x00020000);
  const int lo = lane * 16;
  auto wload = [&](int soff) __attribute__((always_inline)) { return __builtin_amdgcn_raw_buffer_load_b128(rw, lo, soff, 0); };
  // fragment s of the wave's j-th slice (s may run into the next slice; past the last slice that one again)
  auto foff = [&](int j, int s) __attribute__((always_inline)) -> int {
    if (s >= KK) { j += 1; s -= KK; }
    j = j < njobs ? j : njobs - 1;
    return ((w + NW * (j > 0 ? j : 0)) * KK + s) * 1024;
  };
  mlp_u32x4 wf[RING];
#pragma unroll
  for (int s = 0; s < RING; ++s) wf[s] = wload(foff(0, s));
  auto y_off = [&](int64_t row) __attribute__((always_inline)) { return g.y_rows.identity ? row * g.y_rows.ld : eval_rows_k(&gk->y_rows, row); };
  int64_t ro[2] = {0, 0}, so[2][2]; bool s_ok[2][2];
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    if constexpr (RES) ro[tb] = y_off(min(row0 + 32 * tb + l32, g.M - 1));      // the residual's rows: the lane's tokens
#pragma unroll
    for (int i = 0; i < 2; ++i) {                                               // the rows that the lane stores a 16-byte run of
      const int64_t row = row0 + 32 * tb + 16 * i + (lane >> 2);
      s_ok[tb][i] = row < g.M;
      so[tb][i] = y_off(s_ok[tb][i] ? row : g.M - 1) + (lane & 3) * 8;
    }
  }
  MlpTile<C, NTHR, 64> xt;
  xt.request((const bf16_t*)g.X, row0, g.M, g.x_rows.identity, g.x_rows.ld, &gk->x_rows);
  xt.store(x_l, row0, g.M);
  for (int s = tid; s < g.N / 8; s += 512) b_l[s] = g.bias ? ((const mlp_u32x4*)g.bias)[s] : mlp_u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  if (g.norm) {
    mlp_norm_x_tile<C, NTHR, 64>(x_l, g.norm_eps, (const mlp_u32x4*)g.norm_gamma, (const mlp_u32x4*)g.norm_beta);
    __syncthreads();
  }
  const bf16_t* R = (const bf16_t*)g.residual;
  bf16_t* Y = (bf16_t*)g.Y;
  const bool gelu_on = g.act == SM_ACT_GELU;
  for (int j = 0; j < njobs; ++j) {
    const int sc = w + NW * j;
    int xo = l32 * XP + hf;
    asm volatile("" : "+v"(xo));                        // opaque per slice: the X fragments are re-read, not hoisted
    const mlp_u32x4 bias_v = b_l[sc * 4 + hf], bias_w = b_l[sc * 4 + 2 + hf];
    mlp_u32x4 res[2][2] = {{{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}, {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}};
    if constexpr (RES) {
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        res[tb][0] = *(const mlp_u32x4*)(R + ro[tb] + sc * 32 + hf * 8);
        res[tb][1] = *(const mlp_u32x4*)(R + ro[tb] + sc * 32 + 16 + hf * 8);
      }
    }
    mlp_f32x16 h[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) { h[0][e] = 0.f; h[1][e] = 0.f; }
    mlp_u32x4 fa[2][2] = {{x_l[xo], x_l[xo + 32 * XP]}, {x_l[xo + 2], x_l[xo + 2 + 32 * XP]}};     // two steps ahead
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const mlp_bf16x8 wv = __builtin_bit_cast(mlp_bf16x8, wf[kk % RING]);
      h[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, __builtin_bit_cast(mlp_bf16x8, fa[kk & 1][0]), h[0], 0, 0, 0);
      h[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, __builtin_bit_cast(mlp_bf16x8, fa[kk & 1][1]), h[1], 0, 0, 0);
      wf[kk % RING] = wload(foff(j, kk + RING));
      if (kk + 2 < KK) { fa[kk & 1][0] = x_l[xo + 2 * (kk + 2)]; fa[kk & 1][1] = x_l[xo + 2 * (kk + 2) + 32 * XP]; }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      mlp_u32x4 outv[2];
      if (gelu_on) mlp_finish(h[tb], bias_v, bias_w, res[tb], true, outv); else mlp_finish(h[tb], bias_v, bias_w, res[tb], false, outv);
      mlp_stage_put(st_l + w * 128, l32, hf, outv[0], outv[1]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const mlp_u32x4 v = mlp_stage_get(st_l + w * 128, lane, i);
        if (s_ok[tb][i]) mlp_store16(Y + so[tb][i] + sc * 32, v);
      }
    }
  }
}

template <int C>
static int lin64_launch(const Lin32Args& g, void* stream) {
  const size_t smem = (size_t)64 * (C / 8 + 1) * 16 + 8 * 2048 + (size_t)g.N * 2;
  static std::atomic<size_t> allowed{0};
  if (smem > allowed.load()) {
    hipError_t e = hipFuncSetAttribute((const void*)lin64_kernel<C, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)lin64_kernel<C, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return (int)e;
    allowed.store(smem);
  }
  const dim3 grid((unsigned)((g.M + 63) / 64));
  if (g.residual) lin64_kernel<C, true><<<grid, dim3(512), smem, (hipStream_t)stream>>>(g);
  else lin64_kernel<C, false><<<grid, dim3(512), smem, (hipStream_t)stream>>>(g);
  return (int)hipGetLastError();
}

template <int C, bool RES, int NW>
static int lin32_launch3(const Lin32Args& g, void* stream) {
  const size_t smem = (size_t)32 * (C / 8 + 1) * 16 + (size_t)NW * 2048 + (size_t)g.N * 2;
  static std::atomic<size_t> allowed{0};
  if (smem > allowed.load()) {
    const hipError_t e = hipFuncSetAttribute((const void*)lin32_kernel<C, RES, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return (int)e;
    allowed.store(smem);
  }
  lin32_kernel<C, RES, NW><<<dim3((unsigned)((g.M + 31) / 32)), dim3(64 * NW), smem, (hipStream_t)stream>>>(g);
  return (int)hipGetLastError();
}
template <int C, bool RES>
static int lin32_launch2(const Lin32Args& g, void* stream) {
  // few workgroups (about one per CU) and enough slices to go round: C / 32 waves each
  if constexpr (C / 32 > 4) { if ((g.M + 31) / 32 <= 512 && g.N / 32 >= C / 32) return lin32_launch3<C, RES, C / 32>(g, stream); }
  return lin32_launch3<C, RES, 4>(g, stream);
}
template <int C>
static int lin32_launch(const Lin32Args& g, void* stream) {
  return g.residual ? lin32_launch2<C, true>(g, stream) : lin32_launch2<C, false>(g, stream);
}

bool lin32_supported(int N, int K, int dtype) {
  return dtype == SM_BF16 && (K == 128 || K == 256 || K == 384 || K == 512) && N >= 32 && N % 32 == 0 && N <= 16384;
}

int launch_lin_pack(const void* W, int N, int K, void* packed, void* stream) {
  const int64_t n = (int64_t)N * K / 8;
  lin_pack_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>((const bf16_t*)W, (mlp_u32x4*)packed, N, K);
  return (int)hipGetLastError();
}

int launch_lin32(const Lin32Args& g, void* stream) {
  switch (g.K) {
    case 128: return lin32_launch<128>(g, stream);
    case 256: return lin32_launch<256>(g, stream);
    case 384: return lin32_launch<384>(g, stream);
    case 512: return lin64_launch<512>(g, stream);      // wide rows: 64-token tiles
  }
  return (int)hipErrorInvalidValue;
}

}  // namespace sm
