// Kernels of a decode step (one new token per sequence against a key / value cache; the paper's decoder-only
// workload, Pythia, Table 7, at its memory-bound end).  With at most 32 tokens every Linear is a matrix-vector
// product bound by the stream of its weights from HBM, so the three kernels here are built around that stream:
//
//  * the weights are read in MFMA-fragment order (packed once by launch_lin_pack: fragment (slice, step) is 1 KiB
//    contiguous in lane order; Sec. 3.2.2's rule that a producer writes what its consumer reads best, applied to
//    constants), every wave-load is one fully used 1 KiB run, and a 32 x 32 x 16 MFMA per fragment forms the products
//    for all (up to 32) tokens at once: the matrix core is idle most of the time and costs nothing;
//  * a slice of 32 output features is split along K over the waves of a workgroup, whose partial sums meet in LDS.  W2
//    depends on the first kernel only: its product runs beside the attention, in the same launch, split over workgroups as
//    well; the last kernel adds those parts (fp32, in split order) to Wdense's product.  The attention's own splits of the
//    keys are merged by the workgroup that arrives last (a counter per head, no waiting anywhere, every order of arrival
//    gives the same sum order);
//  * the layout operators of the step are addresses of these kernels' loads and stores: the query / key / value
//    Slices and Permutes and the Concat behind the cache are the store of the first kernel (the new key / value row
//    goes straight to position L of the cache), the head merge is the store of the attention kernel.
#include <algorithm>
#include "device_common.h"
#include "kernels.h"

namespace sm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 dc_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float dc_f32x16;
typedef unsigned int dc_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int dc_u32x2 __attribute__((ext_vector_type(2)));

constexpr int DC_CNT_STRIDE = 64;   // ints between two arrival counters: one counter per 256 bytes, so that the
                                    // increments of different slices / heads do not queue up on one cache line
constexpr int DC_PF = 8;       // weight fragments per register set of a wave (two sets)
constexpr int DC_PF_LONG = 16; // the same where a wave's stream is longer than 16: 32 steps (E = 2048, F = 8192) are requested up front
constexpr int DC_ATTN_NW = 8;  // waves of a workgroup of the attention
constexpr int DC_ATTN_NIT = 2; // key rows (and value rows) a lane of the attention holds: with two sets of two a wave stays within 128
                               // registers, so that a workgroup of W2's product runs beside one of the attention

__device__ __forceinline__ void dc_unpack8(dc_u32x4 v, float* f) {
#pragma unroll
  for (int e = 0; e < 4; ++e) { f[2 * e] = __uint_as_float(v[e] << 16); f[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u); }
}
__device__ __forceinline__ float dc_load_f32(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ void dc_store_f32(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// true in exactly one workgroup per counter: the one whose increment is the n-th.  The partial results a workgroup
// hands over are written with dc_store_f32 (device-scope stores that go through to memory) and read with dc_load_f32:
// once the wave's stores have completed (vmcnt 0) and the workgroup has met at the barrier, the increment can only be
// observed after them.  No cache write-back and no invalidation is involved: a release fence here would flush the L2 once per
// workgroup, and behind an acquire fence the merge of 64 heads took 14 us instead of 3.
__device__ __forceinline__ bool dc_arrived_last(int* counter, int n, int* flag_lds) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) *flag_lds = (__hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1);
  __syncthreads();
  const bool last = *flag_lds != 0;
  asm volatile("" ::: "memory");      // the partial results are read with device-scope loads, issued after the increment has returned
  return last;
}

// The weight stream of one wave: steps k in [k0, k1) of a slice, fragment k at byte 1024 k of the slice (16 bytes a lane; descriptor
// and offset are scalar, so that a load costs one instruction).  Two register sets of PF fragments.  preload issues both sets' first
// loads (before the activation tile is ready, so that the prologue's latency and the first weights overlap; unconditionally, so that
// the compiler can count what is in flight behind the prologue's own loads); consume forms acc += W(k) x X(k) for all steps,
// reloading a set right after the products that read it, where there is more to read.  X fragments come from LDS: step k at
// xl + (k - kbase) * 32 bytes.  Loads past the end within a set re-read the last step and their products are formed with a zero
// operand.
template <int PF> struct DcStream {
  __amdgpu_buffer_rsrc_t r; int lo;
  dc_u32x4 a[PF], b[PF];
  __device__ __forceinline__ dc_u32x4 load(int k) const { return __builtin_amdgcn_raw_buffer_load_b128(r, lo, k * 1024, 0); }
  __device__ __forceinline__ void preload(const void* W, int64_t slice, int steps, int lane, int k0, int k1) {
    r = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(W) + slice * steps * 1024, 0, steps * 1024, 0x00020000);
    lo = lane * 16;
#pragma unroll
    for (int i = 0; i < PF; ++i) a[i] = load(min(k0 + i, k1 - 1));
#pragma unroll
    for (int i = 0; i < PF; ++i) b[i] = load(min(k0 + PF + i, k1 - 1));
  }
  // the products of the set that starts at step kk
  static __device__ __forceinline__ void products(const dc_u32x4 (&f)[PF], const unsigned char* xl, int kbase, int kk, int k1, dc_f32x16& acc) {
    const dc_u32x4 zero = {0u, 0u, 0u, 0u};
    dc_u32x4 x[PF];
    if (kk + PF <= k1) {
#pragma unroll
      for (int i = 0; i < PF; ++i) x[i] = *(const dc_u32x4*)(xl + (size_t)(kk + i - kbase) * 32);
    } else {
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        x[i] = *(const dc_u32x4*)(xl + (size_t)(min(kk + i, k1 - 1) - kbase) * 32);
        if (kk + i >= k1) x[i] = zero;
      }
    }
#pragma unroll
    for (int i = 0; i < PF; ++i)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(dc_bf16x8, f[i]), __builtin_bit_cast(dc_bf16x8, x[i]), acc, 0, 0, 0);
  }
  __device__ __forceinline__ void consume(const unsigned char* xl, int kbase, int k0, int k1, dc_f32x16& acc) {
    for (int kk = k0; kk < k1; kk += 2 * PF) {
      products(a, xl, kbase, kk, k1, acc);
      if (kk + 2 * PF < k1)
#pragma unroll
        for (int i = 0; i < PF; ++i) a[i] = load(min(kk + 2 * PF + i, k1 - 1));
      if (kk + PF < k1) products(b, xl, kbase, kk + PF, k1, acc);
      if (kk + 3 * PF < k1)
#pragma unroll
        for (int i = 0; i < PF; ++i) b[i] = load(min(kk + 3 * PF + i, k1 - 1));
    }
  }
};

// cos and sin of position x theta_i, theta_i = base^(-2 i / rot): the angle in revolutions, its fraction to the hardware
__device__ __forceinline__ void dc_rope_cs(int pos, int i, int rot, float base, float* c, float* s) {
  const float rev = (float)pos * (exp2f(-2.f * (float)i / (float)rot * log2f(base)) * 0.15915494309189535f);
  const float f = __builtin_amdgcn_fractf(rev);
  *c = __builtin_amdgcn_cosf(f); *s = __builtin_amdgcn_sinf(f);
}

// ---------------------------------------------------------------------------------------------------------------
// First kernel: [q | k | v] = LayerNorm-1(x) . Wqkv^T + bqkv with the rotary embedding on the first `rot` features of
// every query and key head, and hid = GELU(LayerNorm-2(x) . W1^T + b1): the two Linears that depend on x alone
// (parallel residual), one launch.  A workgroup owns 64 consecutive output features (two slices of 32) so that both
// members of a rotary pair (i, i + rot/2), rot/2 <= 32, are in the same workgroup; eight waves: slice = wave / 4,
// K quarter = wave % 4.  59 MB of weights at E = 2048, F = 8192: 15.4 -> 12.9 us for one token, all there 9 us after the start.
template <int MAXP, int PF>      // 16-byte pieces of a token row per lane: E <= 512 MAXP; fragments per register set
__global__ __launch_bounds__(512) void decode_in_kernel(DecodeInArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dc_smem[];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int B = a.B, E = a.E;
  const int pitch = E + 8;                                          // elements: rows 16 bytes apart modulo the banks
  bf16_t* xs = (bf16_t*)dc_smem;                                    // [B][pitch] normalised x
  float* red = (float*)(dc_smem + (size_t)B * pitch * 2);           // [8 waves][32 rows][B]
  float* vals = red + 8 * 32 * B;                                   // [64 rows][B]
  if (blockIdx.x == 0) for (int i = tid; i < a.n_counters; i += 512) a.counters[i * DC_CNT_STRIDE] = 0;
  const int n0 = blockIdx.x * 64;
  const bool fc1 = n0 >= 3 * E;
  const bf16_t* gam = fc1 ? a.ln2_g : a.ln1_g;
  const bf16_t* bet = fc1 ? a.ln2_b : a.ln1_b;
  // the wave's K quarter of its slice
  const int KS = E / 16, per = (KS + 3) / 4;
  const int k0 = (w & 3) * per, k1 = min(KS, k0 + per);
  const int slice = (fc1 ? (n0 - 3 * E) : n0) / 32 + (w >> 2);
  const void* Wm = fc1 ? a.w1_p_ : a.wqkv_p_;
  // Loads return in the order they were asked for: first what the prologue needs (this wave's first token row, gamma, beta, the
  // biases), then the weights, which arrive under the LayerNorm.  (Behind the weights, the LayerNorm starts when the last of
  // them is there: one token 3 us later.)  Long rows need the registers for the LayerNorm first.
  const int nch = E / 8;
  dc_u32x4 xv[MAXP], gv[MAXP], bv[MAXP];      // gv / bv hold one piece at a time when MAXP > 4
  auto load_row = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < MAXP; ++j) xv[j] = *(const dc_u32x4*)(a.x + (int64_t)b * E + 8 * min(lane + 64 * j, nch - 1));
  };
  const float bias = bf2f((fc1 ? a.b1 - 3 * E : a.bqkv)[n0 + lane]);      // of feature `lane`
  if constexpr (MAXP <= 4) {
    load_row(min(w, B - 1));
#pragma unroll
    for (int j = 0; j < MAXP; ++j) { const int c = min(lane + 64 * j, nch - 1); gv[j] = *(const dc_u32x4*)(gam + 8 * c); bv[j] = *(const dc_u32x4*)(bet + 8 * c); }
  }
  __builtin_amdgcn_sched_barrier(0);
  DcStream<PF> fr;
  if constexpr (MAXP <= 4) fr.preload(Wm, slice, KS, lane, k0, k1);
  __builtin_amdgcn_sched_barrier(0);
  // LayerNorm of the tokens this workgroup needs (all of them), two-pass statistics, bf16 result in LDS
  for (int b = w; b < B; b += 8) {
    if (MAXP > 4 || b != w) load_row(b);
    float f[8], s = 0.f;
#pragma unroll
    for (int j = 0; j < MAXP; ++j) {
      if (lane + 64 * j < nch) {
        dc_unpack8(xv[j], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) s += f[e];
      }
    }
    const float mean = wave_sum(s) / (float)E;
    s = 0.f;
#pragma unroll
    for (int j = 0; j < MAXP; ++j) {
      if (lane + 64 * j < nch) {
        dc_unpack8(xv[j], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float dlt = f[e] - mean; s = fmaf(dlt, dlt, s); }
      }
    }
    const float rstd = rsqrtf(wave_sum(s) / (float)E + a.eps);
#pragma unroll
    for (int j = 0; j < MAXP; ++j) {
      const int c = lane + 64 * j;
      if (c < nch) {
        float g[8], bt[8];
        if constexpr (MAXP > 4) { gv[j] = *(const dc_u32x4*)(gam + 8 * c); bv[j] = *(const dc_u32x4*)(bet + 8 * c); }      // long rows: registers go to x
        dc_unpack8(xv[j], f); dc_unpack8(gv[j], g); dc_unpack8(bv[j], bt);
        dc_u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = (unsigned)f2bf(fmaf((f[2 * e] - mean) * rstd, g[2 * e], bt[2 * e])) | ((unsigned)f2bf(fmaf((f[2 * e + 1] - mean) * rstd, g[2 * e + 1], bt[2 * e + 1])) << 16);
        *(dc_u32x4*)(xs + (size_t)b * pitch + 8 * c) = o;
      }
    }
  }
  if constexpr (MAXP > 4) fr.preload(Wm, slice, KS, lane, k0, k1);
  __syncthreads();
  const unsigned char* xl = (const unsigned char*)xs + (size_t)min(l32, B - 1) * pitch * 2 + hf * 16;
  dc_f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  fr.consume(xl, 0, k0, k1, acc);
  if (l32 < B) {
#pragma unroll
    for (int i = 0; i < 16; ++i) red[(w * 32 + (i / 4) * 8 + hf * 4 + (i & 3)) * B + l32] = acc[i];
  }
  __syncthreads();
  for (int idx = tid; idx < 64 * B; idx += 512) {
    const int r = idx / B, b = idx - r * B, s4 = (r >> 5) * 4, rr = r & 31;
    float v = __shfl(bias, r, 64);
#pragma unroll
    for (int p = 0; p < 4; ++p) v += red[((s4 + p) * 32 + rr) * B + b];
    vals[idx] = v;
  }
  __syncthreads();
  for (int idx = tid; idx < 64 * B; idx += 512) {
    const int r = idx / B, b = idx - r * B;
    float v = vals[idx];
    if (fc1) {
      v = 0.5f * v * (1.f + erff(v * 0.70710678118654752f));
      a.hid[(int64_t)b * a.F + (n0 - 3 * E) + r] = f2bf(v);
    } else {
      const int n = n0 + r, d = a.d, hh = n / (3 * d), rem = n - hh * 3 * d, t = rem / d, e = rem - t * d;
      if (t < 2 && e < a.rot) {                                   // rotary pair (i, i + rot/2) at position L
        const int half = a.rot >> 1, i = e < half ? e : e - half;
        const float other = vals[(e < half ? r + half : r - half) * B + b];
        float c, s;
        dc_rope_cs(a.L, i, a.rot, a.rope_base, &c, &s);
        v = e < half ? v * c - other * s : v * c + other * s;
      }
      a.dst[t][(int64_t)b * a.dst_b[t] + (int64_t)hh * a.dst_h[t] + e] = f2bf(v);
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Attention of one query per (sequence, head) over n_keys cached tokens, the keys split over gridDim.x workgroups
// (equal shares of whole blocks of DC_ATTN_NW waves x DC_ATTN_NIT x 4 keys).  A key row (D elements) is read by 16 adjacent
// lanes (one DPP row), D / 16 elements each in 16-byte pieces (8-byte for D = 64), so a wave-load covers four rows in
// runs of 256 bytes and the dot product's cross-lane sum is four DPP adds (no LDS traffic).  A lane keeps its query
// features in registers and holds the value rows of exactly the keys whose scores it ends up with (the reduction
// leaves a key's score in every lane of its row), so a wave runs its own online softmax over its keys with no LDS and
// no barrier: blocks of DC_ATTN_NIT key rows and value rows per lane, two register sets, one in flight while the
// other is consumed.  At the end the waves merge through LDS; a workgroup that has all keys of its head stores the result, else
// it leaves (max, sum, unnormalised output) in `part`, and the one that arrives last for its (sequence, head) merges them.
template <int D> struct DcRow;      // a lane's share of a key / value row: D / 16 elements
template <> struct DcRow<256> { dc_u32x4 p[2]; };
template <> struct DcRow<128> { dc_u32x4 p[1]; };
template <> struct DcRow<64> { dc_u32x2 p[1]; };
template <int D> __device__ __forceinline__ DcRow<D> dc_row_load(const bf16_t* row, int lk) {
  DcRow<D> r;
  if constexpr (D == 256) { r.p[0] = *(const dc_u32x4*)(row + 8 * lk); r.p[1] = *(const dc_u32x4*)(row + 128 + 8 * lk); }
  else if constexpr (D == 128) r.p[0] = *(const dc_u32x4*)(row + 8 * lk);
  else r.p[0] = *(const dc_u32x2*)(row + 4 * lk);
  return r;
}
// the lane's D / 16 features as floats, in the order element e of piece j
template <int D> __device__ __forceinline__ void dc_row_unpack(const DcRow<D>& r, float* f) {
  if constexpr (D == 256) { dc_unpack8(r.p[0], f); dc_unpack8(r.p[1], f + 8); }
  else if constexpr (D == 128) { dc_unpack8(r.p[0], f); }
  else {
#pragma unroll
    for (int e = 0; e < 2; ++e) { f[2 * e] = __uint_as_float(r.p[0][e] << 16); f[2 * e + 1] = __uint_as_float(r.p[0][e] & 0xffff0000u); }
  }
}
// feature index of float i of dc_row_unpack for lane lk of a row
template <int D> __device__ __forceinline__ int dc_row_feature(int lk, int i) {
  if constexpr (D == 256) return (i >> 3) * 128 + 8 * lk + (i & 7);
  else if constexpr (D == 128) return 8 * lk + i;
  else return 4 * lk + i;
}
// sum over the 16 lanes of a DPP row, result in every lane: xor 1, xor 2 (quad permutes), then the mirrors of 8 and 16
__device__ __forceinline__ float dc_row_sum16(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));
  return v;
}

template <int D>
struct DcKV { DcRow<D> k[DC_ATTN_NIT], v[DC_ATTN_NIT]; };

// row u of a block: key0 + 32 u (eight waves x four rows of lanes).  Rows past the end re-read the last key (no
// branch around a load, so that the loads of one set stay in flight while the other set is consumed); their scores
// are masked.
template <int D>
__device__ __forceinline__ void dc_attn_load(DcKV<D>& r, const bf16_t* Kp, const bf16_t* Vp, int lk, int key0, int t1) {
#pragma unroll
  for (int u = 0; u < DC_ATTN_NIT; ++u) r.k[u] = dc_row_load<D>(Kp + (int64_t)min(key0 + 4 * DC_ATTN_NW * u, t1 - 1) * D, lk);
#pragma unroll
  for (int u = 0; u < DC_ATTN_NIT; ++u) r.v[u] = dc_row_load<D>(Vp + (int64_t)min(key0 + 4 * DC_ATTN_NW * u, t1 - 1) * D, lk);
}

template <int D>
__device__ __forceinline__ void dc_attn_block(const DcKV<D>& r, const float* qf, int key0, int t1, float& m, float& l, float* acc) {
  constexpr int NF = D / 16;
  float s[DC_ATTN_NIT], mb = -INFINITY;
#pragma unroll
  for (int u = 0; u < DC_ATTN_NIT; ++u) {
    float kf[NF], dot = 0.f;
    dc_row_unpack<D>(r.k[u], kf);
#pragma unroll
    for (int e = 0; e < NF; ++e) dot = fmaf(qf[e], kf[e], dot);
    dot = dc_row_sum16(dot);
    s[u] = key0 + 4 * DC_ATTN_NW * u < t1 ? dot : -INFINITY;
    mb = fmaxf(mb, s[u]);
  }
  mb = fmaxf(mb, __shfl_xor(mb, 16, 64));
  mb = fmaxf(mb, __shfl_xor(mb, 32, 64));
  const float mn = fmaxf(m, mb);
  if (mn == -INFINITY) return;                       // no valid key in this block for the whole wave (wave-uniform)
  const float f = exp2f(m - mn);                     // 0 when m was -inf
  m = mn; l *= f;
#pragma unroll
  for (int e = 0; e < NF; ++e) acc[e] *= f;
#pragma unroll
  for (int u = 0; u < DC_ATTN_NIT; ++u) {
    const float p = exp2f(s[u] - mn);                // 0 for masked keys
    float vf[NF];
    dc_row_unpack<D>(r.v[u], vf);
    l += p;
#pragma unroll
    for (int e = 0; e < NF; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
  }
}

template <int D>
__device__ __forceinline__ void decode_attn(const DecodeAttnArgs& a, const int bh, const int split, const int nsplit) {
  constexpr int NF = D / 16, BLOCK = 4 * DC_ATTN_NW * DC_ATTN_NIT;
  __shared__ float s_red[DC_ATTN_NW][D + 2];
  __shared__ int s_flag;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lk = lane & 15, kq = lane >> 4;
  const int b = bh / a.h, hh = bh - b * a.h;
  // blocks are dealt to the workgroups of a (sequence, head) in turn, so that at any time they read one contiguous
  // stretch of the cache together (a softmax does not care about the order of its keys)
  const int t1 = a.n_keys, stride = nsplit * BLOCK;
  const bf16_t* Kp = a.K + (int64_t)b * a.kv_b + (int64_t)hh * a.kv_h;
  const bf16_t* Vp = a.V + (int64_t)b * a.kv_b + (int64_t)hh * a.kv_h;
  const DcRow<D> qv = dc_row_load<D>(a.q + (int64_t)b * a.q_b + (int64_t)hh * a.q_h, lk);
  const int first = split * BLOCK + 4 * w + kq;      // this lane's key in row u = 0 of the workgroup's first block
  DcKV<D> ra, rb;
  dc_attn_load<D>(ra, Kp, Vp, lk, first, t1);
  float qf[NF], acc[NF], m = -INFINITY, l = 0.f;
  dc_row_unpack<D>(qv, qf);
#pragma unroll
  for (int e = 0; e < NF; ++e) { qf[e] *= a.scale_log2e; acc[e] = 0.f; }
  for (int base = split * BLOCK; base < t1; base += 2 * stride) {
    const int kb = base + 4 * w + kq;
    dc_attn_load<D>(rb, Kp, Vp, lk, kb + stride, t1);
    dc_attn_block<D>(ra, qf, kb, t1, m, l, acc);
    dc_attn_load<D>(ra, Kp, Vp, lk, kb + 2 * stride, t1);
    dc_attn_block<D>(rb, qf, kb + stride, t1, m, l, acc);
  }
  // the wave's four rows of lanes hold disjoint keys: sums over the rows; then the waves through LDS
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    l += __shfl_xor(l, o, 64);
#pragma unroll
    for (int e = 0; e < NF; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  }
  if (kq == 0) {
#pragma unroll
    for (int e = 0; e < NF; ++e) s_red[w][dc_row_feature<D>(lk, e)] = acc[e];
    if (lk == 0) { s_red[w][D] = m; s_red[w][D + 1] = l; }
  }
  __syncthreads();
  float M = s_red[0][D], f[DC_ATTN_NW], lsum = 0.f, osum = 0.f;
#pragma unroll
  for (int i = 1; i < DC_ATTN_NW; ++i) M = fmaxf(M, s_red[i][D]);
#pragma unroll
  for (int i = 0; i < DC_ATTN_NW; ++i) { f[i] = s_red[i][D] == -INFINITY ? 0.f : exp2f(s_red[i][D] - M); lsum += f[i] * s_red[i][D + 1]; }
#pragma unroll
  for (int i = 0; i < DC_ATTN_NW; ++i) osum += f[i] * s_red[i][min(tid, D - 1)];
  if (nsplit == 1) {
    if (tid < D) a.o[(int64_t)b * a.o_b + (int64_t)hh * a.o_h + tid] = f2bf(osum / lsum);
    return;
  }
  float* part = a.part + ((int64_t)bh * nsplit + split) * (D + 2);
  if (tid < D) dc_store_f32(part + tid, osum);
  if (tid == 0) { dc_store_f32(part + D, M); dc_store_f32(part + D + 1, lsum); }
  if (!dc_arrived_last(a.counters + bh * DC_CNT_STRIDE, nsplit, &s_flag)) return;
  if (tid < D) {      // the partial results are read eight workgroups at a time (independent loads, one round trip)
    const float* p0 = a.part + (int64_t)bh * nsplit * (D + 2);
    float M = -INFINITY;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
      float ms[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) ms[i] = dc_load_f32(p0 + (int64_t)min(s0 + i, nsplit - 1) * (D + 2) + D);
#pragma unroll
      for (int i = 0; i < 8; ++i) M = fmaxf(M, ms[i]);
    }
    float o = 0.f, ls = 0.f;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
      float ms[8], os[8], lv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float* ps = p0 + (int64_t)min(s0 + i, nsplit - 1) * (D + 2);
        ms[i] = dc_load_f32(ps + D); os[i] = dc_load_f32(ps + tid); lv[i] = dc_load_f32(ps + D + 1);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float f = (s0 + i >= nsplit || ms[i] == -INFINITY) ? 0.f : exp2f(ms[i] - M);
        o = fmaf(f, os[i], o);
        ls = fmaf(f, lv[i], ls);
      }
    }
    a.o[(int64_t)b * a.o_b + (int64_t)hh * a.o_h + tid] = f2bf(o / ls);
  }
}

// ---------------------------------------------------------------------------------------------------------------
// W2 . hid for one slice of 32 output features and one of `nf` splits of F: fp32 sums to part[split][b][E]; the split's
// activation rows go to LDS (after the wave's first weight fragments are requested).
__device__ __forceinline__ void decode_fc2(const DecodeFc2Args& a, const int slice, const int ks, unsigned char* smem) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int B = a.B, KM = a.F / 16, per = (KM + a.nf - 1) / a.nf, g0 = min(KM, ks * per), g1 = min(KM, g0 + per);
  const int perw = (g1 - g0 + 7) / 8, k0 = min(g1, g0 + w * perw), k1 = min(g1, k0 + perw);
  // the activation rows before the weights (which would return first otherwise): up to four pieces a thread wait in registers
  const int pitch = per * 16 + 8, nch = (g1 - g0) * 2, n = B * nch;
  bf16_t* xs = (bf16_t*)smem;
  dc_u32x4 early[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = min(tid + 512 * i, max(n - 1, 0)), b = nch ? idx / nch : 0, c = idx - b * nch;
    early[i] = *(const dc_u32x4*)(a.hid + (int64_t)b * a.F + (n ? 16 * g0 + 8 * c : 0));
  }
  __builtin_amdgcn_sched_barrier(0);
  DcStream<DC_PF> fr;
  fr.preload(a.w2_p_, slice, KM, lane, k0, k1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = tid + 512 * i, b = nch ? idx / nch : 0, c = idx - b * nch;
    if (idx < n) *(dc_u32x4*)(xs + (size_t)b * pitch + 8 * c) = early[i];
  }
  for (int idx = tid + 2048; idx < n; idx += 512) {
    const int b = idx / nch, c = idx - b * nch;
    *(dc_u32x4*)(xs + (size_t)b * pitch + 8 * c) = *(const dc_u32x4*)(a.hid + (int64_t)b * a.F + 16 * g0 + 8 * c);
  }
  __syncthreads();
  const unsigned char* xl = (const unsigned char*)xs + (size_t)min(l32, B - 1) * pitch * 2 + hf * 16;
  dc_f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  fr.consume(xl, g0, k0, k1, acc);
  __syncthreads();
  float* red = (float*)smem;                        // over the rows, which are used up
  if (l32 < B) {
#pragma unroll
    for (int i = 0; i < 16; ++i) red[(w * 32 + (i / 4) * 8 + hf * 4 + (i & 3)) * B + l32] = acc[i];
  }
  __syncthreads();
  for (int idx = tid; idx < 32 * B; idx += 512) {
    const int b = idx >> 5, r = idx & 31;
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) v += red[(i * 32 + r) * B + b];
    a.part[((int64_t)ks * B + b) * a.E + slice * 32 + r] = v;
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Middle kernel: attention and W2 . hid in one launch (both depend on the first kernel only).  The attention's workgroups come
// first: theirs is the longer chain, and W2's stream fills the memory's time while they start and merge.  8 sequences x 2047 keys
// (168 MB) 27.8 us and 5.2 in the last kernel, one sequence x 150 11.4 + 4.6; with W2's product in the last kernel 29.8 + 14.6 and
// 8.8 + 12.2.
template <int D>
__global__ __launch_bounds__(512, 4) void decode_mid_kernel(DecodeAttnArgs a, DecodeFc2Args f, int nsplit) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dc_smem[];
  const int n_attn = a.B * a.h * nsplit, i = blockIdx.x;
  if (i < n_attn) { decode_attn<D>(a, i / nsplit, i % nsplit, nsplit); return; }
  const int j = i - n_attn, slices = f.E / 32;
  decode_fc2(f, j % slices, j / slices, dc_smem);
}

// ---------------------------------------------------------------------------------------------------------------
// Last kernel: y = x + bdense + b2 + Wdense . o + the parts of W2 . hid.  One workgroup per slice of 32 features, K over its
// sixteen waves (their sums are added in wave order), everything requested before anything is waited for; no exchange between
// workgroups, which costs more than the few CUs' bandwidth that a split over more of them would add.
__global__ __launch_bounds__(1024) void decode_out_kernel(DecodeOutArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dc_smem[];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hf = lane >> 5;
  const int B = a.B, E = a.E, slice = blockIdx.x, KM = E / 16;
  const int perw = (KM + 15) / 16, k0 = min(KM, w * perw), k1 = min(KM, k0 + perw);
  const int pitch = E + 8, nch = E / 8;
  bf16_t* xs = (bf16_t*)dc_smem;
  // in the order of their use: the rows of o, the weights, what is added to the product
  dc_u32x4 early[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = min(tid + 1024 * i, B * nch - 1), b = idx / nch, c = idx - b * nch;
    early[i] = *(const dc_u32x4*)(a.o + (int64_t)b * E + 8 * c);
  }
  __builtin_amdgcn_sched_barrier(0);
  DcStream<4> fr;
  fr.preload(a.wdense_p_, slice, KM, lane, k0, k1);
  __builtin_amdgcn_sched_barrier(0);
  const int ob = min(tid >> 5, B - 1), n = slice * 32 + (tid & 31);      // one output per thread
  const bf16_t bd = a.bdense[n], b2 = a.b2[n], xr = a.x[(int64_t)ob * E + n];
  float pv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) pv[i] = a.part[((int64_t)min(i, a.nf - 1) * B + ob) * E + n];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int idx = tid + 1024 * i, b = idx / nch, c = idx - b * nch;
    if (idx < B * nch) *(dc_u32x4*)(xs + (size_t)b * pitch + 8 * c) = early[i];
  }
  for (int idx = tid + 2048; idx < B * nch; idx += 1024) {
    const int b = idx / nch, c = idx - b * nch;
    *(dc_u32x4*)(xs + (size_t)b * pitch + 8 * c) = *(const dc_u32x4*)(a.o + (int64_t)b * E + 8 * c);
  }
  __syncthreads();
  const unsigned char* xl = (const unsigned char*)xs + (size_t)min(l32, B - 1) * pitch * 2 + hf * 16;
  dc_f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  fr.consume(xl, 0, k0, k1, acc);
  __syncthreads();
  float* red = (float*)dc_smem;                     // over the rows, which are used up
  if (l32 < B) {
#pragma unroll
    for (int i = 0; i < 16; ++i) red[(w * 32 + (i / 4) * 8 + hf * 4 + (i & 3)) * B + l32] = acc[i];
  }
  __syncthreads();
  if ((tid >> 5) < B) {
    float v = bf2f(bd) + bf2f(b2);                  // then the parts in split order, the waves in theirs, the residual
#pragma unroll
    for (int i = 0; i < 4; ++i) v += i < a.nf ? pv[i] : 0.f;
    for (int i = 4; i < a.nf; ++i) v += a.part[((int64_t)i * B + ob) * E + n];
#pragma unroll
    for (int i = 0; i < 16; ++i) v += red[(i * 32 + (tid & 31)) * B + ob];
    a.y[(int64_t)ob * E + n] = f2bf(v + bf2f(xr));
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Explicit chain only: the Concat behind the cache as a copy, out[bh][t] = t < L ? cache[bh][t] : fresh[bh], rows of
// d elements in 16-byte vectors.
__global__ void decode_concat_kernel(const dc_u32x4* cache, int64_t cache_bh, const dc_u32x4* fresh, dc_u32x4* out, int L, int dv, int64_t total) {
  const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= total) return;
  const int c = (int)(o % dv);
  const int64_t row = o / dv;
  const int t = (int)(row % (L + 1));
  const int64_t bh = row / (L + 1);
  out[o] = t < L ? cache[bh * cache_bh + (int64_t)t * dv + c] : fresh[bh * dv + c];
}

size_t decode_in_smem(int B, int E) { return (size_t)B * (E + 8) * 2 + (size_t)(8 * 32 + 64) * B * 4; }

// dynamic LDS up to the CU's
template <typename F> static int dc_allow_lds(F f) { return (int)hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); }
template <int MAXP, int PF> static int decode_in_launch(const DecodeInArgs& a, hipStream_t s) {
  static const int attr = dc_allow_lds(decode_in_kernel<MAXP, PF>);
  if (attr) return attr;
  decode_in_kernel<MAXP, PF><<<dim3((unsigned)((3 * a.E + a.F) / 64)), dim3(512), decode_in_smem(a.B, a.E), s>>>(a);
  return (int)hipGetLastError();
}
int launch_decode_in(const DecodeInArgs& a, void* stream) {
  // a wave's stream is E / 64 fragments: requested at once up to 32 (decode_in 1024 < E <= 2048); long rows need the registers
  // for the LayerNorm first
  if (a.E <= 1024) return decode_in_launch<4, DC_PF>(a, (hipStream_t)stream);
  if (a.E <= 2048) return decode_in_launch<4, DC_PF_LONG>(a, (hipStream_t)stream);
  return decode_in_launch<16, DC_PF>(a, (hipStream_t)stream);
}

int decode_attn_block(int) { return 4 * DC_ATTN_NW * DC_ATTN_NIT; }
int decode_counter_stride() { return DC_CNT_STRIDE; }      // keys of one block of the attention kernel

static size_t decode_fc2_smem(int B, int F, int nf) {
  const int per = (F / 16 + nf - 1) / nf;
  return std::max((size_t)B * (per * 16 + 8) * 2, (size_t)8 * 32 * B * 4);
}
// K splits of W2's product: about a workgroup per CU, with at least 8 steps per wave, and a split's activation rows within 48 KiB
int decode_fc2_splits(int B, int E, int F) {
  const int slices = E / 32;
  int s = std::max(1, std::min((256 + slices - 1) / slices, F / 16 / 64));
  while (s < 64 && decode_fc2_smem(B, F, s) > 48 * 1024) ++s;
  return s;
}

template <int D> static int decode_mid_launch(const DecodeAttnArgs& a, const DecodeFc2Args& f, int nsplit, hipStream_t s) {
  const size_t smem = decode_fc2_smem(f.B, f.F, f.nf);
  if (smem > 48 * 1024) return (int)hipErrorInvalidValue;
  decode_mid_kernel<D><<<dim3((unsigned)(a.B * a.h * nsplit + f.E / 32 * f.nf)), dim3(512), smem, s>>>(a, f, nsplit);
  return (int)hipGetLastError();
}
int launch_decode_mid(const DecodeAttnArgs& a, const DecodeFc2Args& f, int nsplit, void* stream) {
  if (nsplit < 1 || f.nf < 1) return (int)hipErrorInvalidValue;
  switch (a.d) {
    case 64: return decode_mid_launch<64>(a, f, nsplit, (hipStream_t)stream);
    case 128: return decode_mid_launch<128>(a, f, nsplit, (hipStream_t)stream);
    case 256: return decode_mid_launch<256>(a, f, nsplit, (hipStream_t)stream);
  }
  return (int)hipErrorInvalidValue;
}

int launch_decode_out(const DecodeOutArgs& a, void* stream) {
  static const int attr = dc_allow_lds(decode_out_kernel);
  if (attr) return attr;
  const size_t smem = std::max((size_t)a.B * (a.E + 8) * 2, (size_t)16 * 32 * a.B * 4);
  if (smem > 160 * 1024) return (int)hipErrorInvalidValue;
  decode_out_kernel<<<dim3((unsigned)(a.E / 32)), dim3(1024), smem, (hipStream_t)stream>>>(a);
  return (int)hipGetLastError();
}

int launch_decode_concat(const void* cache, int64_t cache_bh_elems, const void* fresh, void* out, int BH, int L, int d, void* stream) {
  const int dv = d / 8;
  const int64_t total = (int64_t)BH * (L + 1) * dv;
  decode_concat_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>(
      (const dc_u32x4*)cache, cache_bh_elems / 8, (const dc_u32x4*)fresh, (dc_u32x4*)out, L, dv, total);
  return (int)hipGetLastError();
}

}  // namespace sm
