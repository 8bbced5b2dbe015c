// Linears on few rows: the chip is filled by cutting the OUTPUT COLUMNS of every Linear over workgroups, where the
// row-owning kernels of k_mlp.hip (a workgroup streams every weight of the block for its 32 or 64 tokens) would leave
// most compute units idle.  Two forms of one kernel:
//   single   one Linear (with LayerNorm folded, GELU, residual, row maps): one workgroup per output tile;
//   chained  the tail of a transformer block in one launch: output projection + residual, LayerNorm + FC1 + GELU,
//            FC2 + residual and, inside a stage, the next block's LayerNorm + QKV: up to four Linears whose tiles are
//            tasks of one ordered list.
//
// What bounds it: latency.  A tile is 32 or 64 rows x 32 or 64 columns; its operands (at most 128 KiB) are requested
// at once by LDS-DMA, so a task costs about one memory latency, one pass over LDS and one store latency.
// Measured: one image at C = 512 (196 tokens), attention + chain 31 us per block against 101 with the row-owning kernel; the
// rules for both forms carry their figures (split_tile below, split_tail_use in blocks.cpp).
//
// The chained form needs every row of a Linear's input before the next Linear starts.  Exchanging activations between
// workgroups through memory at device scope costs about 13 us per Linear (2.5 us each for the loads and the stores and
// 4 us for the flags, which all have to pass the XCDs' incoherent L2s; a kernel boundary costs 4), so a row never leaves
// its XCD: the rows are cut into groups, a group is claimed by an XCD (the one its workgroups read from the XCC_ID
// register), and all its tasks run there, exchanging through that XCD's L2: stores are acknowledged by the L2, flags are
// L2 atomics, and a reader invalidates its L1 (buffer_inv sc0) before it reads.  Every XCD streams all weights.
// Tasks of a group are numbered Linear by Linear.  A workgroup takes the next number from its XCD's counter, waits until
// the tasks it depends on (the previous Linear's tiles of its own rows: one arrival counter per Linear and row tile)
// have arrived, and runs it.  A number is only handed out to a running workgroup, every task depends on smaller numbers
// of the same counter only, and a workgroup finishes its task before it waits for the next: the smallest unfinished
// task of an XCD is always being worked on, so every wait ends whatever the number of resident workgroups and whatever
// else shares the GPU.  Groups are claimed one after the other, so all of them run however the workgroups are spread.
// split_order.h holds this order and what becomes of it when the counters are not what the launch left in them.
#include <algorithm>
#include <cstring>
#include "device_common.h"
#include "kernels.h"
#include "split.h"

namespace sm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 sp_bf16x8;
typedef float sp_f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int sp_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int sp_u32x2 __attribute__((ext_vector_type(2)));

#define SP_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define SP_LPTR(p) ((__attribute__((address_space(3))) void*)(p))
#define SP_LDS16(at) ((const __attribute__((address_space(3))) sp_u32x4*)(uintptr_t)(at))

// LDS accesses as assembly: next to outstanding LDS-DMA loads the compiler would wait for all of them first
__device__ __forceinline__ void lds_write16(unsigned addr, sp_u32x4 v) { asm volatile("ds_write_b128 %0, %1" ::"v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ sp_u32x4 lds_read16(unsigned addr) { sp_u32x4 v; asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr) : "memory"); return v; }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_mem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <typename T> __device__ __forceinline__ void sp_unpack(sp_u32x4 v, float* f) {
  if constexpr (sizeof(T) == 2) unpack8(v, f);
  else {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(v[e]);
  }
}
// CV adjacent elements as the words they take: to and from memory, and floats
template <typename T, int CV> struct SpRun {
  static constexpr int NWORD = CV * (int)sizeof(T) / 4, NV = NWORD / 4;      // words; 16-byte pieces of them
  unsigned w[NWORD];
  __device__ __forceinline__ void load(const T* p) {
    if constexpr (NV > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const sp_u32x4 q = ((const sp_u32x4*)p)[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * i + e] = q[e];
      }
    } else if constexpr (NWORD == 2) { const sp_u32x2 q = *(const sp_u32x2*)p; w[0] = q[0]; w[1] = q[1]; }
    else w[0] = *(const unsigned*)p;
  }
  __device__ __forceinline__ void store(T* p) const {
    if constexpr (NV > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) ((sp_u32x4*)p)[i] = sp_u32x4{w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]};
    } else if constexpr (NWORD == 2) *(sp_u32x2*)p = sp_u32x2{w[0], w[1]};
    else *(unsigned*)p = w[0];
  }
  __device__ __forceinline__ float get(int e) const {
    if constexpr (sizeof(T) == 2) return __uint_as_float(e & 1 ? w[e / 2] & 0xffff0000u : w[e / 2] << 16);
    else return __uint_as_float(w[e]);
  }
  __device__ __forceinline__ void pack(const float* f) {
#pragma unroll
    for (int i = 0; i < NWORD; ++i) {
      if constexpr (sizeof(T) == 2) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const f32x2 q = {f[2 * i], f[2 * i + 1]};
        w[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(q, bf16x2));
      } else w[i] = __float_as_uint(f[i]);
    }
  }
};
template <typename T> __device__ __forceinline__ sp_u32x4 sp_pack(const float* f) {
  if constexpr (sizeof(T) == 2) return pack8(f);
  sp_u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(f[e]);
  return o;
}

constexpr int NW = 8, NTHR = 64 * NW;      // waves of a tile: two per SIMD, so that one's LDS and vector latencies hide behind the other

// sum over groups of eight (N = 8) or sixteen adjacent lanes, by DPP
template <int N> __device__ __forceinline__ float lane_group_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));        // lane ^ 1
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true));        // lane ^ 2
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, true));                             // 7 - lane
  if constexpr (N == 16) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xf, 0xf, true));      // 15 - lane
  return v;
}
template <typename T, int MI, int NT>
__device__ __forceinline__ void split_norm(unsigned a_at, unsigned g_at, int nkt, int K, float eps) {
  constexpr int VEC = Elem<T>::VEC, BM = 32 * MI, TPR = NTHR / BM, TPT = TPR / 8;      // threads per row; K-tiles they take together
  const int r = threadIdx.x / TPR, p0 = threadIdx.x & 7, t1 = (threadIdx.x % TPR) >> 3;
  const unsigned row = a_at + r * 128 + p0 * 16, sw = (unsigned)((r >> 1) & 7);
  const int c0 = t1 * 8 + (int)(p0 ^ sw);                  // this thread's chunk of the row; the next ones are 8 TPT further on
  sp_u32x4 v[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) v[t] = lds_read16(row + min(t * TPT + t1, nkt - 1) * BM * 128);
  wait_lds();
  // gamma and beta: all on their way under the statistics where the row is short, else two pieces at a time where they are used.
  // Loads that the compiler sees (no LDS-DMA is outstanding here, for which it would wait): it may move or keep such a register across
  // the statistics as it likes, and waits before the first use of one
  constexpr int NG = NT <= 4 ? NT : 2;
  sp_u32x4 gv[NG], bv[NG];
  auto norm_load = [&](int u0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      const unsigned gc = min(c0 + (u0 + u) * 8 * TPT, K / VEC - 1);
      gv[u] = *SP_LDS16(g_at + gc * 16);
      bv[u] = *SP_LDS16(g_at + (K / VEC + gc) * 16);
    }
  };
  if constexpr (NG == NT) {
    norm_load(0);
    __builtin_amdgcn_sched_barrier(0);
  }
  // the row stays in fp32 registers between the passes where there is room (unpacked again for each, the norm of 32 x 512 took 2.0 us
  // of a task)
  constexpr bool HELD = NT * VEC <= 64;
  float x[HELD ? NT : 1][8], sum = 0.f, sq = 0.f;
  auto values = [&](int t, bool first) __attribute__((always_inline)) -> float* {
    float* f = x[HELD ? t : 0];
    if (!HELD || first) { asm volatile("" : "+v"(v[t])); sp_unpack<T>(v[t], f); }
    return f;
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bool in = (c0 + t * 8 * TPT) * VEC < K;
    const float* f = values(t, true);
    float part = 0.f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) part += f[e];
    sum += in ? part : 0.f;
  }
  const float mean = lane_group_sum<TPR>(sum) / (float)K;
  // a second pass for the variance: the mean of the squares minus the square of the mean loses the variance of a row
  // whose mean is large against its spread (768 elements of 100 and one of 100.5, all exact in bf16: nothing is left)
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bool in = (c0 + t * 8 * TPT) * VEC < K;
    float* f = values(t, false);
    float part = 0.f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) { f[e] -= mean; part += f[e] * f[e]; }
    sq += in ? part : 0.f;
  }
  const float rstd = rsqrtf(lane_group_sum<TPR>(sq) / (float)K + eps);
#pragma unroll
  for (int u0 = 0; u0 < NT; u0 += NG) {
    if (u0 * TPT >= nkt) break;
    if constexpr (NG != NT) norm_load(u0);
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      const int kt = (u0 + u) * TPT + t1;
      float* f = values(u0 + u, false);
      float g8[8], b8[8];
      sp_unpack<T>(gv[u], g8);
      sp_unpack<T>(bv[u], b8);
#pragma unroll
      for (int e = 0; e < VEC; ++e) f[e] = fmaf((HELD ? f[e] : f[e] - mean) * rstd, g8[e], b8[e]);
      if (kt < nkt) lds_write16(row + kt * BM * 128, sp_pack<T>(f));      // (chunks past K: never read)
    }
  }
}

// One task of `p`: rows row0 .. + 32 MI, columns ct * 32 WN .. + 32 WN.  Eight waves: WN along the columns, the other
// factor WK = 8 / WN cuts every group of K-tiles (their partial sums meet in LDS).  A K-tile is 128 bytes per row, held in LDS in
// 16-byte chunks at an XOR swizzle (chunk c of row r in slot c ^ ((r >> 1) & 7), conflict-free for the fragment reads).
//   RING = false: the whole A panel (32 MI x K) and W panel (32 WN x K) are resident; LN normalises the A panel in place;
//   RING = true:  four stages of KS K-tiles (no LN), for a K too long for that.
// CHAIN: a task of the chained form; a ninth wave (`ctl`) takes part in the barriers only.  keep (with LN): the workgroup's previous
// task was of the same Linear and rows, the normalised A panel is still there (the result tile lies over W then).
template <typename T, int MI, int WN, bool LN, bool RING, bool CHAIN, typename Next>
__device__ __forceinline__ void split_task(const SM_KARG LinPhase* p, int M, int row0, int ct, bool ctl, bool keep, unsigned lds_w, unsigned lds_g, unsigned lds_base, unsigned char* smem, Next&& next) {
  constexpr int VEC = Elem<T>::VEC, TILE = 8 * VEC, BM = 32 * MI, BN = 32 * WN, WK = NW / WN;
  constexpr int KS = 4 / MI, NS = 4;
  constexpr int EP = BN + 4;                               // pitch of the fp32 result tile
  // a thread finishes CV columns of a row: two, four or eight, so that all of them work (with eight for every tile, a quarter of them
  // did in a 32 x 32 one; with that and gamma and beta read ahead in the norm a net on one image takes 857 us instead of 884)
  constexpr int CV = BM * BN / NTHR, OPR = BN / CV;
  const int N = p->N, K = p->K;
  const int nkt = (K + TILE - 1) / TILE;
  const int nst = RING ? (nkt + KS - 1) / KS : 0;
  if (CHAIN && ctl) {
    wg_barrier();                                          // dependencies arrived
    wg_barrier();                                          // operands landed (RING: stage 0)
    if (LN && !keep) wg_barrier();
    if (RING) for (int s = 1; s < nst; ++s) wg_barrier();
    wg_barrier();                                          // main loop done
    wg_barrier();                                          // result tile in LDS
    next();
    wg_barrier();                                          // stores drained
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5, wn = wave % WN, wk = wave / WN;
  const int lrow = lane >> 3, lpos = lane & 7;
  const int n0 = ct * BN;
  const T* A = (const T*)p->A;

  // this lane's source row of A and of W: a wave-load is eight rows of a K-tile, the eight waves cover TA (TW) K-tiles
  constexpr int TA = 2 / MI, TW = 2 / WN;
  const int32_t* at = p->a_tab ? p->a_tab : (const int32_t*)p->W;      // (tables: looked up at once, waited for at their first use;
  const int ar = (wave % (4 * MI)) * 8 + lrow, agr = min(row0 + ar, M - 1), at1 = wave / (4 * MI);      //  without one, a valid word that is not used)
  const int araw = at[p->a_tab ? agr : 0];
  const int achk = lpos ^ ((ar >> 1) & 7);
  const T* asrc = A;
  auto load_a = [&](int kt, unsigned dst) {                // K-tile kt of the A rows to LDS address dst
    const int k = kt * TILE + achk * VEC;
    const T* s = asrc + (k < K ? k : kt * TILE);           // a chunk past K: any valid address, its k-steps are skipped
    __builtin_amdgcn_global_load_lds(SP_GPTR(s), SP_LPTR(smem + dst + (wave % (4 * MI)) * 1024), 16, 0, 0);
  };
  const int wr = (wave % (4 * WN)) * 8 + lrow, wt1 = wave / (4 * WN);
  const T* wsrc = (const T*)p->W + (int64_t)min(n0 + wr, N - 1) * K;
  const int wchk = lpos ^ ((wr >> 1) & 7);
  auto load_w = [&](int kt, unsigned dst) {
    const int k = kt * TILE + wchk * VEC;
    const T* s = wsrc + (k < K ? k : kt * TILE);
    __builtin_amdgcn_global_load_lds(SP_GPTR(s), SP_LPTR(smem + dst + (wave % (4 * WN)) * 1024), 16, 0, 0);
  };
  constexpr unsigned ATB = BM * 128, WTB = BN * 128;       // bytes of a K-tile

  // where this thread's results go, and everything else that comes through registers: requested before the weights, so
  // that waiting for it is not waiting for them
  const int32_t* ot = p->o_tab ? p->o_tab : (const int32_t*)p->W;
  const int32_t* rt = p->r_tab ? p->r_tab : (const int32_t*)p->W;
  const int orow = row0 + tid / OPR, ocol = n0 + (tid % OPR) * CV, og = min(orow, M - 1), oc = min(ocol, N - CV);
  const int oraw = ot[p->o_tab ? og : 0], rraw = rt[p->r_tab ? og : 0];
  SpRun<T, CV> bias;
  bias.load(p->bias ? (const T*)p->bias + oc : (const T*)p->W);      // (no bias: any valid words, not used)

  if (LN && !keep) {
    const int nch = K / VEC;
    for (int c0 = wave * 64; c0 < nch; c0 += NTHR)
      if (c0 + lane < nch) {
        __builtin_amdgcn_global_load_lds(SP_GPTR((const sp_u32x4*)p->ln_g + c0 + lane), SP_LPTR(smem + lds_g + c0 * 16), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(SP_GPTR((const sp_u32x4*)p->ln_b + c0 + lane), SP_LPTR(smem + lds_g + (nch + c0) * 16), 16, 0, 0);
      }
  }
  asm volatile("" ::: "memory");
  // weights do not depend on other tasks: requested before the dependencies are waited for
  if constexpr (RING) {
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
#pragma unroll
      for (int i = wt1; i < KS; i += TW) load_w(min(s * KS + i, nkt - 1), lds_w + (s * KS + i) * WTB);
  } else {
    for (int kt = wt1; kt < nkt; kt += TW) load_w(kt, lds_w + kt * WTB);
  }
  if constexpr (CHAIN) {
    wg_barrier();                                          // the tasks this one depends on have arrived
    asm volatile("buffer_inv sc0" ::: "memory");           // their results are in this XCD's L2: drop what this CU's L1 holds
  }
  asrc = A + (p->a_tab ? (int64_t)araw * p->a_mul : (int64_t)agr * p->a_ld);
  SpRun<T, CV> res;
  if (p->res) res.load((const T*)p->res + (p->r_tab ? (int64_t)rraw : (int64_t)og * p->r_ld) + oc);
  else {
#pragma unroll
    for (int i = 0; i < SpRun<T, CV>::NWORD; ++i) res.w[i] = 0u;
  }
  sp_f32x16 acc[MI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[mi][i] = 0.f;

  // KS K-tiles from tile kt0 on, whose A / W tiles lie at LDS addresses a_at / w_at: this wave's k-steps of each
  auto compute = [&](int kt0, unsigned a_at, unsigned w_at) {
    constexpr int NST = KS * 4 / WK;                       // k-steps (two chunks each) of the group that are this wave's
    sp_u32x4 fa[NST][MI], fw[NST];
    const unsigned sw = (unsigned)((l32 >> 1) & 7);
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      const int t = (wk * NST + s) >> 2, j = (wk * NST + s) & 3;
      const unsigned c = ((unsigned)(2 * j + hf) ^ sw) << 4;
      fw[s] = lds_read16(lds_base + w_at + t * WTB + (wn * 32 + l32) * 128 + c);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) fa[s][mi] = lds_read16(lds_base + a_at + t * ATB + (mi * 32 + l32) * 128 + c);
    }
    wait_lds();
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      asm volatile("" : "+v"(fw[s]));
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) asm volatile("" : "+v"(fa[s][mi]));
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      const int t = (wk * NST + s) >> 2, j = (wk * NST + s) & 3;
      if ((kt0 + t) * TILE + j * 2 * VEC < K) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
          if constexpr (sizeof(T) == 2) {
            acc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sp_bf16x8, fw[s]), __builtin_bit_cast(sp_bf16x8, fa[s][mi]), acc[mi], 0, 0, 0);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[mi] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fw[s][e]), __uint_as_float(fa[s][mi][e]), acc[mi], 0, 0, 0);
          }
        }
      }
    }
  };

  if constexpr (!RING) {
    if (!keep)
      for (int kt = at1; kt < nkt; kt += TA) load_a(kt, kt * ATB);
    wait_mem();
    wg_barrier();
    if (LN && !keep) {
      // LayerNorm of the A panel in place: TPR threads per row, each with its chunks in registers (one pass over LDS), fp32
      // two-pass statistics, rounded as a norm kernel stores it
      if (nkt <= 4 * TA) split_norm<T, MI, 4>(lds_base, lds_base + lds_g, nkt, K, p->eps);
      else if (nkt <= 8 * TA) split_norm<T, MI, 8>(lds_base, lds_base + lds_g, nkt, K, p->eps);
      else if constexpr (!CHAIN) split_norm<T, MI, 12>(lds_base, lds_base + lds_g, nkt, K, p->eps);      // (the chain's rows are 8 TA K-tiles at most)
      wg_barrier();
    }
    for (int kt = 0; kt < nkt; kt += KS) compute(kt, kt * ATB, lds_w + kt * WTB);
  } else {
    constexpr int LA = KS / TA, LW = KS / TW;              // a wave's loads per stage
    auto stage_a = [&](int s) {
#pragma unroll
      for (int i = at1; i < KS; i += TA) load_a(min(s * KS + i, nkt - 1), ((s % NS) * KS + i) * ATB);
    };
    auto stage_w = [&](int s) {
#pragma unroll
      for (int i = wt1; i < KS; i += TW) load_w(min(s * KS + i, nkt - 1), lds_w + ((s % NS) * KS + i) * WTB);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) stage_a(s);           // (a stage past the end repeats the last K-tile: the counts below stay exact)
    for (int s = 0; s < nst; ++s) {
      // stage s has landed once at most the younger loads are outstanding: NS - 2 stages' A loads right after the start,
      // NS - 2 whole stages later, and fewer when nothing more is issued
      if (s < NS - 1 && s + NS - 2 <= max(NS - 2, nst - 1)) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * LA) : "memory");
      else if (s + NS - 2 < nst) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * (LA + LW)) : "memory");
      else wait_mem();
      wg_barrier();
      if (s + NS - 1 < nst) { stage_w(s + NS - 1); stage_a(s + NS - 1); }      // into the stage read last before this barrier
      compute(s * KS, (s % NS) * KS * ATB, lds_w + (s % NS) * KS * WTB);
    }
    wait_mem();
  }

  // the partial sums of the WK wave groups, through LDS (over the A panel, over W where A may be kept): lane owns row mi 32 + l32, columns
  // wn 32 + 8 g4 + 4 hf .. + 3
  const unsigned r_at = lds_base + (CHAIN && LN ? lds_w : 0u);
  wg_barrier();
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4)
      lds_write16(r_at + (((wk * BM + mi * 32 + l32) * EP) + wn * 32 + g4 * 8 + hf * 4) * 4,
                  sp_u32x4{__float_as_uint(acc[mi][4 * g4]), __float_as_uint(acc[mi][4 * g4 + 1]), __float_as_uint(acc[mi][4 * g4 + 2]), __float_as_uint(acc[mi][4 * g4 + 3])});
  wg_barrier();
  // the thread's columns of the WK sums, in their order
  constexpr int PW = CV < 4 ? CV : 4;                      // words per read
  typedef unsigned int Part __attribute__((ext_vector_type(PW)));
  Part part[WK][CV / PW];
#pragma unroll
  for (int w = 0; w < WK; ++w)
#pragma unroll
    for (int e = 0; e < CV / PW; ++e) {
      const unsigned at = r_at + ((w * BM + tid / OPR) * EP + (tid % OPR) * CV + e * PW) * 4;
      if constexpr (PW == 4) asm volatile("ds_read_b128 %0, %1" : "=v"(part[w][e]) : "v"(at) : "memory");
      else asm volatile("ds_read_b64 %0, %1" : "=v"(part[w][e]) : "v"(at) : "memory");
    }
  wait_lds();
  float v[CV];
#pragma unroll
  for (int w = 0; w < WK; ++w)
#pragma unroll
    for (int e = 0; e < CV / PW; ++e) {
      asm volatile("" : "+v"(part[w][e]));
#pragma unroll
      for (int x = 0; x < PW; ++x) v[e * PW + x] = (w ? v[e * PW + x] : 0.f) + __uint_as_float(part[w][e][x]);
    }
  if (p->bias) {
#pragma unroll
    for (int e = 0; e < CV; ++e) v[e] += bias.get(e);
  }
  if (p->act == SM_ACT_GELU) {
#pragma unroll
    for (int e = 0; e < CV; ++e) v[e] = sizeof(T) == 2 ? gelu_poly(v[e]) : gelu_erf(v[e]);
  }
#pragma unroll
  for (int e = 0; e < CV; ++e) v[e] += res.get(e);
  if (orow < M && ocol < N) {
    SpRun<T, CV> out;
    out.pack(v);
    out.store((T*)p->out + (p->o_tab ? (int64_t)oraw * p->o_mul : (int64_t)orow * p->o_ld) + ocol);
  }
  if constexpr (CHAIN) { wait_mem(); wg_barrier();}
}

__device__ __forceinline__ unsigned lds_offset(const void* p) { return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)p; }

// one Linear.  Every XCD takes a run of the tiles, so that tiles that share a panel run behind one L2: in column-major order
// (the panels of W), in row-major order where there are more than twice as many row tiles as column tiles.  A tall result cut
// by columns leaves every row, and with narrow rows every cache line, in two L2s, and the kernel that reads it pays (a block of
// C = 96 on 6272 tokens 38.0 us by rows, 44.5 by columns; C = 192, 3136 tokens 44.9 / 51.4; fp32 C = 96, 3136 tokens 58.0 / 65.7)
template <typename T, int MI, int WN, bool LN, bool RING>
__global__ __launch_bounds__(NTHR) void split_single_kernel(SplitArgs a) {
  const SM_KARG SplitArgs* g = kernarg_ptr<SplitArgs>();
  extern __shared__ __align__(16) unsigned char sp_smem[];
  const int at = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const bool tall = g->tiles_m > 2 * g->tiles_n[0];
  const int minor = tall ? g->tiles_n[0] : g->tiles_m, major = at / minor, rest = at - major * minor;
  const int ct = tall ? rest : major, rt = tall ? major : rest;
  if (ct >= g->tiles_n[0] || rt >= g->tiles_m) return;
  split_task<T, MI, WN, LN, RING, false>(&g->ph[0], g->M, rt * 32 * MI, ct, false, false, g->lds_w, g->lds_g, lds_offset(sp_smem), sp_smem, [] {});
}

// Counters: read-modify-write at the L2, also to look at one (as assembly: the compiler turns an addition of zero into
// a load, which could be served by the L1 for ever)
__device__ __forceinline__ int l2_add(int* p, int v) {
  int old;
  asm volatile("global_atomic_add %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=&v"(old) : "v"(p), "v"(v) : "memory");
  return old;
}

struct L2Mem {
  static __device__ __forceinline__ int take(int* p, int v) { return l2_add(p, v); }
  static __device__ __forceinline__ int look(int* p) { return l2_add(p, 0); }
  static __device__ __forceinline__ int take_device(int* p, int v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  static __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(1); }
};

// the chain: one more wave takes task numbers, waits for dependencies and reports arrivals (split_order.h)
template <typename T, int MI, int WNL>
__global__ __launch_bounds__(NTHR + 64) void split_chain_kernel(SplitArgs a) {
  const SM_KARG SplitArgs* g = kernarg_ptr<SplitArgs>();
  extern __shared__ __align__(16) unsigned char sp_smem[];
  int* slot = (int*)(sp_smem + g->lds_slot);               // [2][task, group]
  constexpr int WNP = MI;                                  // columns per wave group of the unnormalised Linears
  const bool ctl = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == NW;
  const unsigned base = lds_offset(sp_smem);
  int* mine = g->counters + SPLIT_LINE * (1 + (__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15));      // hwreg XCC_ID: this XCD's number counter and claims
  TaskOrder order{g->counters, mine, (unsigned)g->group_tasks, g->n_groups, SPLIT_SPINS, ~0u, 0, false};
  if (threadIdx.x == NTHR) task_of<L2Mem>(order, (unsigned)l2_add(mine, 1), slot);
  wg_barrier();
  int last_ph = -1, last_rt = -1;
  for (int it = 0;; ++it) {
    const int k = __builtin_amdgcn_readfirstlane(slot[2 * (it & 1)]), grp = __builtin_amdgcn_readfirstlane(slot[2 * (it & 1) + 1]);
    if (k < 0) break;
    int ph = 0;
    while (k >= g->first[ph + 1]) ++ph;
    const int rem = k - g->first[ph];
    const int ct = rem / g->group_rows, rl = rem - ct * g->group_rows, rt = grp * g->group_rows + rl;
    const SM_KARG LinPhase* p = &g->ph[ph];
    int* done = g->counters + SPLIT_LINE * 17 + grp * g->group_words + rl;
    const bool keep = ph == last_ph && rt == last_rt && p->ln_g;      // (what it depends on has arrived already)
    last_ph = ph; last_rt = rt;
    if (ctl && threadIdx.x == NTHR && ph && !keep) wait_arrivals<L2Mem>(order, done + (ph - 1) * g->group_rows, g->tiles_n[ph - 1]);
    // the next number is asked for now and looked at when this task's results are on their way
    int n_next = 0;
    if (ctl && threadIdx.x == NTHR) n_next = __hip_atomic_fetch_add(mine, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto next = [&] { if (threadIdx.x == NTHR) task_of<L2Mem>(order, (unsigned)n_next, slot + 2 * ((it + 1) & 1)); };
    const int row0 = rt * 32 * MI;
    if (p->ln_g) split_task<T, MI, WNL, true, false, true>(p, g->M, row0, ct, ctl, keep, g->lds_w, g->lds_g, base, sp_smem, next);
    else if (p->ring) split_task<T, MI, WNP, false, true, true>(p, g->M, row0, ct, ctl, keep, g->lds_w, g->lds_g, base, sp_smem, next);
    else split_task<T, MI, WNP, false, false, true>(p, g->M, row0, ct, ctl, keep, g->lds_w, g->lds_g, base, sp_smem, next);
    if (ctl && threadIdx.x == NTHR) asm volatile("global_atomic_add %0, %1, off" ::"v"(done + ph * g->group_rows), "v"(1) : "memory");
  }
}

// a pitch or a table, whose offsets are whole vectors (sufficient: the pitch, or the program's constant and coefficients are)
static bool split_rows_ok(const RowProg& r, int vec) {
  if (r.identity) return r.ld <= INT32_MAX && r.ld % vec == 0;
  if (!r.table || r.c0 % vec) return false;
  for (int t = 0; t < r.nterm; ++t)
    if (r.t_coef[t] % vec) return false;
  return true;
}

namespace {
constexpr size_t kLds = 160 * 1024;
struct Layout { size_t w, g, total; };       // LDS: [A], [W], [norm constants]; the result tile over them
size_t up(size_t a, size_t b) { return (a + b - 1) / b * b; }
// A (or result tile, whichever is larger) and W bytes of one Linear in a tile of 32 mi rows x 32 wn columns
void need(int K, int es, int mi, int wn, bool ln, bool ring, size_t* a, size_t* w, size_t* g) {
  const int ks = 4 / mi;
  const size_t tiles = ring ? 4 * (size_t)ks : up(((size_t)K * es + 127) / 128, ks);
  const int wk = NW / wn;
  *a = std::max(tiles * 32 * mi * 128, (size_t)wk * 32 * mi * (32 * wn + 4) * 4);
  *w = tiles * 32 * wn * 128;
  *g = ln ? (size_t)2 * K * es : 0;
}
template <typename F> int set_lds(F f, size_t bytes) {
  return (int)hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <typename T, int MI, int WN, bool LN, bool RING>
int single_launch(SplitArgs& a, const Layout& l, hipStream_t s) {
  static const int attr = set_lds(split_single_kernel<T, MI, WN, LN, RING>, kLds);
  if (attr) return attr;
  a.tiles_m = (a.M + 32 * MI - 1) / (32 * MI);
  a.tiles_n[0] = (a.ph[0].N + 32 * WN - 1) / (32 * WN);
  const int64_t grid = ((int64_t)a.tiles_n[0] * a.tiles_m + 7) / 8 * 8;
  if (grid > INT32_MAX) return (int)hipErrorInvalidValue;
  split_single_kernel<T, MI, WN, LN, RING><<<dim3((unsigned)grid), dim3(NTHR), l.total, s>>>(a);
  return (int)hipGetLastError();
}
template <typename T>
int single_pick(SplitArgs& a, int mi, int wn, hipStream_t s) {
  const LinPhase& p = a.ph[0];
  size_t ab, wb, gb;
  need(p.K, (int)sizeof(T), mi, wn, p.ln_g != nullptr, p.ring, &ab, &wb, &gb);
  // the result tile takes the place of both panels and the norm constants, all dead by then: two workgroups per CU where the
  // panels are short (fp32, 3136 x 384 x 96 + LN + GELU, 294 tiles: 14.5 us with one)
  const size_t panel = wb / (32 * wn) * (32 * mi);
  const Layout l{panel, panel + wb, std::max(ab, panel + wb + gb)};
  if (l.total > kLds || (p.ln_g && (size_t)p.K * sizeof(T) > (size_t)12 * 128 * (2 / mi))) return (int)hipErrorInvalidValue;
  a.lds_w = (unsigned)l.w; a.lds_g = (unsigned)l.g;
#define SP_CASE(MI_, WN_) \
  if (mi == MI_ && wn == WN_) return p.ln_g ? single_launch<T, MI_, WN_, true, false>(a, l, s) : (p.ring ? single_launch<T, MI_, WN_, false, true>(a, l, s) : single_launch<T, MI_, WN_, false, false>(a, l, s));
  SP_CASE(1, 1) SP_CASE(1, 2) SP_CASE(2, 2)
#undef SP_CASE
  return (int)hipErrorInvalidValue;
}
template <int MI, int WNL>
int chain_launch(const SplitArgs& a, size_t lds, int grid, hipStream_t s) {
  static const int attr = set_lds(split_chain_kernel<bf16_t, MI, WNL>, kLds);
  if (attr) return attr;
  split_chain_kernel<bf16_t, MI, WNL><<<dim3((unsigned)grid), dim3(NTHR + 64), lds, s>>>(a);
  return (int)hipGetLastError();
}
}  // namespace

int launch_split_single(SplitArgs& a, int dtype, int mi, int wn, void* stream) {
  return dtype == SM_F32 ? single_pick<float>(a, mi, wn, (hipStream_t)stream) : single_pick<bf16_t>(a, mi, wn, (hipStream_t)stream);
}

// Which Linears run in this form, and in which tile (32 mi x 32 wn; mi = 0: none).  The smallest tile whose grid is
// about one round of workgroups on the 256 CUs.  Beyond that: bf16, the tiled kernel of k_gemm.hip with its lower traffic
// per flop (from 256 tiles of 64 x 64 on; measured us, this form / the tiled one: 196 x 1536 x 512 + LN 5.8 / 12.2,
// 3136 x 192 x 192 4.1 / 5.0, 50 x 768 x 3072 7.4 / 19.7, 64 x 4096 x 11008 32 / 142; but 784 x 1536 x 512 + LN 12.9 / 12.3,
// 3136 x 768 x 192 9.6 / 6.5; long K, a second round: 333 x 4096 x 11008 76 / 53, 500 x 4096 x 4096 34 / 25, 342 x 3072 x 2048 19 / 12); fp32, whose matrix instructions
// are sixteen times slower so that a task is longer than its latencies, up to three rounds of 64 x 64 tiles
// (3136 x 288 x 96 + LN 6.9 / 13.1, 784 x 384 x 1536 24 / 67, 12544 x 96 x 96 10.2 / 12.3, 3466 x 768 x 1536 97 / 112, 23466 x 96 x 96 + LN
// 17.6 / 18.7), a fourth only where the tiled kernel's 128 columns are half empty (57600 x 32 x 3072 244 / 399, but 6400 x 512 x 768
// 70 / 62, 2133 x 1536 x 1536 127 / 112, 50176 x 96 x 384 75 / 67).  Narrower tiles while the grid is one round: with a ring up to 320
// (620 x 512 x 288 8.8, against 9.3 in 64 x 64 tiles; 540 of them, 1440 x 384 x 384, 13.4 against 10.8); under LayerNorm from K = 384 on,
// whose 64-row panels do not fit, up to two and a half rounds of 32 x 64 (3306 x 384 x 384 + LN 26 / 29, 1546 x 768 x 384 + LN 23.6 / 27.6;
// 2311 x 1152 x 384 + LN, five rounds, 46.4 / 44.5).
// Rows under LayerNorm whose panels of 64 rows or columns do not fit LDS (wide ones): wide_norm_split below.
struct SplitTile { int mi, wn; };
static SplitTile split_tile(int64_t M, int N, int K, int dtype, bool ring) {
  const int64_t t11 = ((M + 31) / 32) * ((N + 31) / 32), t12 = ((M + 31) / 32) * ((N + 63) / 64), t22 = ((M + 63) / 64) * ((N + 63) / 64);
  if (t11 <= (ring && dtype == SM_F32 ? 320 : 256)) return {1, 1};
  if (!ring && t12 <= 256) return {1, 2};
  if (t22 <= 256) return {2, 2};
  if (dtype != SM_F32) return {0, 0};
  if (!ring && t12 <= 640 && K >= 384) return {1, 2};
  return t22 <= (N <= 64 ? 1024 : 768) ? SplitTile{2, 2} : SplitTile{0, 0};
}
static bool split_fits(const SplitTile& t, int K, int es, bool ln, bool ring) {
  size_t ab, wb, gb;
  need(K, es, t.mi, t.wn, ln, ring, &ab, &wb, &gb);
  return ab + wb + gb <= kLds && (!ln || (size_t)K * es <= (size_t)12 * 128 * (2 / t.mi));
}
// LayerNorm over a wide row in 32 x 32 tiles, one workgroup per CU: by rounds of 256 tiles against the tiled kernel with its
// folded norm, whose time grows with K and hardly with the tiles.  Measured us, this form / the tiled one, bf16: K = 576, three
// rounds (300 x 1728) 16.5 / 13.8; K = 768, 576 tiles (245 x 2304) 16.3 / 16.6, 600 (784 x 768) 17.0 / 16.5, 672 (196 x 3072)
// 17.7 / 16.8; K = 896, three rounds (700 x 896) 17.9 / 18.4; K = 1024, two (500 x 1024) 13.2 / 20.3, three (196 x 3072) 19.0 / 20.8,
// four (784 x 1024) 24.0 / 20.4.  fp32: K = 512, four (2560 x 320) 29.7 / 33.5, five (5760 x 192) 39.5 / 33.6; K = 288, seven
// (1066 x 1536) 35.5 / 24.1.
static bool wide_norm_split(int64_t t11, int K, int dtype) { return t11 <= (dtype == SM_F32 ? 1024 : (K > 768 ? 768 : (K == 768 ? 576 : 512))); }
static bool split_linear_plan(const GemmArgs& g, SplitTile* t, bool* ring) {
  const int es = g.dtype == SM_F32 ? 4 : 2, vec = 16 / es;
  if (g.a_gran > 0 || g.rope_cols || g.c_transposed || g.c_cols_on || g.C2 || g.norm == 2 || (g.act != SM_ACT_NONE && g.act != SM_ACT_GELU)) return false;
  if (g.M > INT32_MAX / 2 || g.ldw != g.K || g.K % (2 * vec) || g.N % 8 || g.N < 8 || !split_rows_ok(g.a_rows, vec) || !split_rows_ok(g.c_rows, vec)) return false;
  if (g.norm && !g.norm_beta) return false;
  *ring = !g.norm && (size_t)g.K * es > 1024;
  *t = split_tile(g.M, g.N, g.K, g.dtype, *ring);
  if (t->mi && split_fits(*t, g.K, es, g.norm != 0, *ring)) return true;
  *t = SplitTile{1, 1};
  return g.norm && split_fits(*t, g.K, es, true, false) && wide_norm_split(((g.M + 31) / 32) * ((g.N + 31) / 32), g.K, g.dtype);
}
bool split_linear_use(const GemmArgs& g) { SplitTile t; bool ring; return split_linear_plan(g, &t, &ring); }
bool launch_split_linear(const GemmArgs& g, void* stream, int* rc) {
  SplitTile t; bool ring;
  if (!split_linear_plan(g, &t, &ring)) return false;
  SplitArgs a; std::memset(&a, 0, sizeof(a));
  a.M = (int)g.M; a.n_ph = 1;
  LinPhase& p = a.ph[0];
  p.A = g.A; p.W = g.W; p.bias = g.bias; p.res = g.residual; p.out = g.C; p.N = g.N; p.K = g.K; p.act = g.act; p.ring = ring;
  if (g.norm) { p.ln_g = g.norm_gamma; p.ln_b = g.norm_beta; p.eps = g.norm_eps; }
  p.a_tab = g.a_rows.identity ? nullptr : g.a_rows.table; p.a_ld = (int)g.a_rows.ld;
  p.o_tab = p.r_tab = g.c_rows.identity ? nullptr : g.c_rows.table; p.o_ld = p.r_ld = (int)g.c_rows.ld; p.a_mul = p.o_mul = 1;
  *rc = launch_split_single(a, g.dtype, t.mi, t.wn, stream);
  return true;
}

// counters: [groups claimed] [per XCD: next number, group of each run of numbers] [per group: arrivals per Linear and row tile]
namespace {
struct Groups { int rows, n, words; };      // row tiles per group, groups, counters per group
Groups groups_of(int64_t M, int mi) {
  const int tiles = (int)((M + 32 * mi - 1) / (32 * mi));
  Groups g;
  g.rows = (tiles + 7) / 8;                 // one group per XCD
  g.n = (tiles + g.rows - 1) / g.rows;
  g.words = (int)up(4 * (size_t)g.rows, SPLIT_LINE);
  return g;
}
}
size_t split_counter_ints(int64_t M) {
  const Groups g = groups_of(M, 1);         // the narrower tiles have the most counters
  return SPLIT_LINE * 17 + (size_t)g.n * g.words + SPLIT_LINE;
}

int launch_split_chain(SplitArgs& a, int* counters, int mi, void* stream) {
  const Groups gr = groups_of(a.M, mi);
  a.group_rows = gr.rows; a.n_groups = gr.n; a.group_words = gr.words; a.counters = counters;
  int kmax = 0;
  for (int i = 0; i < a.n_ph; ++i) if (a.ph[i].ln_g) kmax = std::max(kmax, a.ph[i].K);
  if (kmax > (mi == 2 ? 512 : 1024)) return (int)hipErrorInvalidValue;      // rows under LayerNorm: 8 K-tiles per thread of split_norm
  const int wnl = mi == 2 || kmax <= 512 ? 2 : 1;
  size_t ab = 0, wb = 0, gb = 0;
  int most = 0;
  a.first[0] = 0;
  for (int i = 0; i < a.n_ph; ++i) {
    const int wn = a.ph[i].ln_g ? wnl : mi;
    size_t x, y, z;
    need(a.ph[i].K, 2, mi, wn, a.ph[i].ln_g != nullptr, a.ph[i].ring, &x, &y, &z);
    if (a.ph[i].ln_g) { const size_t panel = y / (32 * wn) * (32 * mi); y = std::max(y, x); x = panel; }      // the result tile over W
    ab = std::max(ab, x); wb = std::max(wb, y); gb = std::max(gb, z);
    a.tiles_n[i] = (a.ph[i].N + 32 * wn - 1) / (32 * wn);
    a.first[i + 1] = a.first[i] + a.tiles_n[i] * gr.rows;
    most = std::max(most, a.tiles_n[i] * gr.rows);
  }
  const size_t lds = ab + wb + gb + 16;
  if (lds > kLds) return (int)hipErrorInvalidValue;
  a.lds_w = (unsigned)ab; a.lds_g = (unsigned)(ab + wb); a.lds_slot = (unsigned)(ab + wb + gb);
  a.group_tasks = a.first[a.n_ph];
  const int grid = 8 * std::min(most, 32);
  hipStream_t s = (hipStream_t)stream;
  if (mi == 2) return chain_launch<2, 2>(a, lds, grid, s);
  return wnl == 2 ? chain_launch<1, 2>(a, lds, grid, s) : chain_launch<1, 1>(a, lds, grid, s);
}

}  // namespace sm
