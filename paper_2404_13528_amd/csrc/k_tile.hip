// Mapped Linear, large tiles: the bf16 products of launch_gemm whose grid fills the chip with tiles of 128 .. 256 rows and
// columns (tile_linear_plan below says which).  Same epilogues as gemm_kernel (k_gemm.hip) and the same sums in the same order: a
// choice between the two never changes a result.  Rows of A at a pitch (who gathers them folds a norm in as well, which is
// gemm_kernel's), rows of the result and residual at a pitch or by a table of offsets.
//
// What bounds it: the LDS.  A wave that owns 64 x 64 outputs reads 1 KiB of fragments per 32 x 32 x 16 MFMA, which at eight waves
// and 128 bytes a clock is more LDS time than matrix time; 128 x 128 outputs per wave need half of it, 96 x 96 two thirds, and the
// L2 -> LDS traffic per flop falls the same way.  So a workgroup is four waves (2 x 2), one per SIMD, with (32 MI) x (32 NI)
// outputs each (up to 256 accumulator registers), and nothing but the wave's own instruction order hides latencies:
//   - a K-tile is 128 bytes per row, in LDS in 16-byte chunks at the XOR swizzle of gemm_kernel, filled by LDS-DMA; its rows are
//     two halves, A0 / A1 and B0 / B1 (each wave's first and last blocks), and a K-tile is multiplied in four phases, A0 B0, A0 B1,
//     A1 B0, A1 B1, each over the whole depth of the tile;
//   - a phase's operands are read into registers during earlier phases (B1 in the first, A1 in the second, the next K-tile's A0 and
//     B0 in the last two), between the MFMAs: after two phases every fragment of the tile is in registers and its stage is free;
//   - the K-tile NS further on is requested into it a quarter per phase (A0, B0 in the last two phases, A1, B1 in the next tile's
//     first two), so that the L2 -> LDS path, which takes half as long for a tile's bytes as the matrix cores for its flops, is
//     never asked for a whole tile at once (all of it in one phase: 4096^3 in 256 x 256 tiles 111 us);
//   - two barriers per K-tile, each behind a wait for loads that are at least two phases old;
//   - the stream of K-tiles runs on over output tiles: the last steps of a tile request the first K-tiles of the workgroup's next
//     one, which arrive behind the epilogue (which has LDS of its own).
#include <algorithm>
#include <type_traits>
#include "device_common.h"
#include "kernels.h"
#include "tile.h"

namespace sm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 tl_bf16x8;
typedef float tl_f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int tl_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int tl_u32x2 __attribute__((ext_vector_type(2)));
typedef float tl_f32x2 __attribute__((ext_vector_type(2)));
typedef float tl_f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 tl_bf16x2 __attribute__((ext_vector_type(2)));

#define TL_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define TL_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

namespace {

struct TileGrid { int tiles_m, tiles_n, strip, group; int splits, nk, nk_more; float* part; };      // the last four: EPI_PART only
struct TileCols { int half, rope_cols, rope_dim; };
// EPI_PART: K is cut into `splits` runs of `nk` K-tiles (one more in the first `nk_more`), one workgroup per tile and run, and the
// sums of run s are left in fp32 at part[s M N + r N + n] for sum_parts_kernel
enum { EPI_PLAIN = 0, EPI_GELU = 1, EPI_GLU = 2, EPI_ROPE = 3, EPI_PART = 4 };
// order of the logical columns: a block of 32 is two runs of 16 columns of W that belong together (GLU: value and gate of 16
// outputs; ROPE: 16 first and 16 second members of rotary pairs; else 32 adjacent columns), so that partners sit in one lane
template <int EPI> __device__ __forceinline__ int tile_col(const TileCols& cm, int n) {
  if (EPI == EPI_GLU) return (n & 16 ? cm.half : 0) + (n >> 5) * 16 + (n & 15);
  if (EPI == EPI_ROPE && n < cm.rope_cols) {
    const int head = n / cm.rope_dim, u = n - head * cm.rope_dim;
    return head * cm.rope_dim + (u >> 5) * 16 + (u & 15) + (u & 16 ? cm.rope_dim >> 1 : 0);
  }
  return n;
}
// LDS accesses as assembly: next to outstanding LDS-DMA loads the compiler would wait for all of them first
__device__ __forceinline__ void lds_write8(unsigned at, int off, tl_u32x2 v) { asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(at), "v"(v), "n"(off) : "memory"); }
// an accumulator register's value.  As assembly, so that the accumulators stay where they are until their turn comes (the compiler
// copies all of them to vector registers after the K loop, and spills); the caller has waited for the last MFMA
__device__ __forceinline__ float acc_read(float a) { float v; asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a)); return v; }

// stages of K-tiles; blocks of 32 columns that a wave stores at a time (their LDS beside the stages: 32 rows of 16 PIECES + 16 bytes per wave)
constexpr int tile_stages(int mi, int ni) { return mi + ni >= 7 ? 2 : 3; }
constexpr int tile_chunk(int mi, int ni, int epi) { return epi == EPI_GLU ? (mi == 2 && ni == 4 ? 2 : ni) : (ni % 2 || mi + ni == 6 ? 1 : 2); }
constexpr int tile_pieces(int mi, int ni, int epi) { return tile_chunk(mi, ni, epi) * (epi == EPI_GLU ? 2 : 4); }
constexpr size_t tile_lds(int mi, int ni, int epi) {
  return (size_t)tile_stages(mi, ni) * 64 * (mi + ni) * 128 + 4 * 32 * (tile_pieces(mi, ni, epi) * 16 + 16);
}

template <int MI, int NI, int EPI>
__global__ __launch_bounds__(256, 1) void tile_kernel(GemmArgs g, TileCols cm, TileGrid ts) {
  constexpr int BM = 64 * MI, BN = 64 * NI, A_BYTES = BM * 128, STAGE = (BM + BN) * 128, NS = tile_stages(MI, NI);
  constexpr int LA = 2 * MI, LB = 2 * NI, LPT = LA + LB;      // wave-loads (8 rows, 1 KiB) of a wave per K-tile
  constexpr int MA0 = (MI + 1) / 2, MA1 = MI - MA0, NB0 = (NI + 1) / 2, NB1 = NI - NB0;      // blocks of a wave in each half
  constexpr int H0 = 2 * (MA0 + NB0), H1 = LPT - H0;
#define TL_PIN(x) asm volatile("" : "+s"(x))
  int c_ident = g.c_rows.identity, n_cols = g.N;
  int64_t a_ld = g.a_rows.ld, c_ld = g.c_rows.ld, m_rows = g.M, ldw = g.ldw;
  const int32_t* c_tab = g.c_rows.table;
  const void* bias_p = g.bias;
  const void* res_p = g.residual;
  void* c_p = g.C;
  TL_PIN(c_ident); TL_PIN(n_cols); TL_PIN(a_ld); TL_PIN(c_ld); TL_PIN(m_rows); TL_PIN(ldw);
  TL_PIN(c_tab); TL_PIN(bias_p); TL_PIN(res_p); TL_PIN(c_p);
  TL_PIN(cm.half); TL_PIN(cm.rope_cols); TL_PIN(cm.rope_dim);
  TL_PIN(ts.tiles_m); TL_PIN(ts.tiles_n); TL_PIN(ts.strip); TL_PIN(ts.group);
  if constexpr (EPI == EPI_PART) { TL_PIN(ts.splits); TL_PIN(ts.nk); TL_PIN(ts.nk_more); TL_PIN(ts.part); }
#undef TL_PIN
  extern __shared__ __align__(16) unsigned char tl_smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, hf = lane >> 5;
  // tile order over the XCDs: as in gemm_kernel
  const int one = ts.tiles_m * ts.tiles_n, n_tiles = EPI == EPI_PART ? one * ts.splits : one;
  const int q8 = n_tiles >> 3, r8 = n_tiles & 7, strip_tiles = ts.strip * ts.tiles_m;
  int run = 0;                                               // which part of K
  auto decode = [&](int vb_, int64_t& m0_, int& n0_) {
    const int xcd = vb_ & 7;
    int t = xcd * q8 + min(xcd, r8) + (vb_ >> 3);
    if constexpr (EPI == EPI_PART) { run = __builtin_amdgcn_readfirstlane(t / one); t -= run * one; }
    const int sidx = min(t / strip_tiles, (ts.tiles_n - 1) / ts.strip), rem = t - sidx * strip_tiles;
    const int sw = min(ts.strip, ts.tiles_n - sidx * ts.strip);
    const int gidx = rem / (ts.group * sw), r2 = rem - gidx * ts.group * sw, gh = min(ts.group, ts.tiles_m - gidx * ts.group);
    const int gcol = r2 / gh;
    m0_ = (int64_t)(gidx * ts.group + (r2 - gcol * gh)) * BM;
    n0_ = (sidx * ts.strip + gcol) * BN;
  };
  int vb = blockIdx.x;
  int64_t m0;
  int n0;
  decode(vb, m0, n0);

  // LDS-DMA: a wave-load fills eight rows; byte offsets of this lane's chunks (the launcher has checked that they fit 32 bits).
  // Loads 0 .. H0 - 1 of a wave are its share of A0 and B0, the others of A1 and B1
  const int lrow = lane >> 3, lpos = lane & 7;
  auto a_group = [&](int i) __attribute__((always_inline)) {      // eight-row group of the wave's A load i < LA
    const int half = i >= 2 * MA0, idx = half ? wave * 2 * MA1 + i - 2 * MA0 : wave * 2 * MA0 + i, per = 4 * (half ? MA1 : MA0);
    return idx / per * 4 * MI + (half ? 4 * MA0 : 0) + idx % per;
  };
  auto b_group = [&](int i) __attribute__((always_inline)) {
    const int half = i >= 2 * NB0, idx = half ? wave * 2 * NB1 + i - 2 * NB0 : wave * 2 * NB0 + i, per = 4 * (half ? NB1 : NB0);
    return idx / per * 4 * NI + (half ? 4 * NB0 : 0) + idx % per;
  };
  unsigned src_a[LA], src_b[LB];
  auto src_at = [&](int64_t m0_, int n0_, int half) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      if ((i >= 2 * MA0) != half) continue;
      const int rr = a_group(i) * 8 + lrow;
      const int64_t r = min(m0_ + rr, m_rows - 1);      // rows past M repeat the last row: their outputs are never stored
      src_a[i] = (unsigned)(r * a_ld) * 2u + (unsigned)((lpos ^ ((rr >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      if ((i >= 2 * NB0) != half) continue;
      const int rr = b_group(i) * 8 + lrow;
      src_b[i] = (unsigned)((int64_t)tile_col<EPI>(cm, min(n0_ + rr, n_cols - 1)) * ldw) * 2u + (unsigned)((lpos ^ ((rr >> 1) & 7)) * 16);
    }
  };
  // (by buffer loads: a K-tile past the workgroup's last one is requested from a descriptor of no bytes, which costs no traffic,
  // so that the MFMA loops need no branches)
  const int64_t k_first = EPI == EPI_PART ? (int64_t)(run * ts.nk + min(run, ts.nk_more)) * 128 : 0;      // bytes of a row before the run
  const __amdgpu_buffer_rsrc_t a_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>((const char*)g.A + k_first), 0, 0xffffffffu, 0x00020000);
  const __amdgpu_buffer_rsrc_t w_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>((const char*)g.W + k_first), 0, 0xffffffffu, 0x00020000);
  const __amdgpu_buffer_rsrc_t no_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.W), 0, 0, 0x00020000);
  auto dma = [&](int half, int i, const __amdgpu_buffer_rsrc_t& ab, const __amdgpu_buffer_rsrc_t& wb, int k_at, unsigned stage) __attribute__((always_inline)) {
    const int na = 2 * (half ? MA1 : MA0);
    if (i < na) {
      const int q = half * 2 * MA0 + i;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ab, TL_LPTR(tl_smem + stage + a_group(q) * 1024), 16, (int)src_a[q], k_at, 0, 0);
    } else {
      const int q = half * 2 * NB0 + i - na;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(wb, TL_LPTR(tl_smem + stage + A_BYTES + b_group(q) * 1024), 16, (int)src_b[q], k_at, 0, 0);
    }
  };

  // fragments: step j of a K-tile is chunks 2 j + hf; the swizzle of a row depends on l32 alone
  const unsigned lds0 = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)tl_smem;
  const unsigned key = (unsigned)((l32 >> 1) & 7);
  const unsigned a_at = lds0 + (wm * 32 * MI + l32) * 128, b_at = lds0 + A_BYTES + (wn * 32 * NI + l32) * 128;
  tl_u32x4 fa[MI][4], fb[NI][4];
  auto read_a = [&](int mi, int j, unsigned stage_) __attribute__((always_inline)) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fa[mi][j]) : "v"(a_at + stage_ + (((unsigned)(2 * j + hf) ^ key) << 4)), "n"(mi * 4096));
  };
  auto read_b = [&](int ni, int j, unsigned stage_) __attribute__((always_inline)) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fb[ni][j]) : "v"(b_at + stage_ + (((unsigned)(2 * j + hf) ^ key) << 4)), "n"(ni * 4096));
  };

  tl_f32x16 acc[MI][NI];
  // phase P of a K-tile: its MFMAs; between them the fragment reads that belong there (of this K-tile in `st`, of the next in `sn`)
  // and half of the wave-loads of one half of a K-tile, from byte `k_at` of the rows, into `fill`.  FIRST: the first K-tile of a tile
  auto phase = [&](auto P_, auto FIRST, unsigned st, unsigned sn, const __amdgpu_buffer_rsrc_t& ab, const __amdgpu_buffer_rsrc_t& wb, int k_at, unsigned fill) __attribute__((always_inline)) {
    constexpr int P = decltype(P_)::value;
    constexpr bool first = decltype(FIRST)::value;
    constexpr int M0 = P < 2 ? 0 : MA0, MC = P < 2 ? MA0 : MA1, N0 = P & 1 ? NB0 : 0, NC = P & 1 ? NB1 : NB0;
    constexpr int NMF = 4 * MC * NC;                                                     // MFMAs
    constexpr int NR = 4 * (P == 0 ? NB1 : (P == 1 ? MA1 : (P == 2 ? MA0 : NB0)));       // fragment reads
    constexpr int HALF = P < 2, HL = HALF ? H1 : H0, D0 = P & 1 ? HL / 2 : 0, ND = P & 1 ? HL - HL / 2 : HL / 2;
#pragma unroll
    for (int m = 0; m < NMF; ++m) {
      const int j = m / (MC * NC), mi = M0 + m % (MC * NC) / NC, ni = N0 + m % NC;
      const tl_bf16x8 vw = __builtin_bit_cast(tl_bf16x8, fb[ni][j]), va = __builtin_bit_cast(tl_bf16x8, fa[mi][j]);
      if (first && j == 0) {
        const tl_f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vw, va, z, 0, 0, 0);
      } else {
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vw, va, acc[mi][ni], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NR; ++i)
        if (i * NMF / (NR + NR / 4) == m) {
          if constexpr (P == 0) read_b(NB0 + i % NB1, i / NB1, st);
          else if constexpr (P == 1) read_a(MA0 + i % MA1, i / MA1, st);
          else if constexpr (P == 2) read_a(i % MA0, i / MA0, sn);
          else read_b(i % NB0, i / NB0, sn);
        }
#pragma unroll
      for (int i = 0; i < ND; ++i)
        if ((2 * i + 1) * NMF / (2 * ND) == m) dma(HALF, D0 + i, ab, wb, k_at, fill);
      __builtin_amdgcn_sched_barrier(0);
    }
    // what was read is here (waited for before any branch: a register copied at one would be copied too early)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    auto tie_a = [&](int m0_, int n_) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < n_; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(fa[m0_ + i][j]));
    };
    auto tie_b = [&](int n0_, int n_) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < n_; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(fb[n0_ + i][j]));
    };
    if constexpr (P == 0) tie_b(NB0, NB1);
    else if constexpr (P == 1) tie_a(MA0, MA1);
    else if constexpr (P == 2) tie_a(0, MA0);
    else tie_b(0, NB0);
  };
  using P0 = std::integral_constant<int, 0>; using P1 = std::integral_constant<int, 1>;
  using P2 = std::integral_constant<int, 2>; using P3 = std::integral_constant<int, 3>;
  using Yes = std::true_type; using No = std::false_type;

  // ---- epilogue: acc[mi][ni][i] is the output of row m0 + (wm MI + mi) 32 + l32 and logical column
  // n0 + (wn NI + ni) 32 + 8 (i / 4) + 4 hf + i % 4.  A wave's 32 rows x CH blocks of columns go through its own LDS region and
  // leave as 16-byte pieces with a row's pieces in adjacent lanes (as gemm_kernel's short epilogue, in the same arithmetic)
  constexpr int CH = tile_chunk(MI, NI, EPI), PC = tile_pieces(MI, NI, EPI), PITCH = PC * 16 + 16;
  const unsigned wreg = lds0 + NS * STAGE + wave * (32 * PITCH);
  tl_u32x2 braw[NI][4];
  int64_t ro_t[MI];
  auto epi_loads = [&]() __attribute__((always_inline)) {      // bias words and output rows of this tile: requested at its start
    if constexpr (EPI == EPI_PART) return;
    const bool bias_on = bias_p && n_cols >= 4;
    const bf16_t* bp = bias_on ? (const bf16_t*)bias_p : (const bf16_t*)g.W;
    const int pmax = bias_on ? ((n_cols - 4) & ~3) : 0;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int pc = tile_col<EPI>(cm, n0 + (wn * NI + ni) * 32 + 16 * h) + hf * 4;
        braw[ni][2 * h] = *(const tl_u32x2*)(bp + min(pc, pmax));
        braw[ni][2 * h + 1] = *(const tl_u32x2*)(bp + min(pc + 8, pmax));
      }
    int rt[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int64_t r = m0 + (wm * MI + mi) * 32 + l32;
      rt[mi] = 0;
      if (!c_ident) rt[mi] = c_tab[min(r, m_rows - 1)];
    }
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const int64_t r = m0 + (wm * MI + mi) * 32 + l32;
      ro_t[mi] = r >= m_rows ? INT64_MIN : (c_ident ? r * c_ld : (int64_t)rt[mi]);
    }
  };
  // the compiler waits for them where they are first touched: here, where everything older has landed anyway, not in the epilogue,
  // where it would wait for the next tile's K-tiles as well
  auto epi_tie = [&]() __attribute__((always_inline)) {
    if constexpr (EPI == EPI_PART) return;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(braw[ni][q]));
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) asm volatile("" : "+v"(ro_t[mi]));
  };
  const int nk = EPI == EPI_PART ? ts.nk + (run < ts.nk_more) : g.K >> 6;
  unsigned stage = 0;                                        // of the K-tile about to be multiplied
  int64_t m0_n = 0;
  int n0_n = 0;
  bool more = false, on = true;                              // on: the K-tile whose first half was requested last is a real one
  int k_at = 0;                                              // ... and its byte offset in the rows
  auto ktile = [&](int kt, auto FIRST) __attribute__((always_inline)) {
    const unsigned sp = stage == 0 ? (NS - 1) * STAGE : stage - STAGE, sn = stage + STAGE == NS * STAGE ? 0 : stage + STAGE;
    // A1, B1 of this K-tile have landed: younger are A0, B0 of the next one and the whole tiles after it
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(H0 + (NS - 2) * LPT) : "memory");
    __builtin_amdgcn_s_barrier();
    if (kt == nk - NS + 1 && more) src_at(m0_n, n0_n, 1);
    {
      const __amdgpu_buffer_rsrc_t ab = on ? a_buf : no_buf, wb = on ? w_buf : no_buf;
      phase(P0{}, FIRST, stage, sn, ab, wb, k_at, sp);      // A1, B1 of K-tile kt + NS - 1
      phase(P1{}, FIRST, stage, sn, ab, wb, k_at, sp);
    }
    // A0, B0 of the next K-tile have landed, and every wave has all of this one in registers
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(H1 + (NS - 2) * LPT) : "memory");
    __builtin_amdgcn_s_barrier();
    if constexpr (decltype(FIRST)::value) epi_tie();
    k_at += 128;
    if (kt == nk - NS) { if (more) src_at(m0_n, n0_n, 0); k_at = 0; }
    on = kt + NS < nk || more;
    {
      const __amdgpu_buffer_rsrc_t ab = on ? a_buf : no_buf, wb = on ? w_buf : no_buf;
      phase(P2{}, FIRST, stage, sn, ab, wb, k_at, stage);      // A0, B0 of K-tile kt + NS
      phase(P3{}, FIRST, stage, sn, ab, wb, k_at, stage);
    }
    stage = sn;
  };

  auto epilogue = [&]() __attribute__((always_inline)) {
    bf16_t* C = (bf16_t*)c_p;
    const bf16_t* R = (const bf16_t*)res_p;
    const int n_out = EPI == EPI_GLU ? cm.half : n_cols;
    const unsigned rope_m0 = EPI == EPI_ROPE ? (unsigned)(m0 % g.rope_seq) : 0u;
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");      // the last MFMA has written its accumulators
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EPI == EPI_PART) {      // 32 rows x 32 bytes a store, the four stores of a block fill its rows' 128-byte lines
      float* P = ts.part + (int64_t)run * m_rows * n_cols;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        const int64_t r = m0 + (wm * MI + mi) * 32 + l32;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const int col = n0 + (wn * NI + ni) * 32 + g4 * 8 + hf * 4;
            const tl_f32x4 v = {acc_read(acc[mi][ni][4 * g4]), acc_read(acc[mi][ni][4 * g4 + 1]), acc_read(acc[mi][ni][4 * g4 + 2]), acc_read(acc[mi][ni][4 * g4 + 3])};
            if (r < m_rows && col < n_cols) *(tl_f32x4*)(P + r * n_cols + col) = v;
          }
      }
      return;
    }
#pragma unroll
    for (int c0 = 0; c0 < NI; c0 += CH) {
      float bv[CH][16];
#pragma unroll
      for (int nb = 0; nb < CH; ++nb)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const unsigned b0 = bias_p ? braw[c0 + nb][g4].x : 0u, b1 = bias_p ? braw[c0 + nb][g4].y : 0u;
          bv[nb][4 * g4] = __uint_as_float(b0 << 16); bv[nb][4 * g4 + 1] = __uint_as_float(b0 & 0xffff0000u);
          bv[nb][4 * g4 + 2] = __uint_as_float(b1 << 16); bv[nb][4 * g4 + 3] = __uint_as_float(b1 & 0xffff0000u);
        }
      int run0[CH], run1[CH];                                  // columns of the block's two runs of 16
      bool rope[CH];
      float theta[EPI == EPI_ROPE ? CH : 1][8];
#pragma unroll
      for (int nb = 0; nb < CH; ++nb) {
        const int n = n0 + (wn * NI + c0 + nb) * 32;
        run0[nb] = tile_col<EPI>(cm, n);
        run1[nb] = tile_col<EPI>(cm, n + 16);
        rope[nb] = EPI == EPI_ROPE && n < cm.rope_cols;
        if constexpr (EPI == EPI_ROPE) {
          const int e0 = __builtin_amdgcn_readfirstlane(run0[nb]) % cm.rope_dim;      // index of the pair, < rope_dim / 2
          const float k2 = -2.f / (float)cm.rope_dim * log2f(g.rope_base);
          if (rope[nb]) {
#pragma unroll
            for (int i = 0; i < 8; ++i) theta[nb][i] = exp2f((float)(e0 + (i >> 2) * 8 + hf * 4 + (i & 3)) * k2) * 0.15915494309189535f;
          }
        }
      }
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int nb = 0; nb < CH; ++nb) {
          float v[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) v[i] = acc_read(acc[mi][c0 + nb][i]) + bv[nb][i];
          if constexpr (EPI == EPI_GLU) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = g.act == SM_ACT_SWIGLU ? silu_f(v[i]) * v[8 + i] : v[i] * gelu_poly(v[8 + i]);
          } else if constexpr (EPI == EPI_GELU) {
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = gelu_poly(v[i]);
          } else if constexpr (EPI == EPI_ROPE) {
            if (rope[nb]) {
              const float pos = (float)((rope_m0 + (unsigned)((wm * MI + mi) * 32 + l32)) % (unsigned)g.rope_seq);
#pragma unroll
              for (int i = 0; i < 8; ++i) {
                float sn, cs;
                rope_sincos(pos * theta[nb][i], &sn, &cs);
                const float a = v[i], b = v[8 + i];
                v[i] = a * cs - b * sn;
                v[8 + i] = b * cs + a * sn;
              }
            }
          }
#pragma unroll
          for (int g4 = 0; g4 < (EPI == EPI_GLU ? 2 : 4); ++g4) {
            const tl_f32x2 p0 = {v[4 * g4], v[4 * g4 + 1]}, p1 = {v[4 * g4 + 2], v[4 * g4 + 3]};
            const int piece = EPI == EPI_GLU ? 2 * nb + g4 : (EPI == EPI_ROPE ? (g4 >> 1) * 2 * CH + 2 * nb + (g4 & 1) : 4 * nb + g4);
            lds_write8(wreg + l32 * PITCH + hf * 8, piece * 16,
                       tl_u32x2{__builtin_bit_cast(unsigned, __builtin_convertvector(p0, tl_bf16x2)), __builtin_bit_cast(unsigned, __builtin_convertvector(p1, tl_bf16x2))});
          }
        }
        lds_write8(wreg + l32 * PITCH, PC * 16, __builtin_bit_cast(tl_u32x2, ro_t[mi]));
        // (wave-private data: the LDS queue keeps a wave's accesses in order)
        constexpr int NIT = PC / 2;
        tl_u32x4 d[NIT], rr[NIT];
        tl_u32x2 ro2v[NIT];
        int64_t off[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int idx = it * 64 + lane, rl = idx / PC, p = idx - rl * PC;
          asm volatile("ds_read_b128 %0, %1" : "=v"(d[it]) : "v"(wreg + rl * PITCH + p * 16));
          asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(ro2v[it]) : "v"(wreg + rl * PITCH), "n"(PC * 16));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int it = 0; it < NIT; ++it) { asm volatile("" : "+v"(d[it])); asm volatile("" : "+v"(ro2v[it])); }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int idx = it * 64 + lane, rl = idx / PC, p = idx - rl * PC;
          const int64_t ro2 = __builtin_bit_cast(int64_t, ro2v[it]);
          int col;
          if constexpr (EPI == EPI_GLU) col = ((n0 >> 5) + wn * NI + c0) * 16 + p * 8;
          else if constexpr (EPI == EPI_ROPE) {
            const bool second = p >= 2 * CH;
            const int nb = (second ? p - 2 * CH : p) >> 1;
            col = second ? run1[0] : run0[0];
#pragma unroll
            for (int b = 1; b < CH; ++b) col = nb == b ? (second ? run1[b] : run0[b]) : col;
            col += (p & 1) * 8;
          } else col = n0 + (wn * NI + c0) * 32 + p * 8;
          off[it] = (ro2 == INT64_MIN || col >= n_out) ? INT64_MIN : ro2 + col;
        }
        if (R) {
#pragma unroll
          for (int it = 0; it < NIT; ++it) rr[it] = *(const tl_u32x4*)(R + (off[it] == INT64_MIN ? 0 : off[it]));      // element 0: a valid address, not used
#pragma unroll
          for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const tl_f32x2 pr = {__uint_as_float(d[it][e] << 16) + __uint_as_float(rr[it][e] << 16), __uint_as_float(d[it][e] & 0xffff0000u) + __uint_as_float(rr[it][e] & 0xffff0000u)};
              d[it][e] = __builtin_bit_cast(unsigned, __builtin_convertvector(pr, tl_bf16x2));
            }
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it)
          if (off[it] != INT64_MIN) *(tl_u32x4*)(C + off[it]) = d[it];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // ---- start: the first NS K-tiles but for the last one's second half, the first phase's fragments  (nk >= NS)
  src_at(m0, n0, 0);
  src_at(m0, n0, 1);
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    k_at = t * 128;
#pragma unroll
    for (int i = 0; i < H0; ++i) dma(0, i, a_buf, w_buf, k_at, t * STAGE);
    if (t + 1 < NS) {
#pragma unroll
      for (int i = 0; i < H1; ++i) dma(1, i, a_buf, w_buf, k_at, t * STAGE);
    }
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(H1 + H0 + (NS - 2) * LPT) : "memory");
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int i = 0; i < MA0; ++i) read_a(i, j, 0u);
#pragma unroll
    for (int i = 0; i < NB0; ++i) read_b(i, j, 0u);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int i = 0; i < MA0; ++i) asm volatile("" : "+v"(fa[i][j]));
#pragma unroll
    for (int i = 0; i < NB0; ++i) asm volatile("" : "+v"(fb[i][j]));
  }
  for (;;) {
    const int vb_n = vb + (int)gridDim.x;
    more = EPI != EPI_PART && vb_n < n_tiles;
    if (more) decode(vb_n, m0_n, n0_n);
    epi_loads();
    ktile(0, Yes{});
    for (int kt = 1; kt < nk; ++kt) ktile(kt, No{});
    epilogue();
    if (!more) break;
    vb = vb_n; m0 = m0_n; n0 = n0_n;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing is on its way to LDS when the workgroup gives it back
}

template <int MI, int NI, int EPI>
int tile_launch2(const GemmArgs& g, const TileCols& cm, hipStream_t s, int splits = 1, float* part = nullptr) {
  constexpr size_t smem = tile_lds(MI, NI, EPI);
  static_assert(smem <= 160 * 1024, "LDS of a compute unit");
  static const hipError_t attr = hipFuncSetAttribute((const void*)tile_kernel<MI, NI, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return (int)attr;
  const int tiles_n = (g.N + 64 * NI - 1) / (64 * NI);
  const int64_t tiles_m = (g.M + 64 * MI - 1) / (64 * MI);
  if (tiles_m * tiles_n > INT32_MAX) return (int)hipErrorInvalidValue;
  const int xn = xcd_strips(g.M, g.N, tiles_n);
  const int nk = g.K >> 6;
  const TileGrid ts{(int)tiles_m, tiles_n, (tiles_n + xn - 1) / xn, g.K >= 1024 ? (int)std::min<int64_t>(4, tiles_m) : 1, splits, nk / splits, nk % splits, part};
  const int64_t grid = EPI == EPI_PART ? tiles_m * tiles_n * splits : std::min<int64_t>(tiles_m * tiles_n, 256);      // one workgroup per CU (a multiple of 8 where it walks through several tiles)
  tile_kernel<MI, NI, EPI><<<dim3((unsigned)grid), dim3(256), smem, s>>>(g, cm, ts);
  return (int)hipGetLastError();
}
template <int MI, int NI>
int tile_launch(const GemmArgs& g, const TileCols& cm, hipStream_t s) {
  if (g.act == SM_ACT_SWIGLU || g.act == SM_ACT_GEGLU) return tile_launch2<MI, NI, EPI_GLU>(g, cm, s);
  if (g.rope_cols > 0) return tile_launch2<MI, NI, EPI_ROPE>(g, cm, s);
  return g.act == SM_ACT_GELU ? tile_launch2<MI, NI, EPI_GELU>(g, cm, s) : tile_launch2<MI, NI, EPI_PLAIN>(g, cm, s);
}
bool tile_rows_ok(const RowProg& r) {      // a pitch or a table of whole 16-byte vectors
  if (r.identity) return r.ld % 8 == 0;
  if (!r.table || r.c0 % 8) return false;
  for (int t = 0; t < r.nterm; ++t)
    if (r.t_coef[t] % 8) return false;
  return true;
}
}  // namespace

// Which Linears run here, and in which tile: us of each tile, fitted to measured times (K = 640 .. 11008, five epilogues; 2 to 5 %
// standard deviation, 7 % with K >= 4096 and weights from memory), against gemm_kernel's own.  A round of workgroups (one per CU)
// costs a fixed part, a part per K-tile and a part per K-tile that grows with the share of the CUs that work in it (the clock
// falls as more of the chip multiplies); below K = 2048 the residual's bytes at 5 TB/s, which nothing hides (without one
// the costs up to K = 1024 are 4 % high, so that even ones go to the large tile).
// Measured us, gemm_kernel / this: 2048 x 22016 x 4096 SwiGLU 370 / 305 (256 x 256), 2048 x 12288 x 4096 + RoPE 198 / 175 (256 x 192),
// 333 x 22016 x 4096 SwiGLU 114 / 77 (192 x 192), 333 x 12288 x 4096 + RoPE 61 / 54 (128 x 192), 6304 x 768 x 3072 41.5 / 38 (128 x 192),
// 6304 x 2304 x 768 34 / 27 (256 x 256).  Over 823 shapes of 16 to 16384 rows that the column-split kernel leaves, each tile and
// gemm_kernel timed in turn, the choice takes .929 of gemm_kernel's time in the geometric mean (the best variant of each .923), three
// lose more than 2 %, 4.7 % at most.  The lines:
//  - at least 160 tiles: what a tile leaves idle the costs do not tell (16 tiles, 33 x 3072 x 1024 + RoPE 13.4 / 17.8; 110 tiles,
//    600 x 4096 x 11008 99 / 127; every shape of 172 tiles and more that the costs choose is a gain or even);
//  - between K = 1024 and 2048 only where the costs are 5 % apart (4702 x 5184 x 1088 + GELU 68 / 72 at .99 of it);
//  - from K = 8192 on with a residual only where they are 10 % apart: with weights from memory 128 x 256 tiles take 143 to 168 us from
//    one allocation to the next (1550 to 2048 x 4096 x 11008; gemm_kernel 149 to 163);
//  - not below K = 640: a tile's fixed part weighs as much as its K loop and gemm_kernel's two workgroups per CU hide it better
//    (8192 x 2560 x 320 GEGLU 29 / 32, 12544 x 2048 x 512 + GELU 44 / 46).
static bool tile_linear_ok(const GemmArgs& g) {
  if (g.dtype != SM_BF16 || g.K % 64 || g.K < 640 || g.a_gran > 0 || g.norm || g.C2 || g.c_transposed || g.c_cols_on) return false;
  const bool gated = g.act == SM_ACT_SWIGLU || g.act == SM_ACT_GEGLU;
  if (g.N % 8 || (gated && g.N % 64) || (g.act != SM_ACT_NONE && g.rope_cols)) return false;
  return g.a_rows.identity && g.a_rows.ld % 8 == 0 && g.M * g.a_rows.ld <= INT32_MAX && tile_rows_ok(g.c_rows) && (int64_t)g.N * g.ldw <= INT32_MAX;
}
static const struct TileForm { int mi, ni; double fixed, round, step, busy, act; } tile_form[] = {{4, 4, 1.98, 10.22, 0.855, 0.624, 4.80},
                                                                                 {4, 3, 2.86, 8.09, 0.669, 0.467, 2.86},
                                                                                 {3, 4, 3.23, 7.74, 0.678, 0.433, 3.48},
                                                                                 {3, 3, 3.07, 6.68, 0.656, 0.262, 2.18},
                                                                                 {2, 4, 2.89, 6.39, 0.510, 0.280, 1.84},
                                                                                 {3, 2, 3.75, 4.40, 0.429, 0.243, 1.49},
                                                                                 {2, 3, 3.70, 4.38, 0.439, 0.225, 1.69}};
static double tile_cost(const TileForm& f, const GemmArgs& g, int splits) {
  const int64_t tiles = ((g.M + 64 * f.mi - 1) / (64 * f.mi)) * ((g.N + 64 * f.ni - 1) / (64 * f.ni)) * splits;
  const double nk = (double)((g.K / 64 + splits - 1) / splits), rounds = (double)((tiles + 255) / 256);
  const double act = g.act == SM_ACT_GELU ? 1. : (g.act == SM_ACT_SWIGLU || g.act == SM_ACT_GEGLU ? .7 : 0.);
  double us = f.fixed + rounds * (f.round + nk * f.step + act * f.act) + (double)tiles / 256. * nk * f.busy;
  if (g.residual && g.K < 2048) us += .4e-6 * (double)g.M * (act == .7 ? g.N / 2 : g.N);
  if (g.rope_cols && g.K <= 1024) us += 3.5;
  return us;
}
static bool tile_linear_plan(const GemmArgs& g, int* mi, int* ni) {
  if (!tile_linear_ok(g)) return false;
  double least = (g.K <= 1024 ? 1.02 : (g.K < 2048 ? .95 : (g.K >= 8192 && g.residual ? .9 : 1.))) * gemm_kernel_cost(g);
  *mi = 0;
  for (const auto& f : tile_form) {
    if (((g.M + 64 * f.mi - 1) / (64 * f.mi)) * ((g.N + 64 * f.ni - 1) / (64 * f.ni)) < 160) continue;
    const double us = tile_cost(f, g, 1);
    if (us < least) { least = us; *mi = f.mi; *ni = f.ni; }
  }
  return *mi != 0;
}

// Which tile and how many runs of K, by the same costs: the sum kernel takes 0.7 us and the parts' bytes at 9 TB/s (1459 measured
// points with K >= 4096, 70 to 2048 rows; 10 % standard deviation).  Below K = 4096 the parts cost more than the idle CUs they fill
// (500 x 2048 x 2048 10.6 / 20 us, 700 x 1024 x 2816 13 / 20).  `unsplit`: what the Linear (and the norm behind it) takes otherwise.
bool tile_parts_plan(const GemmArgs& g, double unsplit, SplitKPlan* p) {
  p->splits = 0;
  if (g.K < 4096 || g.N > 4096 || g.act != SM_ACT_NONE || g.rope_cols || !tile_linear_ok(g)) return false;
  if (!g.c_rows.identity || g.c_rows.ld != g.N || g.ldw != g.K || g.a_rows.ld != g.K) return false;
  for (const auto& f : tile_form) unsplit = std::min(unsplit, tile_cost(f, g, 1));
  double least = .97 * unsplit;
  for (const auto& f : tile_form)
    for (int s = 2; s <= 8; ++s) {
      const double us = 1.08 * tile_cost(f, g, s) + .7 + 8e-6 * s * (double)g.M * g.N / 9.;
      if (us < least && g.K / 64 / s >= tile_stages(f.mi, f.ni)) { least = us; *p = SplitKPlan{f.mi, f.ni, s}; }
    }
  return p->splits != 0;
}

// (not where the caller or the tuner has picked one of gemm_kernel's tiles)
bool tile_linear_use(const GemmArgs& g, int* mi, int* ni) { return !gemm_tile_chosen(g) && tile_linear_plan(g, mi, ni); }
int launch_tile_linear(const GemmArgs& g, int mi, int ni, void* stream) {
  const TileCols cm{g.N / 2, g.rope_cols, g.rope_dim};
  hipStream_t s = (hipStream_t)stream;
#define TL_CASE(MI_, NI_) if (mi == MI_ && ni == NI_) return tile_launch<MI_, NI_>(g, cm, s);
  TL_CASE(4, 4) TL_CASE(4, 3) TL_CASE(3, 4) TL_CASE(3, 3) TL_CASE(2, 4) TL_CASE(3, 2) TL_CASE(2, 3)
#undef TL_CASE
  return (int)hipErrorInvalidValue;
}

// the parts of a Linear cut over K (k_splitk.hip)
int launch_tile_parts(const GemmArgs& g, int mi, int ni, int splits, float* part, void* stream) {
  const TileCols cm{0, 0, 0};
  if (splits < 1 || (g.K >> 6) / splits < tile_stages(mi, ni)) return (int)hipErrorInvalidValue;
#define TL_CASE(MI_, NI_) if (mi == MI_ && ni == NI_) return tile_launch2<MI_, NI_, EPI_PART>(g, cm, (hipStream_t)stream, splits, part);
  TL_CASE(4, 4) TL_CASE(4, 3) TL_CASE(3, 4) TL_CASE(3, 3) TL_CASE(2, 4) TL_CASE(3, 2) TL_CASE(2, 3)
#undef TL_CASE
  return (int)hipErrorInvalidValue;
}

}  // namespace sm
