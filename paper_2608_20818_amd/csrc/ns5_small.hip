// NS5 products of small weight sets on gfx950: 64 x 64 and 128 x 128 tiles.
//
// The 256 x 256 tiles of ns5.hip need a few hundred tiles per launch to fill
// the chip.  A set of a few matrices has far fewer, and each tile then runs its
// whole K alone on one CU at one wave per SIMD.  This kernel computes the same
// products (Gram, B = bA + cA^2, split product, apply; see ns5.hip for the
// algebra and the workspace layout) on smaller tiles, so that the same work
// spreads over 4 to 16 times as many work groups, and pads the matrices to 64
// or 128 instead of 256.
//
// One launch runs up to two products with a work list each (kind and operands
// are run-time values): products of the factored and the plain group of a chunk,
// which do not depend on each other, or two independent ones of a sequence.
//
// Eight waves, two per SIMD: two groups of 2 x 2 waves, each wave T/2 x T/2 of
// the tile as 32 x 32 MFMA blocks, the groups splitting the k-steps of a stage
// and adding up in LDS at the end (with one wave per SIMD its reads, loads and
// products do not overlap); K in stages of 64 through a ring of NST LDS buffers filled by direct
// global-to-LDS loads, NST - 1 stages ahead: with few work groups in flight the
// load latency, not the MFMA rate, is what a stage costs.  The diagonal terms
// of the split matrices, fp32, are applied in the epilogue from the operands'
// tiles at the output position, which are loaded before the main loop.
#include <type_traits>

#include "prm_device.h"

namespace prm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace small {
constexpr int BK = 64;
// Eight waves: two groups of 2 x 2, each group taking two of a stage's four
// k-steps for the whole tile.
constexpr int KG = 2, KSG = 4 / KG, NWAVES = 4 * KG, NTHREADS = 64 * NWAVES;
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16* lds_v4i16;

template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
}  // namespace small

// T: tile edge (64 or 128); NST: LDS stage buffers.
template <int T, int NST>
__global__ __launch_bounds__(small::NTHREADS) void ns_small_kernel(const MatDesc* __restrict__ md,
                                                                   const Item* __restrict__ items0, int32_t n0,
                                                                   const Item* __restrict__ items1, uint32_t op0,
                                                                   uint32_t op1, NsStepParams sp) {
  using namespace small;
  constexpr int WT = T / 2, MI = WT / 32;
  constexpr int OP_BYTES = T * BK * 2;           // one operand of a stage
  constexpr int STAGE_BYTES = 2 * OP_BYTES;
  constexpr int LPO = T / 8 / NWAVES;            // 1 KB wave loads per operand, wave and stage
  constexpr int LPS = 2 * LPO;
  constexpr int TCH = T / 8;                     // 16-byte chunks in a row of T bf16
  static_assert(4 * T * T <= NST * STAGE_BYTES, "the fp32 output tile fits the stage buffers");
  __shared__ __attribute__((aligned(16))) char lds[NST * STAGE_BYTES];

  // the two work lists of the launch: blocks [0, n0) and the rest
  const bool second = (int)blockIdx.x >= n0;
  const Item it = second ? items1[blockIdx.x - n0] : items0[blockIdx.x];
  if (it.mat < 0) return;  // filler of the XCD-interleaved order (whole work group)
  const uint32_t opw = second ? op1 : op0;  // ns_pack
  struct { int kind, src, use_alpha, last, sx, sy, so; float xshift, yshift; } op;
  op.kind = opw & 3;
  op.src = (opw >> 2) & 1;
  op.use_alpha = (opw >> 3) & 1;
  op.last = (opw >> 4) & 1;
  op.sx = (opw >> 5) & 7;
  op.sy = (opw >> 8) & 7;
  op.so = (opw >> 11) & 7;
  op.xshift = (opw >> 14) & 1 ? sp.a : 0.f;
  op.yshift = (opw >> 15) & 1 ? sp.a : 0.f;
  const bool hilo = (opw >> 16) & 1;
  const MatDesc& d = md[it.mat];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
  const int kind = op.kind;
  const bool tn = kind == GEMM_GRAM;
  const int64_t ld = d.rp;  // every operand has rp columns
  const uint16_t* XTc = op.src == 0 ? d.XT : d.XTn;
  const uint16_t* XTcl = op.src == 0 ? d.XTl : d.XTnl;  // precise mode: low parts
  const int64_t row0 = (int64_t)it.tm * T, col0 = (int64_t)it.tn * T;

  // Operands of K segment 0; in precise mode the apply sums hi Q + lo Q over two
  // segments.  The Gram's hi hi^T + hi lo^T + lo hi^T (`tri`) come from one pass: a
  // stage holds 32 k-rows of four panels, hi and lo of the tile's rows, then of its
  // columns (each loaded once for the products it is in, where three segments
  // would load six).
  const uint16_t *P, *Q;
  int nk, nseg = 1;
  const bool tri = tn && hilo;
  if (kind == GEMM_GRAM) {
    P = XTc; Q = XTc;
    nk = (int)(d.cp / (tri ? BK / 2 : BK));
  } else {
    P = kind == GEMM_APPLY ? XTc : d.S[op.sx];
    Q = d.S[op.sy];
    nk = (int)(d.rp / BK);
    if (hilo && kind == GEMM_APPLY) nseg = 2;
  }
  const int NK = nseg * nk;

  // DMA addressing: a wave-uniform base per load plus a per-lane byte offset.
  // NT: load q of an operand covers tile rows 8 q + lane / 8, physical chunk
  // lane % 8 holding logical chunk (lane % 8) ^ (row / 2 % 8), which only
  // depends on the parity of q.  TN: load q covers k-rows (512 / T) q +
  // lane / TCH, physical chunk lane % TCH holding logical chunk XOR 4 (row % 4)
  // (T = 128) or 4 (row / 2 % 2) (T = 64): the four k-rows of a transposing read
  // then fall into distinct 64-byte bank quarters.
  const uint32_t ldb = (uint32_t)ld * 2;  // bytes of a workspace row
  uint32_t voff[2];
  if (tn) {
    const int sw = T == 128 ? 4 * ((lane >> 4) & 3) : 4 * ((lane >> 4) & 1);
    voff[0] = voff[1] = (uint32_t)(lane / TCH) * ldb + (((lane % TCH) ^ sw) << 4);
  } else {
    voff[0] = (uint32_t)(lane >> 3) * ldb + (((lane & 7) ^ (lane >> 4) ^ (4 * (wave * LPO & 1))) << 4);
    voff[1] = voff[0] ^ 64;  // ldb is a multiple of 128
  }
  const uint64_t lrows = (uint64_t)(tn ? 512 / T : 8) * ldb;              // of one load
  const uint64_t kstep = tn ? (uint64_t)(tri ? BK / 2 : BK) * ldb : (uint64_t)BK * 2;  // between stages
  const uint64_t offA = (tn ? (uint64_t)row0 * 2 : (uint64_t)row0 * ldb) + (uint64_t)(wave * LPO) * lrows;
  const uint64_t offB = (tn ? (uint64_t)col0 * 2 : (uint64_t)col0 * ldb) + (uint64_t)(wave * LPO) * lrows;
  constexpr int PANEL = OP_BYTES / 2;  // of the four of a `tri` stage; two waves load each
  auto uniform64 = [](uint64_t u) __attribute__((always_inline)) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
  };
  // Where the wave's loads of the next stage to be issued start: operand
  // addresses and LDS destination; moves on with every stage.
  uint64_t srcA = uniform64((uint64_t)(uintptr_t)P + offA), srcB = uniform64((uint64_t)(uintptr_t)Q + offB);
  uint64_t qstep = lrows;                                     // between loads q and q + 2
  uint32_t lds0 = wave * LPO * 1024, dstB = OP_BYTES, dstq = 1024;  // of load 0, of odd loads, between q and q + 2
  if (tri) {
    const int panel = wave >> 1, first = (wave & 1) * LPS;
    const uint16_t* src = (panel & 1 ? XTcl : XTc) + (panel & 2 ? col0 : row0);
    srcA = uniform64((uint64_t)(uintptr_t)src + first * lrows);
    srcB = srcA + lrows;
    qstep = 2 * lrows;
    lds0 = panel * PANEL + first * 1024;
    dstB = 1024;
    dstq = 2048;
  }
  lds0 += (uint32_t)(uintptr_t)(lds_ptr)lds;
  int istage = 0, ibuf = 0;
  // One of the wave's LPS loads of that stage (even q: first operand).
  // Assembly, so that the compiler does not wait for the loads at every LDS
  // read; it sees neither the LDS writes nor their wait, which are explicit
  // below.  The s_nop is the wait state an M0 write needs before a load into
  // LDS reads it.  M0 is a register the compiler reserves and does not save
  // around the asm; nothing else in this kernel reads it
  // (tests/test_gpu_small_tiles.py checks the assembly).
  auto issue1 = [&](int q) __attribute__((always_inline)) {
    const int qq = q >> 1;
    const uint64_t src = ((q & 1) ? srcB : srcA) + qq * qstep;
    const uint32_t dst = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + (uint32_t)ibuf * STAGE_BYTES)) +
                         ((q & 1) ? dstB : 0) + qq * dstq;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // the M0 clobber, see above
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff[qq & 1]), "s"(src), "s"(dst) : "m0");
#pragma clang diagnostic pop
  };
  auto issued = [&]() __attribute__((always_inline)) {
    ++istage;
    ibuf = ibuf + 1 == NST ? 0 : ibuf + 1;
    srcA += kstep;
    srcB += kstep;
    if (nseg > 1 && istage == nk) {  // the next K segment
      srcA = uniform64((uint64_t)(uintptr_t)XTcl + offA);
      srcB = uniform64((uint64_t)(uintptr_t)Q + offB);
    }
  };

  const int hl = lane >> 5, m = lane & 31;
  const bool two = kind == GEMM_SPROD || nseg == 2;
  // Output mapping of the epilogue: chunk k of this thread is the 8 columns
  // col0 + wch .. of row row0 + k RPI + wrow.  Its operands there: the first
  // operand's tile for the square, the split product and the apply (there X^T,
  // hi and lo), the second operand's for the split product, and the diagonals
  // of both.  All of them are loaded before anything is stored (a load behind a
  // store waits for the store), under the main loop where registers allow.
  constexpr int RPI = NTHREADS / TCH, ROW_ITS = T / RPI;
  const int wrow = tid / TCH, wch = (tid % TCH) * 8;
  u32x4 x0[ROW_ITS], x1[ROW_ITS];
  float drow[ROW_ITS], dcol[8];
  const uint32_t eoff = (uint32_t)wrow * ldb + (uint32_t)wch * 2;
  const uint64_t tile0 = (uint64_t)row0 * ldb + (uint64_t)col0 * 2, rstep = (uint64_t)RPI * ldb;
  auto at = [&](const uint16_t* base, int k) __attribute__((always_inline)) {
    return (PRM_GLOBAL u32x4*)((PRM_GLOBAL char*)((uint64_t)(uintptr_t)base + tile0 + k * rstep) + eoff);
  };
  auto load_operands = [&]() __attribute__((always_inline)) {
    if (kind == GEMM_GRAM) return;
    const uint16_t* e1 = kind == GEMM_SPROD ? Q : XTcl;
    const float* dX = d.dS[op.sx] + row0;
#pragma unroll
    for (int k = 0; k < ROW_ITS; ++k) {
      x0[k] = *at(P, k);
      if (two) x1[k] = *at(e1, k);
      if (kind != GEMM_APPLY) drow[k] = gptr(dX)[k * RPI + wrow];
    }
    Vec<float>::load8(d.dS[op.sy] + col0 + wch, dcol);
  };
  if constexpr (T == 64) load_operands();
  const float alpha = op.use_alpha ? *d.alpha : 1.0f;
  float* const dout = d.dS[op.so];
  uint16_t* const out = kind == GEMM_APPLY ? (op.src == 0 ? d.XTn : d.XT) : d.S[op.so];
  uint16_t* const outl = op.src == 0 ? d.XTnl : d.XTl;

  floatx16 acc[MI][MI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < NK) {
#pragma unroll
      for (int q = 0; q < LPS; ++q) issue1(q);
      issued();
    }

  // Stage loop.  Before stage s is read, the loads of at most the NST - 2 later
  // stages may be in flight; stage s + NST - 1 is issued after the barrier that
  // every wave reaches once it has read stage s - 1 (whose buffer it takes).
  // While the previous stage's products run from one register set, the stage's
  // fragments are read into the other and the loads are issued, spread between
  // the products: the two waves of a SIMD have little else to hide them behind.
  // NP = 3 (`tri`): the two fragment sets are hi and lo of one k-step, and the
  // products hi hi, hi lo and lo hi; otherwise they are the group's two k-steps.
  auto main_loop = [&](auto rd_a, auto rd_b, auto npc) __attribute__((always_inline)) {
    constexpr int NP = decltype(npc)::value;
    static_assert(KSG == 2, "two fragment sets");
    bf16x8 fa[2][KSG][MI], fb[2][KSG][MI];
    int buf = 0;
    // stage s into set `setc`; PREV: with the previous stage's products; MORE:
    // stage s + NST - 1 exists (-1: decided at run time), static in the main
    // loop so that it has no branches
    auto stage = [&](int s, auto setc, auto prevc, auto morec) __attribute__((always_inline)) {
      constexpr int set = decltype(setc)::value;
      constexpr bool PREV = decltype(prevc)::value;
      constexpr int MORE = decltype(morec)::value;
      const bool more = MORE == 1 || s + NST - 1 < NK;
      if (MORE == 1 || s + NST - 2 < NK) wait_loads<(NST - 2) * LPS>();
      else wait_loads<0>();
      __syncthreads();
      const char* a = lds + buf * STAGE_BYTES;
      const char* b = a + OP_BYTES;
      constexpr int G = NP * MI * MI, F = 2 * KSG * MI;  // products; F fragment reads and LPS loads are spread over them
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (more) {
#pragma unroll
          for (int q = LPS * g / G; q < LPS * (g + 1) / G; ++q) issue1(q);
        }
#pragma unroll
        for (int f = F * g / G; f < F * (g + 1) / G; ++f) {
          const int ks = f / (2 * MI), i = (f / 2) % MI;
          if (f & 1) fb[set][ks][i] = rd_b(b, i, ks);
          else fa[set][ks][i] = rd_a(a, i, ks);
        }
        // operands swapped: accumulates the transposed block (P Q^T)^T = Q P^T
        if constexpr (PREV) {
          const int ks = g / (MI * MI), i = (g / MI) % MI, j = g % MI;
          const int ka = NP == 3 ? ks >> 1 : ks, kb = NP == 3 ? ks & 1 : ks;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set ^ 1][kb][j], fa[set ^ 1][ka][i], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) issued();
      buf = buf + 1 == NST ? 0 : buf + 1;
    };
    auto products = [&](auto setc) __attribute__((always_inline)) {
      constexpr int set = decltype(setc)::value;
#pragma unroll
      for (int ks = 0; ks < NP; ++ks)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < MI; ++j) {
            const int ka = NP == 3 ? ks >> 1 : ks, kb = NP == 3 ? ks & 1 : ks;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][kb][j], fa[set][ka][i], acc[i][j], 0, 0, 0);
          }
    };
    constexpr std::integral_constant<int, 0> set0{};
    constexpr std::integral_constant<int, 1> set1{};
    constexpr std::integral_constant<int, 1> yes{};
    constexpr std::integral_constant<int, -1> rt{};
    stage(0, set0, std::false_type{}, rt);
    int s = 1;
    for (; s + NST < NK; s += 2) {
      stage(s, set1, std::true_type{}, yes);
      stage(s + 1, set0, std::true_type{}, yes);
    }
    for (; s + 1 < NK; s += 2) {
      stage(s, set1, std::true_type{}, rt);
      stage(s + 1, set0, std::true_type{}, rt);
    }
    if (s < NK) {
      stage(s, set1, std::true_type{}, rt);
      products(set1);
    } else {
      products(set0);
    }
  };
  if (tn) {
    // lane L of 16-lane group g = L / 16 reads k-row 8 (g / 2) + 4 kk + (L % 16) / 4
    // of k-step 0 at columns 16 (g % 2) + 4 (L % 4) of its block
    const int g = lane >> 4, jl = lane & 15;
    const int sw = T == 128 ? 4 * (jl >> 2) : 4 * ((jl >> 3) & 1);
    int oa[MI][2], ob[MI][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int kr = 16 * (tri ? 1 : KSG) * kg + 8 * (g >> 1) + 4 * kk + (jl >> 2);
        const int ca = wm * WT + i * 32 + 16 * (g & 1) + 4 * (jl & 3), cb = wn * WT + i * 32 + 16 * (g & 1) + 4 * (jl & 3);
        oa[i][kk] = kr * (2 * T) + (((ca >> 3) ^ sw) << 4) + ((ca & 7) << 1);
        ob[i][kk] = kr * (2 * T) + (((cb >> 3) ^ sw) << 4) + ((cb & 7) << 1);
      }
    // `set` apart: the next k-step, or the low part's panel
    auto rd = [&](const char* base, const int (&off)[2], int set) __attribute__((always_inline)) {
      const v4i16 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(base + off[0] + set));
      const v4i16 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(base + off[1] + set));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    if (tri)
      main_loop([&](const char* base, int i, int ks) __attribute__((always_inline)) { return rd(base, oa[i], ks * PANEL); },
                [&](const char* base, int i, int ks) __attribute__((always_inline)) { return rd(base, ob[i], ks * PANEL); },
                std::integral_constant<int, 3>{});
    else
      main_loop(
          [&](const char* base, int i, int ks) __attribute__((always_inline)) { return rd(base, oa[i], ks * 32 * T); },
          [&](const char* base, int i, int ks) __attribute__((always_inline)) { return rd(base, ob[i], ks * 32 * T); },
          std::integral_constant<int, KSG>{});
  } else {
    const int arow = wm * WT + m, brow = wn * WT + m;
    int oa[KSG], ob[KSG];
#pragma unroll
    for (int ks = 0; ks < KSG; ++ks) {
      const int ch = (KSG * kg + ks) * 2 + hl;
      oa[ks] = arow * 128 + ((ch ^ ((arow >> 1) & 7)) << 4);
      ob[ks] = brow * 128 + ((ch ^ ((brow >> 1) & 7)) << 4);
    }
    main_loop([&](const char* base, int i, int ks) __attribute__((always_inline)) {
                return *reinterpret_cast<const bf16x8*>(base + oa[ks] + i * 32 * 128); },
              [&](const char* base, int i, int ks) __attribute__((always_inline)) {
                return *reinterpret_cast<const bf16x8*>(base + ob[ks] + i * 32 * 128); },
              std::integral_constant<int, KSG>{});
  }

  // ---- epilogue ----
  // The fp32 accumulators pass through LDS (row r: 4 T bytes, 16-byte chunk c at
  // c ^ (r % (T / 4))) so that every thread then handles 8 consecutive columns
  // of a row with 16-byte accesses.  The finished chunk goes to the output row
  // and, as bf16, in place of the first of its two fp32 chunks, from where the
  // mirror and the parameter write read it.
  auto fb4 = [&](int row, int c4) __attribute__((always_inline)) {
    return lds + row * (4 * T) + ((c4 ^ (row & (T / 4 - 1))) << 4);
  };
  auto tb = [&](int row, int col) __attribute__((always_inline)) { return fb4(row, (col >> 3) * 2) + (col & 7) * 2; };
  const bool diag = kind != GEMM_APPLY && it.tm == it.tn;
  const bool last = kind == GEMM_APPLY && op.last;
  if constexpr (T != 64) load_operands();
  __syncthreads();  // every wave is done with the stage buffers
  // the k-step groups add up in turn (fixed order)
#pragma unroll
  for (int gsel = 0; gsel < KG; ++gsel) {
    if (kg == gsel) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // lane L: row 32 i + L % 32 of its wave block, columns 32 j + 8 q + 4 (L / 32) + 0..3
            f32x4_t v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            f32x4_t* const f =
                reinterpret_cast<f32x4_t*>(fb4(wm * WT + 32 * i + m, (wn * WT + 32 * j + 8 * q + 4 * hl) >> 2));
            if (gsel) {
              const f32x4_t o = *f;
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] += o[e];
            }
            *f = v;
          }
    }
    __syncthreads();
  }
  if (diag) {
    // the diagonal goes to dS in fp32 (the bf16 tile keeps 0 there)
    if (tid < T) {
      const float a = *reinterpret_cast<const float*>(fb4(tid, tid >> 2) + (tid & 3) * 4);
      float dv = alpha * alpha * a;
      if (kind != GEMM_GRAM) {
        const float x = d.dS[op.sx][row0 + tid] + op.xshift;
        dv = kind == GEMM_POLY ? sp.b * x + sp.c * (a + x * x) : a + x * (d.dS[op.sy][row0 + tid] + op.yshift);
      }
      dout[row0 + tid] = dv;
    }
    __syncthreads();
  }
  auto rows = [&](auto kindc) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kindc)::value;
    if constexpr (KIND == GEMM_POLY) {
#pragma unroll
      for (int e = 0; e < 8; ++e) dcol[e] = sp.b + sp.c * (dcol[e] + op.yshift);
    } else if constexpr (KIND != GEMM_GRAM) {
#pragma unroll
      for (int e = 0; e < 8; ++e) dcol[e] += op.yshift;
    }
#pragma unroll
    for (int k = 0; k < ROW_ITS; ++k) {
      const int row = k * RPI + wrow;
      char* const own = tb(row, wch);
      const f32x4_t a0 = *reinterpret_cast<const f32x4_t*>(own);
      const f32x4_t a1 = *reinterpret_cast<const f32x4_t*>(fb4(row, (wch >> 2) + 1));
      float v[8] = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
      float x[8], y[8];
      if constexpr (KIND != GEMM_GRAM) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = bf2f((x0[k][e >> 1] >> (16 * (e & 1))) & 0xffffu);
      }
      if (KIND == GEMM_SPROD || (KIND == GEMM_APPLY && two)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = bf2f((x1[k][e >> 1] >> (16 * (e & 1))) & 0xffffu);
      }
      if constexpr (KIND == GEMM_GRAM) {
        // A = alpha^2 X X^T
        const float s2 = alpha * alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = s2 * v[e];
      } else if constexpr (KIND == GEMM_POLY) {
        // A^2 = dA^2 + dA Ao + Ao dA + Ao Ao;  B = b A + c A^2 (b + c dcol is in dcol)
        const float cr = sp.c * (drow[k] + op.xshift);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = sp.c * v[e] + (dcol[e] + cr) * x[e];
      } else if constexpr (KIND == GEMM_SPROD) {
        // (dX + Xo)(dY + Yo) = Xo Yo + dX Yo + Xo dY (+ dX dY on the diagonal)
        const float dr = drow[k] + op.xshift;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] + dr * y[e] + x[e] * dcol[e];
      } else {
        // X'^T = alpha (XT Bo + XT diag(shift + dB))
        if (two) {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] += y[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = alpha * (v[e] + x[e] * dcol[e]);
      }
      if (KIND != GEMM_APPLY && diag) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = row == wch + e ? 0.f : v[e];
      }
      const u32x4 w = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
      *reinterpret_cast<u32x4*>(own) = w;
      if (KIND != GEMM_APPLY || !last) *at(out, k) = w;
      if (KIND == GEMM_APPLY && two && !last) {
        u32x4 l;
#pragma unroll
        for (int e = 0; e < 4; ++e) l[e] = pack_bf2(v[2 * e] - bf2f(w[e] & 0xffffu), v[2 * e + 1] - bf2f(w[e] >> 16));
        *at(outl, k) = l;
      }
    }
  };
  if (kind == GEMM_GRAM) rows(std::integral_constant<int, GEMM_GRAM>{});
  else if (kind == GEMM_POLY) rows(std::integral_constant<int, GEMM_POLY>{});
  else if (kind == GEMM_SPROD) rows(std::integral_constant<int, GEMM_SPROD>{});
  else rows(std::integral_constant<int, GEMM_APPLY>{});
  if (!last && (kind == GEMM_APPLY || diag)) return;
  __syncthreads();

  // mirror: 16-lane group g reads tile rows R0 .. R0 + 7 of columns C0 .. C0 + 15
  const int g = lane >> 4, li = lane & 15;
  auto mirror = [&](int C0, int R0) __attribute__((always_inline)) {
    const int sr = R0 + (li >> 2), sc = C0 + 4 * (li & 3);
    const v4i16 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)tb(sr, sc));
    const v4i16 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)tb(sr + 4, sc));
    return __builtin_bit_cast(u32x4, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  constexpr int RB = T / 32;  // 32-row blocks; a wave takes ROW_ITS blocks of 32 rows x 16 columns
  static_assert(NWAVES * ROW_ITS == RB * (T / 16), "both orders hand out the same number of chunks per lane");
  if (!last) {
#pragma unroll 2
    for (int k = 0; k < ROW_ITS; ++k) {
      const int t = wave * ROW_ITS + k, C0 = (t / RB) * 16, R0 = 32 * (t % RB) + 8 * g;
      *gptr(reinterpret_cast<u32x4*>(out + (col0 + C0 + li) * ld + row0 + R0)) = mirror(C0, R0);
    }
    return;
  }

  // ---- last apply: W <- decay W - lr s dscale X5 (and D), tall: the tile of
  // X^T is a tile of W; wide: its mirror is.  All loads of a batch are issued
  // before its stores. ----
  const int64_t n = d.n, wm0 = d.tall ? row0 : col0, wn0 = d.tall ? col0 : row0;
  const float dscale = d.s * sp.dscale;
  float* const Dp = sp.write_d ? d.D : nullptr;
  auto write = [&](auto wtag) __attribute__((always_inline)) {
    using WT_ = decltype(wtag);
    WT_* W = reinterpret_cast<WT_*>(d.W);
    if ((n & 7) == 0) {
      constexpr int NB = ROW_ITS < 4 ? ROW_ITS : 4;
      for (int k0 = 0; k0 < ROW_ITS; k0 += NB) {
        float w8[NB][8];
        int64_t off[NB];
        u32x4 x[NB];
#pragma unroll
        for (int kk = 0; kk < NB; ++kk) {
          const int k = k0 + kk;
          int64_t wr, wc;
          if (d.tall) {
            wr = wm0 + k * RPI + wrow;
            wc = wn0 + wch;
            x[kk] = *reinterpret_cast<const u32x4*>(tb(k * RPI + wrow, wch));
          } else {
            const int t = wave * ROW_ITS + k, C0 = (t / RB) * 16, R0 = 32 * (t % RB) + 8 * g;
            wr = wm0 + C0 + li;
            wc = wn0 + R0;
            x[kk] = mirror(C0, R0);
          }
          off[kk] = wr < d.m && wc < n ? wr * n + wc : -1;  // n is a multiple of 8: a chunk is whole or outside
          if (off[kk] >= 0) Vec<WT_>::load8(W + off[kk], w8[kk]);
        }
#pragma unroll
        for (int kk = 0; kk < NB; ++kk) {
          if (off[kk] < 0) continue;
          float dv[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            dv[e] = dscale * bf2f((x[kk][e >> 1] >> (16 * (e & 1))) & 0xffffu);
            w8[kk][e] = w8[kk][e] * sp.decay - sp.lr * dv[e];
          }
          Vec<WT_>::store8(W + off[kk], w8[kk]);
          if (Dp) Vec<float>::store8(Dp + off[kk], dv);
        }
      }
    } else {
      // rows that are no multiple of 8 long: consecutive lanes take consecutive elements
      constexpr int NB = 8;
      for (int k0 = 0; k0 < T * T / NTHREADS; k0 += NB) {
        float wv[NB];
        uint16_t x[NB];
#pragma unroll
        for (int kk = 0; kk < NB; ++kk) {
          const int e = (k0 + kk) * NTHREADS + tid, wr = e / T, wc = e % T;
          x[kk] = *reinterpret_cast<const uint16_t*>(d.tall ? tb(wr, wc) : tb(wc, wr));
          if (wm0 + wr < d.m && wn0 + wc < n) wv[kk] = Vec<WT_>::load1(W + (wm0 + wr) * n + wn0 + wc);
        }
#pragma unroll
        for (int kk = 0; kk < NB; ++kk) {
          const int e = (k0 + kk) * NTHREADS + tid, wr = e / T, wc = e % T;
          if (wm0 + wr < d.m && wn0 + wc < n) {
            const float dv = dscale * bf2f(x[kk]);
            Vec<WT_>::store1(W + (wm0 + wr) * n + wn0 + wc, wv[kk] * sp.decay - sp.lr * dv);
            if (Dp) Vec<float>::store1(Dp + (wm0 + wr) * n + wn0 + wc, dv);
          }
        }
      }
    }
  };
  if (sp.wtype == BF16) write(uint16_t{});
  else write(float{});
}

// The products of a launch travel as one packed word each: with the work lists
// they fill the kernel arguments that the dispatcher preloads into scalar
// registers (build.py), so a work group starts on its work item without first
// reading its arguments from host memory.
static uint32_t ns_pack(const NsOp& o, int hilo) {
  return (uint32_t)o.kind | (uint32_t)o.src << 2 | (uint32_t)o.use_alpha << 3 | (uint32_t)o.last << 4 |
         (uint32_t)o.sx << 5 | (uint32_t)o.sy << 8 | (uint32_t)o.so << 11 | (uint32_t)(o.xshift != 0) << 14 |
         (uint32_t)(o.yshift != 0) << 15 | (uint32_t)(hilo != 0) << 16;
}

hipError_t launch_ns_small(int tile, const MatDesc* md, const Item* items0, int32_t n0, const NsOp& op0,
                           const Item* items1, int32_t n1, const NsOp& op1, const NsStepParams& p, hipStream_t s) {
  if (n0 + n1 <= 0) return hipSuccess;
  const dim3 g(n0 + n1), b(small::NTHREADS);
  const uint32_t w0 = ns_pack(op0, p.hilo), w1 = ns_pack(op1, p.hilo);
  // three stages: two to four keep the loads' rate (about 38 bytes per clock
  // and CU at either tile size), and 48 KB let three 64 x 64 tiles share a CU
  if (tile == 64) ns_small_kernel<64, 3><<<g, b, 0, s>>>(md, items0, n0, items1, w0, w1, p);
  else if (tile == 128) ns_small_kernel<128, 3><<<g, b, 0, s>>>(md, items0, n0, items1, w0, w1, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace prm
