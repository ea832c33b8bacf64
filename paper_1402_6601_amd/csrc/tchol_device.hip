// Device side of tchol: one persistent kernel that executes a tile DAG.
//
// Worker loop (one workgroup = one worker, section 2.1 of the paper: a worker
// repeatedly takes a task, runs it, then activates its successors):
//   claim   ticket t = atomicAdd(ticket); (task, part) = items[t]
//   wait    until dep[task] == 0 (agent-scope acquire; bounded by a watchdog)
//   run     the work item (a POTRF tile, a TRSM row strip, a GEMM/SYRK
//           sub-tile, a solve block)
//   publish every global store of the item is a device-scope (write-through)
//           store (st_dev; no result may be written with a plain global
//           store); each wavefront waits for them (vmcnt(0)), then a barrier,
//           then done[task] += 1; the last work item of a task decrements
//           dep[s] of every successor s ("activate").  Readers acquire at
//           agent scope after their wait, so they see the written-through
//           results; no release fence (an L2 write-back) is needed.
// Tickets are handed out in a topological order, so the worker holding the
// oldest unfinished ticket always has its predecessors finished or held by
// running workers: the loop cannot deadlock, whatever the grid size.
//
// All matrices are column-major FP64 with leading dimension `ld`; tile (i, j)
// of the matrix starts at A + (j*nb)*ld + i*nb.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kargs.h"
#include <type_traits>
#include "tchol_kinds.h"

#define NT 256                 // threads per workgroup: 4 wavefronts of 64
#define LDS_DOUBLES 20352      // 162816 bytes of LDS per workgroup (gfx950 allows 163840)
#define LDS_COMPACT_DOUBLES 10112  // of the compact instance, two workgroups per compute unit

typedef double d4 __attribute__((ext_vector_type(4)));

// FP64 matrix-core product on 16x16x4 blocks:  D = A(16x4) * B(4x16) + C.
// Lane l supplies A[l%16][l/16] and B[l/16][l%16]; it receives D[4i + l/16][l%16]
// in element i of the result.  Every caller below passes the B-panel fragment
// as the A operand and the (negated) A-panel fragment as the B operand, so a
// lane's four results are four consecutive COLUMNS of one row of the output
// tile: rows map to l%16 and columns to 4i + l/16.
__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }
__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }

// Value of v in lane l (l wave-uniform), as a scalar broadcast.
__device__ __forceinline__ double readlane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// ---------------------------------------------------------------------------
// Direct global -> LDS loads.  One instruction moves 16 (or 4) bytes per lane
// into LDS at a wave-uniform base (M0) + lane * size, without passing through
// registers, so the K panels stream in while the matrix cores run.
//
// They are issued as inline assembly rather than through the compiler's
// builtin: for the builtin, the compiler cannot tell which LDS stage a load
// writes, so it waits for every outstanding load (vmcnt(0)) before the next
// LDS read, which serialises each chunk's load with the previous chunk's
// products.  Issued this way the compiler does not track them at all, and
// every consumer waits for them explicitly (vmcnt counts, then a workgroup
// barrier) before reading the stage they fill.  M0 is set in the same
// statement; it is a reserved register the compiler sets itself before each of
// its own uses (these kernels have none).
//
// The wait states that the compiler adds to its own code are missing inside an
// assembly statement, so each statement brings them along: one instruction
// between the scalar write of M0 and the transfer that reads it, and a base in
// scalar registers that a scalar instruction of the statement wrote (a copy to
// VCC).  The base itself often comes from a readfirstlane or from a spilled
// scalar, which are vector instructions, and a memory instruction may read a
// scalar register only five wait states after a vector instruction wrote it.
// (the low word of a generic pointer into LDS is the LDS byte address; a cast
// of the pointer to LDS would add a test for null to every transfer)
__device__ __forceinline__ uint32_t lds_addr(double* l) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)l);
}
__device__ __forceinline__ void dma16(const void* g, double* l) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr(l)), "v"(g) : "memory");
}
// The same from a wave-uniform base (scalar registers) plus a per-lane byte
// offset below 4 GB: one 32-bit register per lane instead of a 64-bit address.
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const void*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void dma16s(const void* base, uint32_t off, double* l) {
  asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 vcc, %2\n\tglobal_load_lds_dwordx4 %1, vcc"
               : : "s"(lds_addr(l)), "v"(off), "s"(uniform_ptr(base)) : "memory", "vcc");
}
__device__ __forceinline__ void dma4s(const void* base, uint32_t off, double* l) {
  asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 vcc, %2\n\tglobal_load_lds_dword %1, vcc"
               : : "s"(lds_addr(l)), "v"(off), "s"(uniform_ptr(base)) : "memory", "vcc");
}

// The same with the LDS address as a wave-uniform byte address plus a
// constant, one scalar add.
template <int IMM>
__device__ __forceinline__ void dma16i(uint64_t base, uint32_t off, uint32_t l) {
  asm volatile("s_add_u32 m0, %0, %1\n\ts_mov_b64 vcc, %3\n\tglobal_load_lds_dwordx4 %2, vcc"
               : : "s"(l), "n"(IMM), "v"(off), "s"(base) : "memory", "scc", "vcc");
}
template <int IMM>
__device__ __forceinline__ void dma4i(uint64_t base, uint32_t off, uint32_t l) {
  asm volatile("s_add_u32 m0, %0, %1\n\ts_mov_b64 vcc, %3\n\tglobal_load_lds_dword %2, vcc"
               : : "s"(l), "n"(IMM), "v"(off), "s"(base) : "memory", "scc", "vcc");
}

constexpr int imin_c(int a, int b) { return a < b ? a : b; }

// Makes every value of v available at this point (the compiler waits for
// their loads here).  A value loaded only to be used under a condition would
// otherwise have its load moved under that condition, one load and one wait
// per value; issued unconditionally before this point, the loads overlap.
template <int C>
__device__ __forceinline__ void materialize(double (&v)[C]) {
#pragma unroll
  for (int c = 0; c < C; ++c) asm volatile("" : : "v"(v[c]));
}
template <int R, int C>
__device__ __forceinline__ void materialize(double (&v)[R][C]) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) asm volatile("" : : "v"(v[r][c]));
}

// Store with device (agent) scope: it is written through to the device's
// point of coherence instead of staying dirty in this XCD's L2.  All results
// a work item publishes to other workgroups are written this way.
__device__ __forceinline__ void st_dev(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(float* p, float v) {
  __hip_atomic_store(reinterpret_cast<uint32_t*>(p), __float_as_uint(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

typedef float f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_dev(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// BF16 (the upper half of an FP32 word) rounded to nearest even, and back.
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ double bf16_val(uint32_t h) { return (double)__uint_as_float(h << 16); }
// x as hi + mid + lo, three BF16 terms of decreasing magnitude (each the
// rounded remainder of the previous ones; the remainders are exact in FP64),
// good to about 2^-24 relative, i.e. FP32 level.
__device__ __forceinline__ void split3(double x, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = bf16_rne((float)x);
  const double r1 = x - bf16_val(h);
  m = bf16_rne((float)r1);
  l = bf16_rne((float)(r1 - bf16_val(m)));
}

// f(0), ..., f(N - 1) with compile-time arguments.
template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    static_for<N, F, I + 1>(f);
  }
}

// s_waitcnt vmcnt(N) with the other counters left alone (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier for data in LDS only: it waits for this wavefront's LDS
// accesses, not for its global stores (__syncthreads waits for both, and a
// write-through store takes thousands of cycles).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// ---------------------------------------------------------------------------
// Matrix-core tile product for a result that stays in LDS (the panels of
// potrf_tile and prev_tile, the adjoint's 64 x 64 blocks; whole work items of
// 128 x 128 take gemm_tile, below):
//     C[M x N] - Ap[M x K] * Bp[N x K]^T,   M <= BM, N <= BN, K % KC == 0.
// The four wavefronts form a WGM x (4/WGM) grid; each owns a (BM/WGM) x
// (BN*WGM/4) piece of C as 16x16 MFMA blocks held in registers from the load
// of C to the end.  K is streamed in chunks of KC
// columns through NST LDS stages filled by direct-to-LDS loads, NST-1 chunks
// ahead of the matrix cores.  SEG = 128 moves 16 bytes per lane (rows in
// pairs) and needs even ld, 16-byte aligned panels, and, when M or N is odd,
// one readable row after the panel; SEG = 32 moves 4 bytes per lane and has
// no such needs.  Row indices are clamped into the panel
// (rows past M hold copies and only feed outputs that are never used).
// gemm_core's result goes to LDS at Cl (column-major, leading dimension ldl;
// it must not overlap the NST stages).
//
// The chunk loop is kept free of branches in its steady state (the transfer
// width is fixed per kernel instance, a transfer slot's panel is known at
// compile time, and the last NST-1 chunks are peeled off), so that the
// accumulators stay in the matrix-core registers across chunks.
template <int BM, int BN, int KC, int WGM, int NST, int PAD>
struct GemmShape {
  static constexpr int WGN = 4 / WGM;
  static constexpr int WTM = BM / WGM, WTN = BN / WGN;
  static constexpr int RB = WTM / 16, CB = WTN / 16;
  // LDS rows of the staged panels (one k index each) may be padded
  static constexpr int ALD = BM + PAD, BLD = BN + PAD;
  static constexpr int STAGE = KC * (ALD + BLD);  // doubles per stage
  static_assert(NST * STAGE <= LDS_DOUBLES, "stages must fit the workgroup LDS");
  static_assert(BM % 128 == 0 || 128 % BM == 0, "a 1 KB segment must cover whole rows or a row part");
  static_assert(BN % 128 == 0 || 128 % BN == 0, "a 1 KB segment must cover whole rows or a row part");
  static_assert(PAD == 0 || (BM % 128 == 0 && BN % 128 == 0), "padded rows need segments that stay within a row");
};

// K loop with SEG-double transfers per wavefront instruction (128: 16-byte
// lanes, 32: 4-byte lanes).
template <int BM, int BN, int KC, int WGM, int NST, int PAD, int SEG, int RB, int CB>
__device__ __forceinline__ void gemm_kloop(d4 (&acc)[RB][CB], const double* __restrict__ Ap,
                                           const double* __restrict__ Bp, int64_t ld, int M, int N, int K,
                                           double* lds, int64_t ldb_ = -1) {
  const int64_t ldB = ldb_ < 0 ? ld : ldb_;  // the B panel's leading dimension (default: A's)
  using S = GemmShape<BM, BN, KC, WGM, NST, PAD>;
  static_assert(RB == S::RB && CB == S::CB, "accumulator shape");
  constexpr int ALD = S::ALD, BLD = S::BLD, STAGE = S::STAGE;
  constexpr int QA = KC * BM / SEG, QB = KC * BN / SEG;  // transfers per stage
  static_assert(QA * SEG == KC * BM && QB * SEG == KC * BN, "stage must be whole segments");
  // When both counts divide by four, transfer slot j of every wavefront
  // serves the same panel and every wavefront issues the same number.
  constexpr bool UNIFORM = (QA % 4 == 0) && (QB % 4 == 0);
  constexpr int J = (QA + QB + 3) / 4;  // transfer slots per wavefront
  constexpr int W = (QA + QB) / 4;      // fewest transfers per wavefront and chunk
  static_assert(W >= 1, "every wavefront must issue transfers for every chunk");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WGN, wn = wave % S::WGN;
  const int l16 = lane & 15, lg = lane >> 4;

  // One transfer: segment q of panel X (rows R = BM or BN, valid rows V) of
  // chunk ch.  A segment covers consecutive doubles of the column-major
  // panel: part of one k row, or whole k rows when the row is shorter than
  // the segment (then the rows are unpadded and contiguous).  Each 16-byte
  // lane moves rows (r, r + 1); each 4-byte lane half of one double.
  //
  // The address is split into a wave-uniform base and a per-lane offset.
  // Either a segment lies within one k row (R a multiple of SEG; it starts at
  // row u = e0 % R of k row e0 / R) or it covers whole k rows (R divides
  // SEG, u = 0; lane element le falls in k row e0 / R + le / R).  Rows are
  // clamped to the last valid start row Vc; the base takes min(u, Vc), so
  // the lane offsets are never negative.
  auto xfer = [&](const double* X, int64_t ld, int R, int XLD, int V, int q, int k0, double* dst)
                  __attribute__((always_inline)) {
    const int e0 = q * SEG;
    const int le = SEG == 128 ? 2 * lane : (lane >> 1);
    // a pair starts at an even row no later than V - 1; for odd V the pair
    // (V - 1, V) reads the row after the panel, which the launch contract
    // guarantees to exist (leading dimension above the order)
    const int Vc = SEG == 128 ? ((V - 1) & ~1) : V - 1;
    const int u = e0 % R, cu = e0 / R, ru = imin(u, Vc);
    const int cl = (R % SEG == 0) ? 0 : le / R;
    const int rl = ((R % SEG == 0) ? imin(u + le, Vc) : imin(le % R, Vc)) - ru;
    const double* base = X + (int64_t)(k0 + cu) * ld + ru;
    const uint32_t off = (uint32_t)(((int64_t)cl * ld + rl) * 8);
    if (SEG == 128)
      dma16s(base, off, dst + cu * XLD + u);
    else
      dma4s(base, off + 4 * (lane & 1), dst + cu * XLD + u);
  };
  auto slot = [&](int j, int k0, double* As, double* Bs) __attribute__((always_inline)) {
    const int q = wave + 4 * j;
    if (UNIFORM) {
      if (j < QA / 4) xfer(Ap, ld, BM, ALD, M, q, k0, As);
      else xfer(Bp, ldB, BN, BLD, N, q - QA, k0, Bs);
    } else {
      if (q < QA) xfer(Ap, ld, BM, ALD, M, q, k0, As);
      else if (q < QA + QB) xfer(Bp, ldB, BN, BLD, N, q - QA, k0, Bs);
    }
  };
  auto issue = [&](int ch) __attribute__((always_inline)) {
    double* As = lds + (ch % NST) * STAGE;
    double* Bs = As + KC * ALD;
    const int k0 = ch * KC;
    if constexpr (SEG == 128) {
#pragma unroll
      for (int j = 0; j < J; ++j) slot(j, k0, As, Bs);
    } else {  // many narrow transfers: a rolled loop keeps their addresses out of registers
#pragma unroll 2
      for (int j = 0; j < J; ++j) slot(j, k0, As, Bs);
    }
  };
  // compute(ch, nx): the products of chunk ch; with nx >= 0 the transfers of
  // chunk nx are issued along the way, a few per k-step, so that the matrix
  // cores are not idle while a whole chunk's transfers are issued
  auto compute = [&](int ch, int nx) __attribute__((always_inline)) {
    const double* as = lds + (ch % NST) * STAGE;
    const double* bs = as + KC * ALD;
    double* nAs = lds + ((nx < 0 ? 0 : nx) % NST) * STAGE;
    double* nBs = nAs + KC * ALD;
    constexpr int PER = (J + KC / 4 - 1) / (KC / 4);  // transfer slots per k-step
    // fragments of k-step ks + 1 are read while the MFMAs of ks run
    double fa[2][RB], fb[2][CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) fa[0][rb] = as[lg * ALD + wm * S::WTM + rb * 16 + l16];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) fb[0][cb] = bs[lg * BLD + wn * S::WTN + cb * 16 + l16];
#pragma unroll
    for (int ks = 0; ks < KC / 4; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1;
      if (nx >= 0) {
#pragma unroll
        for (int jj = 0; jj < PER; ++jj)
          if (ks * PER + jj < J) slot(ks * PER + jj, nx * KC, nAs, nBs);
      }
      if (ks + 1 < KC / 4) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) fa[nxt][rb] = as[((ks + 1) * 4 + lg) * ALD + wm * S::WTM + rb * 16 + l16];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) fb[nxt][cb] = bs[((ks + 1) * 4 + lg) * BLD + wn * S::WTN + cb * 16 + l16];
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[rb][cb] =
              __builtin_amdgcn_mfma_f64_16x16x4f64(fb[cur][cb], fa[cur][rb], acc[rb][cb], 0, 0, 2 /* neg B */);
    }
  };

  // Chunk ch has landed once no more than the later chunks' transfers are
  // outstanding.  A wavefront issues W (or, when not UNIFORM, W + 1)
  // transfers per chunk; waiting for "at most W per later chunk" (capped at
  // the counter's range) is exact or stricter, never short.
  //
  // The first chunk waits for everything outstanding: the caller's loads of
  // C are then known complete, and the compiler (which tracks those loads but
  // not the direct-to-LDS ones) inserts no waits of its own into the loop.
  const int nch = K / KC;
  if (nch <= 0) return;
#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nch) issue(p);
  wait_vmcnt<0>();
  __syncthreads();
  compute(0, NST - 1 < nch ? NST - 1 : -1);
  int ch = 1;
  for (; ch + NST - 1 < nch; ++ch) {  // steady state: NST - 2 later chunks in flight
    wait_vmcnt<imin_c((NST - 2) * W, 63)>();
    __syncthreads();
    compute(ch, ch + NST - 1);
  }
  for (; ch < nch; ++ch) {  // the last NST - 1 chunks: nothing more to issue
    const int later = nch - 1 - ch;
    if (later >= 2) wait_vmcnt<imin_c(2 * W, 63)>();
    else if (later == 1) wait_vmcnt<imin_c(W, 63)>();
    else wait_vmcnt<0>();
    __syncthreads();
    compute(ch, -1);
  }
}

// ldc: leading dimension of C when it differs from the panels' (< 0: ld).  The
// result goes to LDS at Cl (column-major, leading dimension ldl).
template <int SEG, int BM, int BN, int KC, int WGM, int NST, int PAD>
__device__ __forceinline__ void gemm_core(const double* __restrict__ C, const double* __restrict__ Ap,
                                          const double* __restrict__ Bp, int64_t ld, int M, int N, int K, double* lds,
                                          double* Cl, int ldl, int64_t ldc = -1) {
  const int64_t ldC = ldc < 0 ? ld : ldc;
  using S = GemmShape<BM, BN, KC, WGM, NST, PAD>;
  constexpr int RB = S::RB, CB = S::CB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WGN, wn = wave % S::WGN;
  const int l16 = lane & 15, lg = lane >> 4;

  d4 acc[RB][CB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * S::WTM + rb * 16 + l16, col = wn * S::WTN + cb * 16 + 4 * i + lg;
        acc[rb][cb][i] = C[(int64_t)imin(col, N - 1) * ldC + imin(row, M - 1)];
      }

  gemm_kloop<BM, BN, KC, WGM, NST, PAD, SEG>(acc, Ap, Bp, ld, M, N, K, lds);
  __syncthreads();  // every wavefront is done with the stages before LDS is reused

#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * S::WTM + rb * 16 + l16, col = wn * S::WTN + cb * 16 + 4 * i + lg;
        if (row < M && col < N) Cl[col * ldl + row] = acc[rb][cb][i];
      }
}

// GEMM / SYRK work item: a 128 x 128 sub-tile of C -= Ap Bp^T (or, zero_c with
// neg, C := Ap Bp^T), M, N <= 128, K a multiple of 16.  2 x 2 wavefronts of
// 64 x 64; the panels stream through four LDS stages of 16 columns, as in
// gemm_kloop (SEG, row clamping and alignment as there).  What differs, to
// keep the matrix cores fed between chunks and at the ends of the item:
//  - a chunk has landed one whole chunk before its products start, so the
//    first fragments of the next chunk are read under the current one's last
//    products, and the barrier between them finds the next products ready;
//  - a transfer costs five scalar-side instructions (a running pointer per
//    panel, the LDS address from one base), and what a k-step issues besides
//    its products is spread between them in small groups: a wavefront issues
//    in order, and whatever takes longer than the product before it leaves
//    the matrix core idle;
//  - the product is accumulated from zero and C is subtracted at the end: C is
//    requested once the last transfer has landed, two chunks before the end,
//    and its memory time passes under their products.
// Per 128 x 128 item, all 256 workgroups busy, K = 1024 (n = 16384) 138 -> 127
// us and K = 256 (tiles of 128, n = 8192) 43 -> 39 us, of which the products
// take 109 and 27 us at 2.4 GHz: 1.9 us per 16-column chunk against 1.7, 2.8
// us before the first product, 1.4 us of C not hidden, 2.4 us of stores.
#define GB 128
template <int SEG>
__device__ __forceinline__ void gemm_tile(double* __restrict__ C, int64_t ldC, const double* __restrict__ Ap, int64_t ld,
                                          const double* __restrict__ Bp, int64_t ldB, int M, int N, int K,
                                          bool lower_only, bool zero_c, bool neg, double* lds) {
  constexpr int KC = 16, NST = 4, XLD = GB + 2, STAGE = 2 * KC * XLD;
  constexpr int Q = KC * GB / SEG;     // transfers per panel and stage
  constexpr int J = 2 * Q / 4;         // per wavefront: J / 2 of A, then J / 2 of B
  constexpr int PER = J / (KC / 4);    // per k-step
  constexpr int ROWS = 4 * SEG / GB;   // k-rows that a round of the four wavefronts covers
  static_assert(NST * STAGE <= LDS_DOUBLES && J * 4 == 2 * Q && PER * (KC / 4) == J && J <= 63 && ROWS >= 1,
                "stages and transfers");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;

  // this wavefront's transfers: segment wave + 4 j of a panel, j counting on
  // from chunk to chunk, so a running pointer per panel; rows clamped to the
  // last valid start row as in gemm_kloop
  const int le = SEG == 128 ? 2 * lane : (lane >> 1);
  const int u = (wave * SEG) % GB, cu = (wave * SEG) / GB;
  auto lane_off = [&](int V) __attribute__((always_inline)) {
    return (uint32_t)(imin(u + le, SEG == 128 ? ((V - 1) & ~1) : V - 1) * 8 + (SEG == 128 ? 0 : 4 * (lane & 1)));
  };
  const uint32_t offa = lane_off(M), offb = lane_off(N);
  uint64_t pa = (uint64_t)(uintptr_t)uniform_ptr(Ap + (int64_t)cu * ld);
  uint64_t pb = (uint64_t)(uintptr_t)uniform_ptr(Bp + (int64_t)cu * ldB);
  const uint64_t da = (uint64_t)(ROWS * 8) * (uint64_t)ld, db = (uint64_t)(ROWS * 8) * (uint64_t)ldB;
  const uint32_t l0 = lds_addr(lds) + (uint32_t)(cu * XLD + u) * 8;
  auto slot = [&](auto jc, uint32_t st) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    constexpr int imm = (j < J / 2 ? j * ROWS : KC + (j - J / 2) * ROWS) * XLD * 8;
    if constexpr (j < J / 2) {
      if constexpr (SEG == 128) dma16i<imm>(pa, offa, st);
      else dma4i<imm>(pa, offa, st);
      pa += da;
    } else {
      if constexpr (SEG == 128) dma16i<imm>(pb, offb, st);
      else dma4i<imm>(pb, offb, st);
      pb += db;
    }
  };
  auto issue = [&](int ch) __attribute__((always_inline)) {
    const uint32_t st = l0 + (uint32_t)(ch % NST) * (STAGE * 8);
    static_for<J>([&](auto jc) __attribute__((always_inline)) { slot(jc, st); });
  };
  d4 acc[4][4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[rb][cb] = d4{0.0, 0.0, 0.0, 0.0};
  double fa[2][4], fb[2][4];
  const double* const fa0 = lds + lg * XLD + wm * 64 + l16;
  const double* const fb0 = lds + (KC + lg) * XLD + wn * 64 + l16;
  auto read_a = [&](int so, int ks, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) fa[buf][rb] = fa0[so + ks * 4 * XLD + rb * 16];
  };
  auto read_b = [&](int so, int ks, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) fb[buf][cb] = fb0[so + ks * 4 * XLD + cb * 16];
  };
  // the products of the chunk in the stage at so (doubles), the first fragments
  // of the next one, at sn; with ISSUE the transfers of the chunk for stage
  // st go out along them, else extra(k-step, group of products) is called
  auto compute = [&](auto issue_c, int so, int sn, uint32_t st, auto extra) __attribute__((always_inline)) {
    constexpr bool ISSUE = decltype(issue_c)::value;
    static_for<KC / 4>([&](auto kc) __attribute__((always_inline)) {
      constexpr int ks = decltype(kc)::value, cur = ks & 1, nxt = cur ^ 1;
      constexpr bool last = ks + 1 == KC / 4;
      auto products = [&](int rb) __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) acc[rb][cb] = mfma_f64(fb[cur][cb], fa[cur][rb], acc[rb][cb]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!ISSUE) extra(kc, rb);
      };
      products(0);
      // (after the last chunk: a stage that is not read, so no condition)
      read_a(last ? sn : so, last ? 0 : ks + 1, nxt);
      __builtin_amdgcn_sched_barrier(0);
      products(1);
      read_b(last ? sn : so, last ? 0 : ks + 1, nxt);
      __builtin_amdgcn_sched_barrier(0);
      products(2);
      if constexpr (ISSUE)
        static_for<PER / 2>([&](auto jj) __attribute__((always_inline)) {
          slot(std::integral_constant<int, ks * PER + decltype(jj)::value>(), st);
        });
      __builtin_amdgcn_sched_barrier(0);
      products(3);
      if constexpr (ISSUE)
        static_for<PER - PER / 2>([&](auto jj) __attribute__((always_inline)) {
          slot(std::integral_constant<int, ks * PER + PER / 2 + decltype(jj)::value>(), st);
        });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  const int nch = K / KC;
#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nch) issue(p);
  // chunks 0 and 1 landed (everything, when there is no third)
  if (nch >= 3) wait_vmcnt<J>();
  else wait_vmcnt<0>();
  lds_barrier();
  read_a(0, 0, 0);
  read_b(0, 0, 0);
  auto nothing = [](auto, int) __attribute__((always_inline)) {};
  int so = 0;  // the current chunk's stage
  auto after = [&](int o) __attribute__((always_inline)) { return o == (NST - 1) * STAGE ? 0 : o + STAGE; };
  int ch = 0;
  for (; ch + NST - 1 < nch; ++ch) {
    const int sn = after(so), sw = so == 0 ? (NST - 1) * STAGE : so - STAGE;
    compute(std::true_type(), so, sn, l0 + (uint32_t)sw * 8, nothing);
    so = sn;
    wait_vmcnt<J>();  // chunk ch + 2 has landed, ch + 3 may be in flight
    lds_barrier();
  }
  for (; ch + 2 < nch; ++ch) {  // at most one: nothing left to issue
    const int sn = after(so);
    compute(std::false_type(), so, sn, 0, nothing);
    so = sn;
    wait_vmcnt<0>();
    lds_barrier();
  }
  // the last two chunks, with C on the way: of a whole tile four loads after
  // every group of the first one's products (all at once they would fill the
  // memory pipeline and hold up the products), at one pointer per column of a lane and
  // constant row offsets (address arithmetic in vector instructions would
  // cost more than the loads)
  const bool whole = M == GB && N == GB;
  double* const Cl = C + (int64_t)(wn * 64 + lg) * ldC + wm * 64 + l16;
  const bool early = whole && !zero_c && nch >= 2;
  double c[4][4][4];
  if (zero_c) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) c[rb][cb][i] = 0.0;
  } else if (!early) {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = wm * 64 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * i + lg;
          c[rb][cb][i] = C[(int64_t)imin(col, N - 1) * ldC + imin(row, M - 1)];
        }
  }
  __builtin_amdgcn_sched_barrier(0);
  if (nch >= 2) {  // (both chunks landed before: no wait, no barrier between them)
    const int sn = after(so);
    compute(std::false_type(), so, sn, 0, [&](auto kc, int g) __attribute__((always_inline)) {
      constexpr int ks = decltype(kc)::value;  // column block ks, element g of its columns
      if (early) {
        const double* const q = Cl + (int64_t)(ks * 16 + 4 * g) * ldC;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) c[rb][ks][g] = q[rb * 16];
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    so = sn;
  }
  compute(std::false_type(), so, after(so), 0, nothing);
  lds_barrier();  // every wavefront is done with the stages before LDS is reused
  const double sgn = neg ? -1.0 : 1.0;
  if (whole && !lower_only) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        double* const q = Cl + (int64_t)(cb * 16 + 4 * i) * ldC;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) st_dev(q + rb * 16, sgn * (c[rb][cb][i] - acc[rb][cb][i]));
      }
  } else {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = wm * 64 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * i + lg;
          if (row < M && col < N && (!lower_only || row >= col))
            st_dev(C + (int64_t)col * ldC + row, sgn * (c[rb][cb][i] - acc[rb][cb][i]));
        }
  }
}

template <int SEG>
__device__ __forceinline__ void gemm_nt(double* C, const double* Ap, const double* Bp, int64_t ld, int M, int N,
                                        int K, bool lower_only, double* lds) {
  gemm_tile<SEG>(C, ld, Ap, ld, Bp, ld, M, N, K, lower_only, false, false, lds);
}

// The same product with C at its own leading dimension ldc (the panels at
// ld), optionally starting from C = 0.
__device__ __forceinline__ void gemm_nt_ex(double* C, int64_t ldc, const double* Ap, const double* Bp, int64_t ld,
                                           int M, int N, int K, bool lower_only, bool zero_c, double* lds) {
  gemm_tile<128>(C, ldc, Ap, ld, Bp, ld, M, N, K, lower_only, zero_c, false, lds);
}

// ---------------------------------------------------------------------------
// FP32 tile product for the mixed-precision factorization:
//     C[M x N] -= Ap[M x K] * Bp[N x K]^T in FP32 storage, FP32 MFMA
// (v_mfma_f32_16x16x4f32, the FP64 instruction's shape and operand layout)
// with FP32 accumulation; 128 x 128 outputs, K % KC == 0.  A stage holds KC
// k-rows laid out as [A row (128) | B row (128) | 16 pad] floats, so one
// 16-byte-per-lane transfer moves one k-row of both panels (lanes 0..31: A,
// lanes 32..63: B) and the padded rows keep the fragment reads free of bank
// conflicts.  Rows are moved four at a time: the row group of the last valid
// row may read up to three rows past the panel, which the mixed working copy
// provides (its leading dimension exceeds the order by at least three).
// The f32 MFMA has no operand negation, so the A fragment is negated.  Its
// 16 x 16 result differs in layout from the f64 instruction's: element i of
// lane l holds row 4 (l / 16) + i (not 4 i + l / 16) of column l % 16.
// CD: the product is added to an FP64 C (Cd, ld ldcd) instead: the diagonal
// tiles of the mixed-precision factorization stay in FP64 throughout.
#define F32_LD 272
template <int KC, int NST, bool CD = false>
__device__ __forceinline__ void gemm_f32_core(float* __restrict__ C, const float* __restrict__ Ap,
                                              const float* __restrict__ Bp, int64_t ld, int M, int N, int K,
                                              bool lower_only, double* lds_d, double* __restrict__ Cd = nullptr,
                                              int64_t ldcd = 0) {
  constexpr int STAGE = KC * F32_LD;  // floats per stage
  constexpr int W = KC / 4;           // transfers per wavefront and chunk
  static_assert(NST * STAGE <= 2 * LDS_DOUBLES, "stages must fit the workgroup LDS");
  static_assert(KC % 4 == 0 && W >= 1, "every wavefront transfers whole k-rows");
  float* lds = reinterpret_cast<float*>(lds_d);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;  // 2 x 2 wavefronts, 64 x 64 each
  const int l16 = lane & 15, lg = lane >> 4;
  const bool arow = lane < 32;
  const float* src0 = arow ? Ap + imin(4 * lane, (M - 1) & ~3) : Bp + imin(4 * (lane - 32), (N - 1) & ~3);

  f4 acc[4][4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * 64 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
        acc[rb][cb][i] = CD ? 0.f : C[(int64_t)imin(col, N - 1) * ld + imin(row, M - 1)];
      }

  static_assert(STAGE % 2 == 0 && F32_LD % 2 == 0, "destinations are addressed in doubles");
  auto issue = [&](int ch) __attribute__((always_inline)) {
    // destinations as double pointers into the shared array (stage and row offsets are even)
    double* st = lds_d + (ch % NST) * (STAGE / 2);
    const int k0 = ch * KC;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int q = wave + 4 * j;  // k-row of the chunk
      dma16(src0 + (int64_t)(k0 + q) * ld, st + q * (F32_LD / 2));
    }
  };
  // as in gemm_kloop: the transfers of chunk nx (if any) are issued along the
  // products of chunk ch, one k-row per k-step
  auto compute = [&](int ch, int nx) __attribute__((always_inline)) {
    const float* st = lds + (ch % NST) * STAGE;
    double* nst = lds_d + ((nx < 0 ? 0 : nx) % NST) * (STAGE / 2);
    constexpr int PER = (W + KC / 4 - 1) / (KC / 4);
    float fa[2][4], fb[2][4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) fa[0][rb] = -st[lg * F32_LD + wm * 64 + rb * 16 + l16];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) fb[0][cb] = st[lg * F32_LD + 128 + wn * 64 + cb * 16 + l16];
#pragma unroll
    for (int ks = 0; ks < KC / 4; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1;
      if (nx >= 0) {
#pragma unroll
        for (int jj = 0; jj < PER; ++jj)
          if (ks * PER + jj < W) {
            const int q = wave + 4 * (ks * PER + jj);
            dma16(src0 + (int64_t)(nx * KC + q) * ld, nst + q * (F32_LD / 2));
          }
      }
      if (ks + 1 < KC / 4) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) fa[nxt][rb] = -st[((ks + 1) * 4 + lg) * F32_LD + wm * 64 + rb * 16 + l16];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
          fb[nxt][cb] = st[((ks + 1) * 4 + lg) * F32_LD + 128 + wn * 64 + cb * 16 + l16];
      }
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[cur][cb], fa[cur][rb], acc[rb][cb], 0, 0, 0);
    }
  };
  // as in gemm_kloop: the first chunk waits for everything, the loads of C included
  const int nch = K / KC;
#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nch) issue(p);
  if (nch > 0) {  // (every loop below is reached only through the first chunk's full wait)
    wait_vmcnt<0>();
    __syncthreads();
    compute(0, NST - 1 < nch ? NST - 1 : -1);
    int ch = 1;
    for (; ch + NST - 1 < nch; ++ch) {
      wait_vmcnt<imin_c((NST - 2) * W, 63)>();
      __syncthreads();
      compute(ch, ch + NST - 1);
    }
    for (; ch < nch; ++ch) {
      const int later = nch - 1 - ch;
      if (later >= 2) wait_vmcnt<imin_c(2 * W, 63)>();
      else if (later == 1) wait_vmcnt<imin_c(W, 63)>();
      else wait_vmcnt<0>();
      __syncthreads();
      compute(ch, -1);
    }
  }
  __syncthreads();
  if constexpr (CD) {
    // read-modify-write of the FP64 tile, two row blocks at a time: the 32
    // old values are requested together (clamped into the tile, which is
    // nb x nb in full) and all taken before the first store, one memory
    // round trip per pair instead of one per value
#pragma unroll
    for (int rp = 0; rp < 4; rp += 2) {
      double old[2][16];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = wm * 64 + (rp + h) * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
            old[h][4 * cb + i] = Cd[(int64_t)imin(col, N - 1) * ldcd + imin(row, M - 1)];
          }
      materialize(old);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = wm * 64 + (rp + h) * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
            if (row < M && col < N && (!lower_only || row >= col))
              st_dev(Cd + (int64_t)col * ldcd + row, old[h][4 * cb + i] + (double)acc[rp + h][cb][i]);
          }
    }
  } else {
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = wm * 64 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
          if (row < M && col < N && (!lower_only || row >= col)) st_dev(C + (int64_t)col * ld + row, acc[rb][cb][i]);
        }
  }
}

__device__ __forceinline__ void gemm_nt_f32(float* C, const float* Ap, const float* Bp, int64_t ld, int M, int N,
                                            int K, bool lower_only, double* lds) {
  if (K % 32 == 0)
    gemm_f32_core<32, 4>(C, Ap, Bp, ld, M, N, K, lower_only, lds);
  else
    gemm_f32_core<16, 4>(C, Ap, Bp, ld, M, N, K, lower_only, lds);
}

// FP32 GEMM item with a 256 x 128 output, C[M x N] -= Ap[M x K] Bp[N x K]^T,
// M <= 256, N <= 128 (the mixed-precision factorization's GEMM items): the
// scheme of gemm_f32_core with twice the rows per wavefront (2 x 2
// wavefronts of 128 x 64).  Per k-row of a chunk one 16-byte transfer of all
// 64 lanes moves the 256 A rows and one of lanes 0-31 the 128 B rows into an
// LDS row [A 256 | B 128 | 16 pad]; three stages of 32 k-rows.
#define F32W_LD 400
template <int KC, int NST>
__device__ __forceinline__ void gemm_f32_wide(float* __restrict__ C, const float* __restrict__ Ap,
                                              const float* __restrict__ Bp, int64_t ld, int M, int N, int K,
                                              double* lds_d) {
  constexpr int STAGE = KC * F32W_LD;  // floats per stage
  constexpr int W = 2 * (KC / 4);      // transfers per wavefront and chunk: two per k-row, KC / 4 k-rows
  static_assert(NST * STAGE <= 2 * LDS_DOUBLES, "stages must fit the workgroup LDS");
  static_assert(KC % 4 == 0 && W <= 63, "every wavefront transfers whole k-rows");
  float* lds = reinterpret_cast<float*>(lds_d);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;  // 2 x 2 wavefronts, 128 x 64 each
  const int l16 = lane & 15, lg = lane >> 4;
  const float* srcA = Ap + imin(4 * lane, (M - 1) & ~3);
  const float* srcB = Bp + imin(4 * (lane & 31), (N - 1) & ~3);

  f4 acc[8][4];
#pragma unroll
  for (int rb = 0; rb < 8; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * 128 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
        acc[rb][cb][i] = C[(int64_t)imin(col, N - 1) * ld + imin(row, M - 1)];
      }

  static_assert(STAGE % 2 == 0 && F32W_LD % 2 == 0, "destinations are addressed in doubles");
  // the two transfers of k-row q of chunk ch (doubles: a row is F32W_LD / 2, B starts at 128)
  auto xfer = [&](int ch, int q) __attribute__((always_inline)) {
    double* st = lds_d + (ch % NST) * (STAGE / 2) + q * (F32W_LD / 2);
    const int64_t k = (int64_t)(ch * KC + q) * ld;
    dma16(srcA + k, st);
    if (lane < 32) dma16(srcB + k, st + 128);
  };
  auto issue = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < KC / 4; ++j) xfer(ch, wave + 4 * j);
  };
  // the products of chunk ch; the transfers of chunk nx (if any) go out along
  // them, one k-row per k-step
  auto compute = [&](int ch, int nx) __attribute__((always_inline)) {
    const float* st = lds + (ch % NST) * STAGE;
    float fa[2][8], fb[2][4];
#pragma unroll
    for (int rb = 0; rb < 8; ++rb) fa[0][rb] = -st[lg * F32W_LD + wm * 128 + rb * 16 + l16];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) fb[0][cb] = st[lg * F32W_LD + 256 + wn * 64 + cb * 16 + l16];
#pragma unroll
    for (int ks = 0; ks < KC / 4; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1;
      if (nx >= 0) xfer(nx, wave + 4 * ks);
      if (ks + 1 < KC / 4) {
#pragma unroll
        for (int rb = 0; rb < 8; ++rb)
          fa[nxt][rb] = -st[((ks + 1) * 4 + lg) * F32W_LD + wm * 128 + rb * 16 + l16];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) fb[nxt][cb] = st[((ks + 1) * 4 + lg) * F32W_LD + 256 + wn * 64 + cb * 16 + l16];
      }
#pragma unroll
      for (int rb = 0; rb < 8; ++rb)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[cur][cb], fa[cur][rb], acc[rb][cb], 0, 0, 0);
    }
  };
  // as in gemm_kloop: the first chunk waits for everything, the loads of C included
  const int nch = K / KC;
#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nch) issue(p);
  if (nch > 0) {  // (every loop below is reached only through the first chunk's full wait)
    wait_vmcnt<0>();
    __syncthreads();
    compute(0, NST - 1 < nch ? NST - 1 : -1);
    int ch = 1;
    for (; ch + NST - 1 < nch; ++ch) {
      wait_vmcnt<imin_c((NST - 2) * W, 63)>();
      __syncthreads();
      compute(ch, ch + NST - 1);
    }
    for (; ch < nch; ++ch) {
      const int later = nch - 1 - ch;
      if (later >= 2) wait_vmcnt<imin_c(2 * W, 63)>();
      else if (later == 1) wait_vmcnt<imin_c(W, 63)>();
      else wait_vmcnt<0>();
      __syncthreads();
      compute(ch, -1);
    }
  }
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < 8; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * 128 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
        if (row < M && col < N) st_dev(C + (int64_t)col * ld + row, acc[rb][cb][i]);
      }
}

// The same with the result added to an FP64 C (Cd, ld ldcd).
__device__ __forceinline__ void gemm_nt_f32_d(double* Cd, int64_t ldcd, const float* Ap, const float* Bp, int64_t ld,
                                              int M, int N, int K, bool lower_only, double* lds) {
  if (K % 32 == 0)
    gemm_f32_core<32, 4, true>(nullptr, Ap, Bp, ld, M, N, K, lower_only, lds, Cd, ldcd);
  else
    gemm_f32_core<16, 4, true>(nullptr, Ap, Bp, ld, M, N, K, lower_only, lds, Cd, ldcd);
}

// ---------------------------------------------------------------------------
// BF16 GEMM item of the BF16-update factorization: C[M x N] (FP32, ld ldc)
// -= A B^T with A (M x K) and B (N x K) each given as three BF16 terms
// (hi + mid + lo, split3), M <= 256, N <= 128, K % 32 == 0.  The six products
// of terms whose orders add up to at most two (hh, hm, mh, mm, hl, lh) run on
// the BF16 matrix cores (v_mfma_f32_16x16x32_bf16) with FP32 accumulation; the
// terms left out are below 2^-24 of the product, so the update keeps FP32
// accuracy.
//
// The panels come in blocks of 1 KB, 16 rows by 32 columns of one term, laid
// out as their LDS image (H_BLOCK: a row's four 16-byte quarters are
// XOR-swizzled by bits 2-3 of the row, so the fragment reads of 16 consecutive
// rows hit distinct banks); a row group's blocks follow each other along a
// column block (nc of them), gs bytes from one row group to the next, hblk
// from one column block to the next and hterm from one term to the next.  A
// transfer is then one contiguous KB at a running scalar pointer, five
// instructions in all: with the rows of a K-contiguous layout (64-byte pieces,
// a 64-bit address per lane) the 18 transfers of a chunk took twice as long to
// issue as its products to run.
// 2 x 2 wavefronts of 128 x 64, chunks of 32 k in two LDS stages; what a chunk
// issues besides its products goes between groups of four of them.  The
// instruction has no operand negation: the accumulators start from -C and -acc
// is stored (C at the end would round less, which changes how many refinement
// steps a solve takes).
// A whole item of K = 1024 with all 256 workgroups busy (n = 32768): 120 -> 88 us
// (the products alone take 41 us; the panels' 2.4 MB then arrive at 6.9 TB/s
// over the chip, mostly from beyond the L2s).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
#define BW_SLOTS_A 1024                               // 16-byte slots per term of A: 256 rows x 4
#define BW_SLOTS_B 512                                // of B: 128 rows x 4
#define BW_STAGE_BYTES (3 * (BW_SLOTS_A + BW_SLOTS_B) * 16)

__device__ __forceinline__ int bw_slot(int row, int q) { return row * 4 + (q ^ ((row >> 2) & 3)); }

__device__ __forceinline__ void gemm_bf16x6_wide(float* __restrict__ C, int64_t ldc, const char* __restrict__ Ha,
                                                 const char* __restrict__ Hb, int64_t gs, int64_t hterm, int64_t hblk,
                                                 int nc, int M, int N, int K, double* lds_d) {
  constexpr int KC = 32;
  static_assert(2 * BW_STAGE_BYTES <= 8 * LDS_DOUBLES, "two stages must fit the workgroup LDS");
  const char* const lds = reinterpret_cast<const char*>(lds_d);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;

  f4 acc[8][4];
  // this wavefront's transfers of a chunk: row groups wave, wave + 4, ... of A
  // (four per term) and of B (two per term); groups past the panel read
  // whatever follows (the workspace reserves it) for outputs never stored
  const uint32_t off = 16u * (uint32_t)lane;
  const uint32_t l0 = lds_addr(lds_d) + 1024u * (uint32_t)wave;
  const uint64_t g4 = 4 * (uint64_t)gs, nta = (uint64_t)hterm - 3 * g4, ntb = (uint64_t)hterm - g4;
  uint64_t qa = (uint64_t)(uintptr_t)uniform_ptr(Ha + wave * gs), qb = (uint64_t)(uintptr_t)uniform_ptr(Hb + wave * gs);
  uint64_t pa = qa, pb = qb;  // running pointers within a chunk
  int cleft = nc;             // chunks left in the column block
  auto next_chunk = [&]() __attribute__((always_inline)) {
    const uint64_t d = --cleft == 0 ? (uint64_t)hblk - 1024u * (uint64_t)(nc - 1) : 1024u;
    if (cleft == 0) cleft = nc;
    pa = qa += d;
    pb = qb += d;
  };
  auto xfer = [&](auto jc, uint32_t st) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if constexpr (j < 12) {
      dma16i<(j / 4) * BW_SLOTS_A * 16 + (j % 4) * 4096>(pa, off, st);
      pa += j % 4 == 3 ? nta : g4;
    } else {
      constexpr int k = j - 12;
      dma16i<(3 * BW_SLOTS_A + (k / 2) * BW_SLOTS_B) * 16 + (k % 2) * 4096>(pb, off, st);
      pb += k % 2 == 1 ? ntb : g4;
    }
  };
  const char* const fa0 = lds + bw_slot(wm * 128 + l16, lg) * 16;
  const char* const fb0 = lds + (3 * BW_SLOTS_A + bw_slot(wn * 64 + l16, lg)) * 16;
  // the products of the chunk in stage so (bytes), with the transfers of the
  // next one into the stage at st
  auto compute = [&](auto issue_c, int so, uint32_t st) __attribute__((always_inline)) {
    constexpr bool ISSUE = decltype(issue_c)::value;
    bf16x8 fb[3][4], fan[2][3];
    auto read_a = [&](int rb, int t) __attribute__((always_inline)) {
      fan[rb & 1][t] = *reinterpret_cast<const bf16x8*>(fa0 + so + (t * BW_SLOTS_A + rb * 64) * 16);
    };
    auto read_b = [&](int t) __attribute__((always_inline)) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        fb[t][cb] = *reinterpret_cast<const bf16x8*>(fb0 + so + (t * BW_SLOTS_B + cb * 64) * 16);
    };
    // in the order of their first use
    read_b(2);
    read_a(0, 0);
    read_b(0);
    read_a(0, 2);
    read_b(1);
    read_a(0, 1);
    __builtin_amdgcn_sched_barrier(0);
    static_for<8>([&](auto rc) __attribute__((always_inline)) {
      constexpr int rb = decltype(rc)::value;
      // term pairs (B term, A term) from the smallest: h l, l h, m m, h m, m h, h h;
      // consecutive instructions go to the four independent accumulators
      // of the row block, so none waits for the previous one's result
      static_for<6>([&](auto pc) __attribute__((always_inline)) {
        constexpr int pr = decltype(pc)::value;
        constexpr int PB[6] = {2, 0, 1, 1, 0, 0}, PA[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[PB[pr]][cb], fan[rb & 1][PA[pr]], acc[rb][cb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (pr < 3) {
          constexpr int T[3] = {0, 2, 1};
          if constexpr (rb + 1 < 8) read_a(rb + 1, T[pr]);
        } else if constexpr (ISSUE && rb < 6) {
          xfer(std::integral_constant<int, 3 * rb + pr - 3>(), st);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  const int nch = K / KC;
  static_for<18>([&](auto jc) __attribute__((always_inline)) { xfer(jc, l0); });
  // C: of a whole tile, one pointer per column of a lane and constant row offsets
  const bool whole = M == 256 && N == 128;
  float* const Cl = C + (int64_t)(wn * 64 + 4 * lg) * ldc + wm * 128 + l16;
  if (whole) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* const q = Cl + (int64_t)(cb * 16 + i) * ldc;
#pragma unroll
        for (int rb = 0; rb < 8; ++rb) acc[rb][cb][i] = -q[rb * 16];
      }
  } else {
#pragma unroll
    for (int rb = 0; rb < 8; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = wm * 128 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
          acc[rb][cb][i] = -C[(int64_t)imin(col, N - 1) * ldc + imin(row, M - 1)];
        }
  }
  wait_vmcnt<0>();
  lds_barrier();
  int so = 0;
  for (int ch = 0; ch + 1 < nch; ++ch) {
    next_chunk();
    compute(std::true_type(), so, l0 + (uint32_t)(BW_STAGE_BYTES - so));
    so = BW_STAGE_BYTES - so;
    wait_vmcnt<0>();
    lds_barrier();
  }
  compute(std::false_type(), so, 0);
  lds_barrier();
  if (whole) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float* const q = Cl + (int64_t)(cb * 16 + i) * ldc;
#pragma unroll
        for (int rb = 0; rb < 8; ++rb) st_dev(q + rb * 16, -acc[rb][cb][i]);
      }
  } else {
#pragma unroll
    for (int rb = 0; rb < 8; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = wm * 128 + rb * 16 + l16, col = wn * 64 + cb * 16 + 4 * lg + i;
          if (row < M && col < N) st_dev(C + (int64_t)col * ldc + row, -acc[rb][cb][i]);
        }
  }
}

// ---------------------------------------------------------------------------
// Panel constants of the diagonal tile's adjoint (panels of PW columns).
#define PW 16
#define PPLD 516                              // LDS leading dimension of the panel
#define P_STAGE_DOUBLES (272 * 8 * 4)         // stages of gemm_core<SEG, 256, 16, 8, 4, 4, 0>

// Factors the 16 x 16 (w x w, rows and columns past w padded with the
// identity) diagonal block at (off, off) of an LDS matrix X (leading
// dimension LDX) on one wavefront: lane r holds row r in registers, the
// pivot and the column entries are broadcast across lanes (readlane), so no
// barrier is needed.  With extra > 0, lanes 16 .. 16 + extra - 1 hold the
// rows off + 16 .. below the block, which the same steps solve against it
// (X := X L_dd^{-T}) at no extra cost.  l = sqrt(d) and 1/l come from the
// hardware reciprocal square root and two Newton steps (y to about an ulp;
// then l = d y with one residual correction), a far shorter dependent chain
// than a correctly rounded square root and division, and exact for powers
// of four; pivots below 2^-900 are scaled by 2^1000 first (exactly), and
// the results back.  No step branches, so the updates of one column overlap
// the next pivot's chain.  Writes L_dd back (and the solved rows below), a
// copy to Ldd[r * LDD + c] (r < 16 + extra) and the reciprocal pivots to
// Linv.  Returns 0, or ibase + the 1-based column of the first pivot that
// is not positive (zero, negative or NaN; the arithmetic goes on and its
// results are discarded).
template <int LDX, int LDD>
__device__ __forceinline__ int diag16_x(double* X, int off, int w, double* Ldd, double* Linv, int lane, int ibase,
                                        int extra = 0) {
  double* As = X;
  const int c0 = off;
  const bool below = lane >= PW && lane < PW + extra;  // a row below the block
  double x[PW];
  const int r = below ? lane : imin(lane, w - 1);
  // every load is issued before any is used (and kept out of the selects below)
  double v[PW];
#pragma unroll
  for (int c = 0; c < PW; ++c) v[c] = As[(c0 + imin(c, w - 1)) * LDX + c0 + r];
  materialize(v);
#pragma unroll
  for (int c = 0; c < PW; ++c)
    x[c] = below ? ((c < w) ? v[c] : 0.0)
                 : ((lane < w) ? (((c <= lane) & (c < w)) ? v[c] : 0.0) : (c == lane ? 1.0 : 0.0));
  int info = 0;
  double pinv[PW];
#pragma unroll
  for (int cc = 0; cc < PW; ++cc) {
    const double d = readlane_f64(x[cc], cc);
    info = (info == 0 && !(d > 0.0)) ? ibase + cc + 1 : info;
    const bool tiny = d < 0x1p-900;
    const double ds = tiny ? d * 0x1p+1000 : d;
    double y = __builtin_amdgcn_rsq(ds);
    y = fma(0.5 * y, fma(-ds, y * y, 1.0), y);
    y = fma(0.5 * y, fma(-ds, y * y, 1.0), y);
    double l = ds * y;
    l = fma(fma(-l, l, ds), 0.5 * y, l);
    l = tiny ? l * 0x1p-500 : l;
    const double inv = tiny ? y * 0x1p+500 : y;
    pinv[cc] = inv;
    // the scaled column is broadcast before the pivot itself is set, which
    // keeps l off the chain to the next pivot; entries above the diagonal
    // (lane < column) are updated too, without a select: they are never
    // read, and the identity padding stays exact
    const double sc = x[cc] * inv;
#pragma unroll
    for (int c2 = cc + 1; c2 < PW; ++c2) {
      const double vv = readlane_f64(sc, c2);
      x[c2] -= sc * vv;
    }
    x[cc] = (lane == cc) ? l : sc;
  }
  if (lane < w) {
#pragma unroll
    for (int c = 0; c < PW; ++c)
      if (c <= lane) As[(c0 + c) * LDX + c0 + lane] = x[c];
  }
  if (below) {
#pragma unroll
    for (int c = 0; c < PW; ++c) {
      As[(c0 + c) * LDX + c0 + lane] = x[c];
      Ldd[lane * LDD + c] = x[c];
    }
  }
  if (lane < PW) {
#pragma unroll
    for (int c = 0; c < PW; ++c) Ldd[lane * LDD + c] = (c <= lane) ? x[c] : 0.0;
    double li = pinv[0];
#pragma unroll
    for (int c = 1; c < PW; ++c) li = (lane == c) ? pinv[c] : li;
    Linv[lane] = li;
  }
  return info;
}

// ---------------------------------------------------------------------------
// Four columns of a 16-column panel at once.  A wavefront holds the panel's
// diagonal block as xd in the layout of an MFMA result (element i of lane l:
// row l % 16, column 4 i + l / 16 of the block; rows and columns past the
// tile's order hold the identity, the strict upper triangle any finite
// values).  Sub-step s broadcasts the 4 x 4 diagonal block of columns
// 4 s .. 4 s + 3 (ten readlanes) and factors it redundantly in every lane,
// with lane l also forming column l / 16 of the block's inverse W.
// The products run on v_mfma_f64_4x4x4_4b: element s of a 16-row block is
// the B operand of four 4 x 4 x 4 blocks (4 rows each) as it stands, and the
// result has the same layout.  One solves four columns of a row block
// (x[s] := x[s] W^T, W in every block of the A operand), and one more per
// later column quad i applies them (x[i] -= x[s] Y_i^T, Y_i the solved rows
// 4 i .. 4 i + 3 of the diagonal block, copied to every block of the A operand
// by row rotations).  Against a 16 x 16 x 4 product per step these take 17
// instead of 64 cycles of the matrix core, give their result after 27 instead
// of 79, and skip the columns that are done.  The chain per four columns is
// four pivots of a reciprocal square root, one third-order step (hardware
// estimate to better than an ulp) and two operations each, plus two products,
// instead of sixteen dependent pivots with a broadcast and a column update.
// The diagonal block's products come first, since the next sub-step waits
// for them; the row blocks' run under the next sub-step's pivots.
// lf: the columns of L_dd (lower triangle), the diagonal from the pivots.
// Returns a mask of the columns (bit 4 S + c) whose pivot is not positive
// (zero, negative or NaN; the arithmetic goes on and its results are
// discarded).
__device__ __forceinline__ double mfma4_f64(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ double mfma4_f64_neg(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 2 /* neg B */);
}

// Lanes 4 Q .. 4 Q + 3 of every row of 16 lanes, copied to the row's other quads.
template <int Q>
__device__ __forceinline__ double quad_to_row(double v) {
  const long long b = __double_as_longlong(v);
  int lo = (int)b, hi = (int)(b >> 32);
  const int lo0 = lo, hi0 = hi;
  lo = __builtin_amdgcn_update_dpp(lo, lo0, 0x120 + 4, 0xf, 1 << ((Q + 1) & 3), false);
  hi = __builtin_amdgcn_update_dpp(hi, hi0, 0x120 + 4, 0xf, 1 << ((Q + 1) & 3), false);
  lo = __builtin_amdgcn_update_dpp(lo, lo0, 0x120 + 8, 0xf, 1 << ((Q + 2) & 3), false);
  hi = __builtin_amdgcn_update_dpp(hi, hi0, 0x120 + 8, 0xf, 1 << ((Q + 2) & 3), false);
  lo = __builtin_amdgcn_update_dpp(lo, lo0, 0x120 + 12, 0xf, 1 << ((Q + 3) & 3), false);
  hi = __builtin_amdgcn_update_dpp(hi, hi0, 0x120 + 12, 0xf, 1 << ((Q + 3) & 3), false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

struct Quad {
  double fw;    // the solve operand
  double d[4];  // the pivots
};

template <int S>
__device__ __forceinline__ unsigned quad_factor(double xs, const double (&e)[4], int l16, Quad& q) {
  double a[10], l[10];
  {
    int n = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) a[n++] = readlane_f64(xs, 16 * j + 4 * S + i);
  }
  auto ix = [](int i, int j) __attribute__((always_inline)) { return i * (i + 1) / 2 + j; };
  unsigned bad = 0;
  double w[4];
  q.fw = 0.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double d = a[ix(c, c)];
#pragma unroll
    for (int t = 0; t < c; ++t) d = fma(-l[ix(c, t)], l[ix(c, t)], d);
    bad |= ((unsigned)__builtin_amdgcn_ballot_w64(!(d > 0.0)) & 1u) << (4 * S + c);
    const double y0 = __builtin_amdgcn_rsq(d);
    const double er = fma(-(d * y0), y0, 1.0);
    const double y = fma(y0 * er, fma(0.375, er, 0.5), y0);
    q.d[c] = d;
#pragma unroll
    for (int i = c + 1; i < 4; ++i) {
      double v = a[ix(i, c)];
#pragma unroll
      for (int t = 0; t < c; ++t) v = fma(-l[ix(i, t)], l[ix(c, t)], v);
      l[ix(i, c)] = v * y;
    }
    // row c of this lane's column of the inverse
    double t = e[c];
#pragma unroll
    for (int u = 0; u < c; ++u) t = fma(-l[ix(c, u)], w[u], t);
    w[c] = t * y;
    q.fw = ((l16 & 3) == c) ? w[c] : q.fw;
  }
  return bad;
}

// The operands of a panel's sub-steps in LDS, 64 doubles each: the four solve
// operands, then those of the updates of quad i after sub-step s < i.
#define QUAD_OPS 10
__device__ __forceinline__ constexpr int quad_op(int s, int i) { return s == i ? s : 4 + (s == 0 ? i - 1 : s == 1 ? i + 1 : 5); }

// One sub-step on the diagonal block xd (L's columns below the diagonal to lf)
// and one row block x of the panel.  e[c] = (l / 16 == c).  Its operands also go
// to Fb; the lanes that hold L's diagonal take the pivot to dv and its
// reciprocal square root, the diagonal of the solve operand, to yv.
// Returns as quad_factor.
template <int S>
__device__ __forceinline__ unsigned panel_quad(d4& xd, d4& lf, d4& x, const double (&e)[4], int lane, double* Fb,
                                               double& dv, double& yv) {
  const int l16 = lane & 15;
  Quad q;
  const unsigned bad = quad_factor<S>(xd[S], e, l16, q);
  const double zd = mfma4_f64(q.fw, xd[S], 0.0);
  double yq[4];  // yq[i]: the solved rows of quad i of the diagonal block
  if constexpr (S < 3) {
    yq[S + 1] = quad_to_row<S + 1>(zd);
    xd[S + 1] = mfma4_f64_neg(yq[S + 1], zd, xd[S + 1]);
  }
  __builtin_amdgcn_sched_barrier(0);
  const double z = mfma4_f64(q.fw, x[S], 0.0);
  if constexpr (S < 2) {
    yq[S + 2] = quad_to_row<S + 2>(zd);
    xd[S + 2] = mfma4_f64_neg(yq[S + 2], zd, xd[S + 2]);
  }
  if constexpr (S < 1) {
    yq[S + 3] = quad_to_row<S + 3>(zd);
    xd[S + 3] = mfma4_f64_neg(yq[S + 3], zd, xd[S + 3]);
  }
  xd[S] = zd;
#pragma unroll
  for (int c = 0; c < 4; ++c) dv = (lane == 16 * c + 4 * S + c) ? q.d[c] : dv;
  yv = (l16 >> 2) == S ? q.fw : yv;
  lf[S] = zd;
  x[S] = z;
#pragma unroll
  for (int i = S + 1; i < 4; ++i) {
    x[i] = mfma4_f64_neg(yq[i], z, x[i]);
    Fb[quad_op(S, i) * 64 + lane] = yq[i];
  }
  Fb[quad_op(S, S) * 64 + lane] = q.fw;
  return bad;
}

// The 16 columns: panel_quad four times.  With x the identity on entry, x is
// L_dd^{-T} on return.  Returns 0, or ibase + the 1-based column of the first
// pivot that is not positive.
__device__ __forceinline__ int panel16(d4& xd, d4& lf, d4& x, const double (&e)[4], int lane, int ibase,
                                       double* Fb) {
  double dv = 1.0, yv = 1.0;
  unsigned bad = panel_quad<0>(xd, lf, x, e, lane, Fb, dv, yv);
  bad |= panel_quad<1>(xd, lf, x, e, lane, Fb, dv, yv);
  bad |= panel_quad<2>(xd, lf, x, e, lane, Fb, dv, yv);
  bad |= panel_quad<3>(xd, lf, x, e, lane, Fb, dv, yv);
  // L's diagonal, all sixteen at once (each on the lane that holds it): d times
  // its reciprocal root, with one correction of the residual d - l^2, which for
  // a pivot near the smallest numbers is taken at 2^1000 times its size
  const bool tiny = dv < 0x1p-900;
  const double ds = tiny ? dv * 0x1p+1000 : dv, ys = tiny ? yv * 0x1p-500 : yv;
  double l = ds * ys;
  l = fma(fma(-l, l, ds), 0.5 * ys, l);
  l = tiny ? l * 0x1p-500 : l;
  const int l16 = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int s = 0; s < 4; ++s) lf[s] = l16 == 4 * s + lg ? l : lf[s];
  return bad ? ibase + __builtin_ctz(bad) + 1 : 0;
}

// Row blocks of the panel solved with the operands that panel16 left in Fb.
template <int NX>
__device__ __forceinline__ void panel16_rows(d4 (&x)[NX], const double* Fb, int lane) {
  double f[QUAD_OPS];
#pragma unroll
  for (int k = 0; k < QUAD_OPS; ++k) f[k] = Fb[k * 64 + lane];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int h = 0; h < NX; ++h) x[h][s] = mfma4_f64(f[quad_op(s, s)], x[h][s], 0.0);
#pragma unroll
    for (int i = s + 1; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < NX; ++h) x[h][i] = mfma4_f64_neg(f[quad_op(s, i)], x[h][s], x[h][i]);
  }
}

// ---------------------------------------------------------------------------
// POTRF of a tile of order m <= 128 on one workgroup, the tile in LDS for the
// whole factorization: right-looking by 16-column panels, every product on
// the matrix cores.  FP64 vector and matrix instructions of a wavefront do
// not overlap, so the chain of diagonal blocks has a wavefront of its own:
//   wavefront 0     factors the diagonal block of panel j, with its inverse
//                   (panel16), while
//   wavefronts 1-3  apply panel j - 1 to the later columns;
//   barrier         (the sub-steps' operands are in LDS)
//   all             solve the panel's row blocks; wavefront 0 takes the block
//                   below the diagonal and applies it to the next diagonal
//                   block;
//   barrier         (the panel is in LDS).
//
// With IV set, the tile's inverse comes along.  The rows of the identity, solved and
// updated like rows below the tile, become L^{-T}; row block r of it enters
// with panel r, where row block r of the tile itself has just become the
// diagonal block.  Its blocks (r, c), c > r, thus take the place of the tile's
// unused upper blocks, (r, r) that of the diagonal block.  L^{-1} goes to IV
// (ldi), zeros above its diagonal included; rows and columns from m to the
// next multiple of 16 are the identity's.
//
// Bound by the chain: per panel about 2800 cycles of panel16 (vector
// instructions issue every 5 to 8 cycles for one wavefront) and 1400 of the
// two products, two barriers and their LDS round trips.  A tile of 128 in a
// factorization of order 1024: 62.7 us, and 31 more for the inverse by TRTRI
// strips, became 31-33 us with the inverse.
// Returns 0, or the 1-based column (within the tile) whose pivot is not
// positive (the columns before its panel's are then stored).
#define SLD 144   // LDS leading dimension of the resident tile (fragment rows 128 bytes apart modulo 256: no conflicts)


__device__ __forceinline__ int potrf_small(double* __restrict__ Akk, int64_t ld, int m, double* lds,
                                           double* __restrict__ IV = nullptr, int64_t ldi = 0) {
  static_assert(128 * SLD + (QUAD_OPS + 4) * 64 <= LDS_DOUBLES, "the tile must fit the workgroup LDS");
  double* As = lds;             // [128][SLD]
  double* Fb = As + 128 * SLD;      // [QUAD_OPS][64] the panel's operands
  double* Lb = Fb + QUAD_OPS * 64;  // [4][64] L_dd as wavefront 0 holds it
  __shared__ int s_sinfo;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int nblk = (m + 15) >> 4;
  const bool inv = IV != nullptr;
  // element i of the 16 x 16 block (rb, cb) in the MFMA result layout, which
  // is also the operand layout of its k-step i
  auto at = [&](int rb, int cb, int i) __attribute__((always_inline)) -> double& {
    return As[(cb * 16 + 4 * i + lg) * SLD + rb * 16 + l16];
  };
  // this lane's element of a block, in the tile and (transposed) in the inverse;
  // a block's own offset is wave-uniform
  double* const Al = Akk + (int64_t)lg * ld + l16;
  double* const Il = inv ? IV + (int64_t)l16 * ldi + lg : nullptr;
  // the lower blocks into LDS, a wavefront's (every fourth, by columns) all in flight at once
  {
    double v[9][4];
    int rb = wave, cb = 0;
    auto settle = [&]() __attribute__((always_inline)) {
      while (rb >= nblk && cb < nblk) {
        ++cb;
        rb = rb - nblk + cb;
      }
    };
    settle();
    const int rb0 = rb, cb0 = cb;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      if (cb < nblk) {
        if (rb * 16 + 16 <= m) {
          const double* const p = Al + (int64_t)cb * 16 * ld + rb * 16;
          // lanes above the diagonal read the diagonal's row instead
#pragma unroll
          for (int i = 0; i < 4; ++i) v[t][i] = p[(int64_t)(4 * i) * ld + (rb == cb ? imax(4 * i + lg - l16, 0) : 0)];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int c = cb * 16 + 4 * i + lg, r = rb * 16 + l16;
            v[t][i] = Akk[(int64_t)imin(c, m - 1) * ld + imin(imax(r, c), m - 1)];
          }
        }
        rb += 4;
        settle();
      }
    }
    rb = rb0;
    cb = cb0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      if (cb < nblk) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = rb * 16 + l16, c = cb * 16 + 4 * i + lg;
          at(rb, cb, i) = (r < m && c < m && r >= c) ? v[t][i] : (r == c ? 1.0 : 0.0);
        }
        rb += 4;
        settle();
      }
    }
  }
  lds_barrier();
  // row block rb of the solved panel j: to LDS, and to the tile or the inverse
  auto put = [&](int rb, int j, const d4& x) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) at(rb, j, i) = x[i];
    if (rb > j) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (rb * 16 + l16 < m) st_dev(Al + (int64_t)(j * 16 + 4 * i) * ld + rb * 16, x[i]);
    } else if (inv) {
#pragma unroll
      for (int i = 0; i < 4; ++i) st_dev(Il + (int64_t)(rb * 16) * ldi + j * 16 + 4 * i, x[i]);
    }
  };
  // Panel j - 1 on column cb = j + q: blocks (rb, cb) of the tile (rb >= cb; the
  // next diagonal block is wavefront 0's) and of the inverse (rb < j).  Three
  // register sets take turns, so that a block's operands are requested before,
  // and its result is written back after, the products of the block in between.
  // Columns q = 0 .. 6 hold 7, 7, 6, 5, 4, 3, 2 blocks (inv): 0 and 6 go to
  // wavefront 1, 1 and 5 to 2, 2 and 4 to 3, and 3 to wavefront 0 after its
  // diagonal block.
  auto trail = [&](int j, int q) __attribute__((always_inline)) {
    struct Set {
      int r;  // row block, past the last: none
      double g[4];
      d4 c;
    };
    const int cb = j + q;
    if (cb >= nblk) return;
    const int r1 = q == 0 ? cb + 1 : cb;  // first row block of the tile
    int rb = inv ? 0 : r1;
    double f[4];
    Set sa, sb, sc;
    const double* const Xp = &at(0, j - 1, 0);
    double* const Cp = &at(0, cb, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = Xp[cb * 16 + 4 * k * SLD];
    auto fetch = [&](Set& u) __attribute__((always_inline)) {
      // (past the last block: that block again, unused, so that every turn
      // issues the same reads and a wait for one set leaves the next in flight)
      u.r = rb;
      const int r = imin(rb, nblk - 1) * 16;
      rb = inv && rb + 1 == j ? r1 : rb + 1;
#pragma unroll
      for (int k = 0; k < 4; ++k) u.g[k] = Xp[r + 4 * k * SLD];
#pragma unroll
      for (int i = 0; i < 4; ++i) u.c[i] = Cp[r + 4 * i * SLD];
    };
    auto multiply = [&](Set& u) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) u.c = __builtin_amdgcn_mfma_f64_16x16x4f64(f[k], u.g[k], u.c, 0, 0, 2 /* neg B */);
    };
    auto back = [&](Set& u) __attribute__((always_inline)) {
      if (u.r >= nblk) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) Cp[u.r * 16 + 4 * i * SLD] = u.c[i];
    };
    fetch(sa);
    sb.r = sc.r = nblk;
    auto turn = [&](Set& cur, Set& nxt) __attribute__((always_inline)) {
      back(nxt);
      fetch(nxt);
      __builtin_amdgcn_sched_barrier(0);
      multiply(cur);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll 1
    while (sa.r < nblk) {
      turn(sa, sb);
      if (sb.r >= nblk) break;
      turn(sb, sc);
      if (sc.r >= nblk) break;
      turn(sc, sa);
    }
    back(sa);
    back(sb);
    back(sc);
  };
  if (wave == 0) {
    double e[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) e[c] = (lg == c) ? 1.0 : 0.0;
    d4 xd;
#pragma unroll
    for (int i = 0; i < 4; ++i) xd[i] = at(0, 0, i);
#pragma unroll 1
    for (int j = 0; j < nblk; ++j) {
      d4 lf, x;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (4 * i + lg == l16) ? 1.0 : 0.0;
      const int info = __builtin_amdgcn_readfirstlane(panel16(xd, lf, x, e, lane, 16 * j, Fb));
      if (lane == 0) s_sinfo = info;
      if (j > 0) trail(j, 3);
      lds_barrier();
      if (info != 0) return info;
      if (j + 1 < nblk) {
        d4 xb[1];
        d4& xr = xb[0];
#pragma unroll
        for (int k = 0; k < 4; ++k) xr[k] = at(j + 1, j, k);
#pragma unroll
        for (int i = 0; i < 4; ++i) xd[i] = at(j + 1, j + 1, i);
        panel16_rows(xb, Fb, lane);
#pragma unroll
        for (int k = 0; k < 4; ++k) xd = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[k], xr[k], xd, 0, 0, 2 /* neg B */);
#pragma unroll
        for (int i = 0; i < 4; ++i) at(j + 1, j, i) = xr[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        Lb[i * 64 + lane] = lf[i];
        at(j, j, i) = x[i];
      }
      lds_barrier();
    }
    return 0;
  }
  // the blocks of panel j that wavefront 0 left in LDS: L_dd and its inverse
  // (wavefront 3), the block below (wavefront 2)
  auto put_chain = [&](int j) __attribute__((always_inline)) {
    if (wave == 3) {
      d4 lf, x;
#pragma unroll
      for (int i = 0; i < 4; ++i) lf[i] = Lb[i * 64 + lane];
      if (inv) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = at(j, j, i);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = j * 16 + l16, c = j * 16 + 4 * i + lg;
        if (r >= c && r < m) st_dev(Al + (int64_t)(j * 16 + 4 * i) * ld + j * 16, lf[i]);
      }
      if (inv) {
#pragma unroll
        for (int i = 0; i < 4; ++i) st_dev(Il + (int64_t)(j * 16) * ldi + j * 16 + 4 * i, x[i]);
      }
    } else if (wave == 2 && j + 1 < nblk) {
      d4 x;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = at(j + 1, j, i);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((j + 1) * 16 + l16 < m) st_dev(Al + (int64_t)(j * 16 + 4 * i) * ld + (j + 1) * 16, x[i]);
    }
  };
#pragma unroll 1
  for (int j = 0; j < nblk; ++j) {
    if (j > 0) {
      trail(j, wave - 1);
      trail(j, 7 - wave);
      put_chain(j - 1);
    } else if (inv) {
      // while the first diagonal block is factored: the zeros of the tile's
      // upper blocks and of the inverse
#pragma unroll 1
      for (int zc = 1; zc < nblk; ++zc)
#pragma unroll 1
        for (int zr = wave - 1; zr < zc; zr += 3) {
          double* const z = IV + ((int64_t)zc * 16 + lg) * ldi + zr * 16 + l16;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            at(zr, zc, i) = 0.0;
            st_dev(z + (int64_t)(4 * i) * ldi, 0.0);
          }
        }
    }
    lds_barrier();
    const int info = __builtin_amdgcn_readfirstlane(s_sinfo);
    if (info != 0) return info;
    // the panel's other row blocks: the tile's below j + 1, the inverse's above j
    {
      // at most three to a wavefront; absent ones are the last again, unused
      auto block = [&](int p) __attribute__((always_inline)) { return inv ? (p < j ? p : p + 2) : j + 2 + p; };
      d4 x[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const int rb = imin(block(wave - 1 + 3 * t), nblk - 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[t][k] = at(rb, j, k);
      }
      panel16_rows(x, Fb, lane);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const int rb = block(wave - 1 + 3 * t);
        if (rb < nblk) put(rb, j, x[t]);
      }
    }
    lds_barrier();
  }
  put_chain(nblk - 1);
  return 0;
}

// ---------------------------------------------------------------------------
// The same by columns (diag16_x, one pivot at a time; rows below by
// substitution, one per thread; products from C on): 62.7 us for a tile of 128
// where potrf_small takes 31.  It serves the BF16-update factorization alone,
// whose results depend on the order of rounding: a rounding of 1e-16 that differs
// in a diagonal tile flips some of the roundings of panel values to 24 bits, the
// flips spread through the trailing updates, and a solution moves with them, by
// 1e-12 at order 4000, 1e-10 at 16000 and up to 1.1e-9 at 32768 (condition
// 1e4, where the refinement leaves it 1e-8 from the exact one).  This order of
// rounding keeps the solutions that the factorization has always had.  The whole
// solve this way / with potrf_small: order 4000 8.4 / 7.0 ms, 8192 15.9 / 12.9,
// 16000 32.3 / 27.2, 32768 118.8 / 114.4.
// Block (bi, bj) of the resident tile -= P(bi) P(bj)^T, P the 16 columns of
// the panel at c0.  A operand: P(bi) (rows on lanes % 16), B operand: P(bj)^T;
// element v of lane l is then row 4v + l/16, column l%16 of the block.
__device__ __forceinline__ void upd16_lds(double* As, int c0, int bi, int bj, int lane) {
  const int l16 = lane & 15, lg = lane >> 4;
  d4 acc;
#pragma unroll
  for (int v = 0; v < 4; ++v) acc[v] = As[(bj * 16 + l16) * SLD + bi * 16 + 4 * v + lg];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const double fa = As[(c0 + 4 * s + lg) * SLD + bi * 16 + l16];
    const double fb = As[(c0 + 4 * s + lg) * SLD + bj * 16 + l16];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa, fb, acc, 0, 0, 2 /* neg B */);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) As[(bj * 16 + l16) * SLD + bi * 16 + 4 * v + lg] = acc[v];
}

__device__ __forceinline__ int potrf_columns(double* __restrict__ Akk, int64_t ld, int m, double* lds) {
  double* As = lds;                      // [128][SLD]
  double* Ldd = As + 128 * SLD;          // [PW][PW + 1]
  double* Linv = Ldd + PW * (PW + 1);    // [PW]
  int& s_sinfo = *reinterpret_cast<int*>(Linv + PW);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nblk = (m + 15) >> 4;
  // the lower triangle into LDS, 16 loads in flight per thread; rows and
  // columns past m hold the identity
  {
    constexpr int PER = 128 * 128 / NT, BATCH = 16;
#pragma unroll 1
    for (int u0 = 0; u0 < PER; u0 += BATCH) {
      double v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int idx = tid + (u0 + u) * NT, c = idx >> 7, r = idx & 127;
        v[u] = Akk[(int64_t)imin(c, m - 1) * ld + imin(imax(r, c), m - 1)];
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int idx = tid + (u0 + u) * NT, c = idx >> 7, r = idx & 127;
        if (c < nblk * 16 && r < nblk * 16) As[c * SLD + r] = (r < m && c < m && r >= c) ? v[u] : (r == c ? 1.0 : 0.0);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    const int info = diag16_x<SLD, PW + 1>(As, 0, imin(16, m), Ldd, Linv, lane, 0);
    if (lane == 0) s_sinfo = info;
  }
  __syncthreads();
  for (int j = 0; j < nblk; ++j) {
    const int c0 = j * 16;
    const int info = __builtin_amdgcn_readfirstlane(s_sinfo);
    if (info != 0) return info;
    // rows below the diagonal block: y := y L_dd^{-T}, one row per thread
#pragma unroll 1
    for (int r = c0 + 16 + tid; r < nblk * 16; r += NT) {
      double y[PW];
#pragma unroll
      for (int c = 0; c < PW; ++c) y[c] = As[(c0 + c) * SLD + r];
#pragma unroll
      for (int c = 0; c < PW; ++c) {
        y[c] *= Linv[c];
#pragma unroll
        for (int c2 = c + 1; c2 < PW; ++c2) y[c2] -= y[c] * Ldd[c2 * (PW + 1) + c];
      }
#pragma unroll
      for (int c = 0; c < PW; ++c) As[(c0 + c) * SLD + r] = y[c];
    }
    __syncthreads();
    if (j + 1 >= nblk) break;
    // the panel's update of the trailing lower blocks; wavefront 0 first
    // updates and factors the next diagonal block (the critical path)
    const int nb2 = nblk - j - 1;
    const int npair = nb2 * (nb2 + 1) / 2;
    if (wave == 0) {
      upd16_lds(As, c0, j + 1, j + 1, lane);
      const int info2 = diag16_x<SLD, PW + 1>(As, c0 + 16, imin(16, m - c0 - 16), Ldd, Linv, lane, c0 + 16);
      if (lane == 0) s_sinfo = info2;
    }
    // block pairs p >= 1 in column-major order of (bi >= bj), after (j+1, j+1),
    // on the other three wavefronts (wavefront 0 is busy with the diagonal)
#pragma unroll 1
    for (int p = (wave == 0 ? npair : wave); p < npair; p += 3) {
      int cj = 0, rem = p;
      while (rem >= nb2 - cj) {
        rem -= nb2 - cj;
        ++cj;
      }
      const int bj = j + 1 + cj;
      upd16_lds(As, c0, bj + rem, bj, lane);
    }
    __syncthreads();
  }
  // the factor to the tile, lower triangle only
  for (int idx = tid; idx < m * 128; idx += NT) {
    const int c = idx >> 7, r = idx & 127;
    if (r < m && r >= c) st_dev(Akk + (int64_t)c * ld + r, As[c * SLD + r]);
  }
  return 0;
}

// ---------------------------------------------------------------------------
// POTRF work item for a tile of order m <= 512 on one workgroup:
// Akk := chol(Akk), lower, in place.  Left-looking by panels of PT_W = 32
// columns, each taken in slabs of up to PT_SLAB = 256 rows that stay in LDS
// from their update to their store:
//  1. the matrix cores apply every earlier column to the slab (256 x 32
//     outputs per K step, the result written to LDS);
//  2. in the first slab, wavefront 0 factors the 32 x 32 diagonal block: its
//     leading 16 x 16 block in registers (diag16_x, which also solves the 16
//     rows below it), their product subtracted from the trailing 16 x 16
//     block on the matrix cores, then that block factored;
//  3. every thread solves one row of the slab below the block against L_dd;
//  4. the slab goes to the tile (write-through stores), where the next
//     panel's update reads it.
// Panels of 32 columns halve the number of panels and the re-reads of the
// factored columns relative to the 16 of the diagonal blocks, and give the
// updates enough outputs per K step to keep the matrix cores busy.
// Returns 0, or the 1-based column (within the tile) whose pivot is not
// positive (zero, negative or NaN).
#define PT_W 32
#define PT_SLAB 256
#define PT_LT 36                               // stride of the columns of L_dd

template <int SEG>
__device__ __forceinline__ int potrf_tile(double* __restrict__ Akk, int64_t ld, int m, double* lds) {
  constexpr int LDP = PT_SLAB + 8;                     // LDS leading dimension of a slab
  constexpr int STAGE = 2 * 16 * (PT_SLAB + PT_W);     // stages of gemm_core<SEG, PT_SLAB, 32, 16, 4, 2, 0>
  static_assert(STAGE + PT_W * LDP + PT_W * (PT_W + 1) + PT_W + PT_W * PT_LT <= LDS_DOUBLES, "LDS budget");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* Ps = lds + STAGE;                 // [PT_W][LDP] the slab
  double* Ldd = Ps + PT_W * LDP;            // [PT_W][PT_W + 1] the diagonal block (lower)
  double* Linv = Ldd + PT_W * (PT_W + 1);   // [PT_W] reciprocal pivots
  double* LT = Linv + PT_W;                 // L_dd by columns: column c at LT[c * PT_LT + c2]
  __shared__ int s_info;
  for (int c0 = 0; c0 < m; c0 += PT_W) {
    const int w = imin(PT_W, m - c0);
    const int R = m - c0;
    double* P = Akk + (int64_t)c0 * ld + c0;
    for (int s0 = 0; s0 < R; s0 += PT_SLAB) {
      const int S = imin(PT_SLAB, R - s0);
      if (c0 > 0) {
        // the slab - L[c0 + s0 :, 0 : c0] L[c0 : c0 + w, 0 : c0]^T into LDS,
        // on a product no taller than the slab needs
        if (S > 128)
          gemm_core<SEG, PT_SLAB, PT_W, 16, 4, 2, 0>(P + s0, Akk + c0 + s0, Akk + c0, ld, S, w, c0, lds, Ps, LDP);
        else if (S > 64)
          gemm_core<SEG, 128, PT_W, 16, 4, 2, 0>(P + s0, Akk + c0 + s0, Akk + c0, ld, S, w, c0, lds, Ps, LDP);
        else
          gemm_core<SEG, 64, PT_W, 16, 4, 2, 0>(P + s0, Akk + c0 + s0, Akk + c0, ld, S, w, c0, lds, Ps, LDP);
      } else if (tid < S) {
        double v[PT_W];
#pragma unroll
        for (int c = 0; c < PT_W; ++c)
          v[c] = P[(int64_t)imin(c, w - 1) * ld + s0 + tid];
#pragma unroll
        for (int c = 0; c < PT_W; ++c) Ps[c * LDP + tid] = v[c];
      }
      __syncthreads();
      if (s0 == 0) {
        if (wave == 0) {
          // the leading 16 x 16 block, the rows 16 .. w-1 below it solved in the same steps
          int info = diag16_x<LDP, PT_W + 1>(Ps, 0, imin(16, w), Ldd, Linv, lane, c0, imax(w - 16, 0));
          if (w > 16) {
            const int wb = w - 16;
            // trailing block -= (those rows)(those rows)^T: element v of lane
            // l is row 16 + 4v + l/16, column 16 + l%16 (rows and columns past
            // w only meet each other and are never read)
            {
              const int l16 = lane & 15, lg = lane >> 4;
              d4 acc;
#pragma unroll
              for (int v = 0; v < 4; ++v) acc[v] = Ps[(16 + l16) * LDP + 16 + 4 * v + lg];
#pragma unroll
              for (int s = 0; s < 4; ++s) {
                const double f = Ps[(4 * s + lg) * LDP + 16 + l16];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f, f, acc, 0, 0, 2 /* neg B */);
              }
#pragma unroll
              for (int v = 0; v < 4; ++v) Ps[(16 + l16) * LDP + 16 + 4 * v + lg] = acc[v];
            }
            const int info_b =
                diag16_x<LDP, PT_W + 1>(Ps, 16, wb, Ldd + 16 * (PT_W + 1) + 16, Linv + 16, lane, c0 + 16);
            info = info != 0 ? info : info_b;
          }
          if (lane == 0) s_info = info;
        }
        __syncthreads();
        const int info = __builtin_amdgcn_readfirstlane(s_info);
        if (info != 0) return info;
        // L_dd by columns for the rows below: column c at LT[c * PT_LT + c2]
        // (c2 > c), the reciprocal pivot at c2 = c
        for (int idx = tid; idx < PT_W * PT_W; idx += NT) {
          const int c = idx / PT_W, c2 = idx - c * PT_W;
          LT[c * PT_LT + c2] = c2 == c ? Linv[c] : (c2 > c ? Ldd[c2 * (PT_W + 1) + c] : 0.0);
        }
        __syncthreads();
      }
      // rows below the diagonal block: y := y L_dd^{-T}, one row per thread
      // (there are such rows only when the panel is 32 wide); each column's
      // entries of L_dd are loaded together before they are used
      {
        const int r = (s0 == 0 ? w : 0) + tid;
        if (r < S) {
          double y[PT_W];
#pragma unroll
          for (int c = 0; c < PT_W; ++c) y[c] = Ps[c * LDP + r];
#pragma unroll
          for (int c = 0; c < PT_W; ++c) {
            double l[PT_W];
#pragma unroll
            for (int c2 = c; c2 < PT_W; ++c2) l[c2] = LT[c * PT_LT + c2];
#pragma unroll
            for (int c2 = c; c2 < PT_W; ++c2) asm volatile("" : : "v"(l[c2]));
            y[c] *= l[c];
#pragma unroll
            for (int c2 = c + 1; c2 < PT_W; ++c2) y[c2] -= y[c] * l[c2];
          }
#pragma unroll
          for (int c = 0; c < PT_W; ++c) Ps[c * LDP + r] = y[c];
        }
      }
      __syncthreads();
      // the slab (lower part) to the tile, one row per thread; the next slab
      // reuses the LDS
      if (tid < S) {
#pragma unroll
        for (int c = 0; c < PT_W; ++c)
          if (c < w && s0 + tid >= c) st_dev(P + (int64_t)c * ld + s0 + tid, Ps[c * LDP + tid]);
      }
      __syncthreads();
    }
    // the panel must be visible to every wavefront before the next panel's
    // update reads it
    wait_vmcnt<0>();
    __syncthreads();
  }
  return 0;
}

// ---------------------------------------------------------------------------
// POTRF of a tile of order m on one workgroup of the compact instance (two per
// compute unit: 256 registers, half the LDS).  Left-looking by panels of
// PT_W = 32 columns in slabs of 128 rows that stay in registers from their
// update to their store; wavefront w holds rows 32 w .. of the slab as 2 x 2
// blocks of 16 x 16:
//  1. the matrix cores apply every earlier column (panels streamed through two
//     LDS stages of 16 columns as in gemm_tile);
//  2. in the first slab, wavefront 0, which holds the 32 x 32 diagonal block,
//     factors it in registers (panel16 on either half, the sub-steps' operands
//     to LDS);
//  3. every wavefront solves its rows below the block with those operands, on
//     the matrix cores, and stores them from registers.
// Slabs in LDS with one thread per row solving and storing (which this
// replaces) spent as long outside the update as in it.  4096 systems of orders
// 16 .. 512 in FP64, 4 right-hand sides: kernel 4.75 -> 3.28 ms, mean POTRF 473
// -> 295 us.  What is left is mostly the update, whose panels are re-read from
// beyond the L2s (680 of 914 us at an order near 500 when the kernel took 3.81
// ms; 120 in the diagonal blocks, 81 in the rows below).  Bound by registers
// too: two workgroups per compute unit leave 256, and 85 (143 with FP32
// storage) are spilled; keeping the four pivots' reciprocal roots of a quad
// alive as well spilled 145 (211) and cost 0.5 ms (1.0).  Three stages instead
// of two were slower (4.12 against 3.81 ms), as was swapping the halves of odd
// k-rows for them.
// With Bf the forward solve L y = b of nrhs <= 4 right-hand sides
// (column-major at Bf, leading dimension ldbf) rides along: a panel's rows of
// b, transposed, are one more row block for step 3 (wavefront 0), and the rows
// below take b -= L(row, panel) y_panel by products of the blocks they hold.
// Bf then holds y.
// IN32: the tile's values are read from the FP32 matrix A32 (leading
// dimension ld32) instead of Akk, and L is written to both (Akk in FP64 for the
// later panels' products, A32 rounded to FP32).
// Needs an even ld, a 16-byte aligned tile and, for odd m, a readable row after
// the last.  Returns 0, or the 1-based column (within the tile) whose pivot is
// not positive (zero, negative or NaN).
#define PT_FWD 4                               // right-hand sides of the fused forward solve
#define PT_ALD 144                             // LDS stride of a staged k-row of the slab's panel
#define PT_STAGE (16 * PT_ALD + 16 * PT_W)     // doubles of a stage
#define PT_NST 2
#define PT_LDS_COMPACT (PT_NST * PT_STAGE + 2 * QUAD_OPS * 64 + 4 * 64 + 8 * 64)
#define FRB_COMPACT_DOUBLES (32 * 4 * 64 + 2 * 4 * 64)  // tile_solve<true>

template <bool IN32>
__device__ __forceinline__ int potrf_slabs(double* __restrict__ Akk, int64_t ld, int m, double* lds,
                                           double* Bf, int64_t ldbf, int nrhs, float* __restrict__ A32, int64_t ld32) {
  double* const Fb = lds + PT_NST * PT_STAGE;       // [2][QUAD_OPS][64] the halves' operands
  double* const Xb = Fb + 2 * QUAD_OPS * 64;   // [4][64] the block below the first half's
  double* const Yb = Xb + 4 * 64;              // [8][64] the panel's rows of y, as operands
  __shared__ int s_pinfo;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const bool fwd = Bf != nullptr;
  double e[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) e[c] = (lg == c) ? 1.0 : 0.0;
  const uint32_t l0 = lds_addr(lds);
  const double* const fa0 = lds + lg * PT_ALD + wave * 32 + l16;
  const double* const fb0 = lds + 16 * PT_ALD + lg * PT_W + l16;
#pragma unroll 1
  for (int c0 = 0; c0 < m; c0 += PT_W) {
    const int w = imin(PT_W, m - c0), R = m - c0;
    double* const P = Akk + (int64_t)c0 * ld + c0;
    float* const P32 = IN32 ? A32 + (int64_t)c0 * ld32 + c0 : nullptr;
#pragma unroll 1
    for (int s0 = 0; s0 < R; s0 += 128) {
      const int S = imin(128, R - s0);
      const int rw = wave * 32;
      const bool mine = rw < S;  // this wavefront has rows
      d4 acc[2][2];
      {
        const int ra = imin(rw + l16, S - 1), rz = imin(rw + 16 + l16, S - 1) - ra;
        if (w == PT_W) {
          const double* const q = P + (int64_t)lg * ld + s0 + ra;
          const float* const q32 = IN32 ? P32 + (int64_t)lg * ld32 + s0 + ra : nullptr;
#pragma unroll
          for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              acc[0][cb][i] = IN32 ? (double)q32[(int64_t)(cb * 16 + 4 * i) * ld32] : q[(int64_t)(cb * 16 + 4 * i) * ld];
              acc[1][cb][i] =
                  IN32 ? (double)q32[(int64_t)(cb * 16 + 4 * i) * ld32 + rz] : q[(int64_t)(cb * 16 + 4 * i) * ld + rz];
            }
        } else {
#pragma unroll
          for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int64_t col = imin(cb * 16 + 4 * i + lg, w - 1);
              acc[0][cb][i] = IN32 ? (double)P32[col * ld32 + s0 + ra] : P[col * ld + s0 + ra];
              acc[1][cb][i] = IN32 ? (double)P32[col * ld32 + s0 + ra + rz] : P[col * ld + s0 + ra + rz];
            }
        }
      }
      if (c0 > 0) {
        // rows c0 + s0 .. and c0 .. of the earlier columns
        const uint32_t offa = (uint32_t)(imin(2 * lane, (S - 1) & ~1) * 8);
        const uint32_t offb = (uint32_t)(((int64_t)(lane >> 4) * ld + imin(2 * (lane & 15), (w - 1) & ~1)) * 8);
        uint64_t pa = (uint64_t)(uintptr_t)uniform_ptr(Akk + (int64_t)wave * ld + c0 + s0);
        uint64_t pb = (uint64_t)(uintptr_t)uniform_ptr(Akk + (int64_t)(4 * wave) * ld + c0);
        const uint64_t da = 32 * (uint64_t)ld, db = 4 * da;
        auto slot = [&](auto jc, uint32_t st) __attribute__((always_inline)) {
          constexpr int j = decltype(jc)::value;
          if constexpr (j < 4) {
            dma16i<j * 4 * PT_ALD * 8>(pa, offa, st + (uint32_t)(wave * PT_ALD * 8));
            pa += da;
          } else {
            dma16i<16 * PT_ALD * 8>(pb, offb, st + (uint32_t)(wave * 1024));
            pb += db;
          }
        };
        auto compute = [&](auto issue_c, int so, uint32_t st) __attribute__((always_inline)) {
          constexpr bool ISSUE = decltype(issue_c)::value;
          double fa[2][2], fb[2][2];
          auto read = [&](int ks, int buf) __attribute__((always_inline)) {
            fa[buf][0] = fa0[so + ks * 4 * PT_ALD];
            fa[buf][1] = fa0[so + ks * 4 * PT_ALD + 16];
            fb[buf][0] = fb0[so + ks * 4 * PT_W];
            fb[buf][1] = fb0[so + ks * 4 * PT_W + 16];
          };
          // (all at once: the other workgroup's products run meanwhile, and the
          // panels come from beyond the L2s more often than not)
          if constexpr (ISSUE) static_for<5>([&](auto jc) __attribute__((always_inline)) { slot(jc, st); });
          read(0, 0);
          static_for<4>([&](auto kc) __attribute__((always_inline)) {
            constexpr int ks = decltype(kc)::value;
            if constexpr (ks < 3) read(ks + 1, (ks + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            if (mine) {
#pragma unroll
              for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
                  acc[rb][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[ks & 1][cb], fa[ks & 1][rb], acc[rb][cb], 0, 0, 2 /* neg B */);
            }
            __builtin_amdgcn_sched_barrier(0);
          });
        };
        const int nch = c0 >> 4;  // even
        static_for<5>([&](auto jc) __attribute__((always_inline)) { slot(jc, l0); });
        int so = 0;
#pragma unroll 1
        for (int ch = 0; ch + 1 < nch; ++ch) {
          wait_vmcnt<0>();
          lds_barrier();
          compute(std::true_type(), so, l0 + (uint32_t)(PT_STAGE - so) * 8);
          so = PT_STAGE - so;
        }
        wait_vmcnt<0>();
        lds_barrier();
        compute(std::false_type(), so, 0);
      }
      if (s0 == 0) {
        if (wave == 0) {
          // the diagonal block: rows and columns past the order are the identity's
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int cb = 0; cb <= rb; ++cb)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int r = rb * 16 + l16, c = cb * 16 + 4 * i + lg;
                acc[rb][cb][i] = (r < w && c < w && r >= c) ? acc[rb][cb][i] : (r == c ? 1.0 : 0.0);
              }
          d4 y[2][1];  // the panel's rows of b, transposed
          if (fwd) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int c = h * 16 + 4 * i + lg;
                const double v = Bf[(int64_t)imin(l16, nrhs - 1) * ldbf + c0 + imin(c, w - 1)];
                y[h][0][i] = c < w ? v : 0.0;
              }
          }
          d4 lf, ld2, none = {0.0, 0.0, 0.0, 0.0};
          d4& x = acc[1][0];
          const int ia = panel16(acc[0][0], lf, x, e, lane, c0, Fb);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], x[k], acc[1][1], 0, 0, 2 /* neg B */);
            Xb[k * 64 + lane] = x[k];
          }
          const int ib = panel16(acc[1][1], ld2, none, e, lane, c0 + 16, Fb + QUAD_OPS * 64);
          if (lane == 0) s_pinfo = ia ? ia : ib;
          if (fwd) {
            panel16_rows(y[0], Fb, lane);
#pragma unroll
            for (int k = 0; k < 4; ++k)
              y[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], y[0][0][k], y[1][0], 0, 0, 2 /* neg B */);
            panel16_rows(y[1], Fb + QUAD_OPS * 64, lane);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int k = 0; k < 4; ++k) Yb[(4 * h + k) * 64 + lane] = quad_to_row<0>(y[h][0][k]);
          }
          lds_barrier();
          if (__builtin_amdgcn_readfirstlane(ia | ib) == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int c = 4 * i + lg;
              if (l16 >= c && l16 < w) {
                st_dev(P + (int64_t)c * ld + l16, lf[i]);
                if constexpr (IN32) st_dev(P32 + (int64_t)c * ld32 + l16, (float)lf[i]);
              }
              if (16 + l16 < w) {
                st_dev(P + (int64_t)c * ld + 16 + l16, x[i]);
                if constexpr (IN32) st_dev(P32 + (int64_t)c * ld32 + 16 + l16, (float)x[i]);
                if (l16 >= c) {
                  st_dev(P + (int64_t)(16 + c) * ld + 16 + l16, ld2[i]);
                  if constexpr (IN32) st_dev(P32 + (int64_t)(16 + c) * ld32 + 16 + l16, (float)ld2[i]);
                }
              }
            }
            if (fwd && l16 < nrhs) {
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const int c = h * 16 + 4 * i + lg;
                  if (c < w) st_dev(Bf + (int64_t)l16 * ldbf + c0 + c, y[h][0][i]);
                }
            }
          }
        } else {
          lds_barrier();
        }
        const int info = __builtin_amdgcn_readfirstlane(s_pinfo);
        if (info != 0) return info;
      }
      // the rows below the block (the panel is then 32 wide)
      if (mine && (s0 > 0 || wave > 0)) {
        double* const bp = fwd ? Bf + (int64_t)imin(lg, nrhs - 1) * ldbf + c0 + s0 : nullptr;
        double b[2] = {0.0, 0.0};
        if (fwd)
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) b[rb] = bp[imin(rw + rb * 16 + l16, S - 1)];
        d4 x1[2] = {acc[0][0], acc[1][0]}, x2[2] = {acc[0][1], acc[1][1]};
        panel16_rows(x1, Fb, lane);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double f = Xb[k * 64 + lane];
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
            x2[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(f, x1[rb][k], x2[rb], 0, 0, 2 /* neg B */);
        }
        panel16_rows(x2, Fb + QUAD_OPS * 64, lane);
        if (fwd) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const double y1 = Yb[k * 64 + lane], y2 = Yb[(4 + k) * 64 + lane];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
              b[rb] = mfma4_f64_neg(y1, x1[rb][k], b[rb]);
              b[rb] = mfma4_f64_neg(y2, x2[rb][k], b[rb]);
            }
          }
        }
        double* const q0 = P + (int64_t)lg * ld + s0 + rw + l16;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          if (rw + rb * 16 + l16 < S) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              st_dev(q0 + (int64_t)(4 * i) * ld + rb * 16, x1[rb][i]);
              st_dev(q0 + (int64_t)(16 + 4 * i) * ld + rb * 16, x2[rb][i]);
              if constexpr (IN32) {
                float* const q32 = P32 + (int64_t)(4 * i + lg) * ld32 + s0 + rw + rb * 16 + l16;
                st_dev(q32, (float)x1[rb][i]);
                st_dev(q32 + 16 * ld32, (float)x2[rb][i]);
              }
            }
            if (fwd && lg < nrhs) st_dev(bp + rw + rb * 16 + l16, b[rb]);
          }
      }
      if (s0 + 128 < R) lds_barrier();  // the next slab's stages
    }
    // the panel must be visible to every wavefront before the next panel's
    // update reads it
    wait_vmcnt<0>();
    lds_barrier();
  }
  return 0;
}

// ---------------------------------------------------------------------------
// TRSM work item: a strip of S <= 32 rows of A_ik, X := X L_kk^{-T}
// (mk = order of L_kk, a multiple of 16; X in FP64 or, in the mixed-precision
// factorization, FP32 storage, computed in FP64 either way).  Transposed, X^T := L_kk^{-1} X^T
// is a forward solve with the strip's rows as 32 right-hand sides (two
// groups of 16).  The strip lives in LDS as Xs[g][c][16] (row 16g + j,
// column c), which the MFMA fragments read without bank conflicts.  For
// each block of 16 columns, wavefronts 0 and 1 solve the block for their
// row group in four 4-column sub-steps on the matrix cores (the exact 4x4
// inverse of the diagonal block's sub-block applied by one MFMA, then one
// MFMA for the columns after it), then every wavefront subtracts the block's
// contribution from its later column blocks.  The solver's L data for the
// next step is requested one step ahead; the update fragments at the start
// of the step, to land during the solve.
//
// REV = 2: the same solve, also storing P^T at Qb (ld ldq): the explicit
// inverse, from identity strips.  rb0: the strip's columns before block rb0
// are zero (an identity strip's before its own rows), so the steps over them
// are left out.
#define TS 32

// Hs (non-null): the solved strip (its first row a multiple of 16 in the
// matrix) is also stored as three BF16 terms (split3) in the 1 KB blocks of
// gemm_bf16x6_wide: Hs is the block of the strip's first row and column, a
// row group's blocks follow each other, the next row group is hgs and the next
// term hterm values further (mk a multiple of 32).
template <typename TX, int REV = 0>
__device__ __forceinline__ void trsm_strip(TX* __restrict__ X, int64_t ldx, const double* __restrict__ Lkk, int64_t ld,
                                           int S, int mk, double* lds, double* Qb = nullptr,
                                           int64_t ldq = 0, uint16_t* Hs = nullptr, int64_t hgs = 0,
                                           int64_t hterm = 0, int rb0 = 0) {
  double* Xs = lds;  // [2][512][16]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int nblk = mk >> 4;
  // L(row, col) of the operator the forward solve applies
  auto lat = [&](int row, int col) __attribute__((always_inline)) { return Lkk[(int64_t)col * ld + row]; };
  // the strip: thread (r, c0) moves rows r of columns c0 + 8u, 16 loads in flight
  {
    const int r = tid & 31, c0 = tid >> 5, rr = imin(r, S - 1);
#pragma unroll 1
    for (int part = 0; part < 4; ++part) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = (double)X[(int64_t)imin(c0 + 8 * (u + 16 * part), mk - 1) * ldx + rr];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int c = c0 + 8 * (u + 16 * part);
        if (c < mk) Xs[(r >> 4) * 8192 + c * 16 + (r & 15)] = (r < S) ? v[u] : 0.0;
      }
    }
  }
  // Step data.  Solver lanes (wavefronts 0, 1): the 4x4 sub-block entries
  // d[a][b] (a >= b) of sub-block s* = l16 / 4 and the update entries
  // L[q0 + l16][q0 + 4s + lg], requested one step ahead; every wavefront:
  // the fragments L[later column block rows, q0 + 4kk + lg], requested at
  // the start of the step and used after the block's solve.
  struct SolveData {
    double d[10];
    double fd[4];
  };
  auto fetch_solve = [&](int rb, SolveData& sd) __attribute__((always_inline)) {
    const int q0 = rb * 16;
    const int sb = q0 + 4 * (l16 >> 2);
    int n = 0;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int bq = 0; bq <= a; ++bq) sd.d[n++] = lat(sb + a, sb + bq);
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) sd.fd[s4] = lat(q0 + l16, q0 + 4 * s4 + lg);
  };
  auto step = [&](int rb, const SolveData& sd, SolveData& sdn) __attribute__((always_inline)) {
    const int q0 = rb * 16;
    __syncthreads();  // the block's columns are final (and, first time, the strip is staged)
    double fl[8][4];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int crow = imin(q0 + 16 + (wave + 4 * t) * 16 + l16, mk - 1);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) fl[t][kk] = lat(crow, q0 + kk * 4 + lg);
    }
    if (wave < 2) {
      if (rb + 1 < nblk) fetch_solve(rb + 1, sdn);
      const int g = wave;
      // column lg of the inverse of sub-block s* = l16 / 4; this lane's A entry is row l16 % 4
      double dd[4][4];
      {
        int n = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int bq = 0; bq < 4; ++bq) dd[a][bq] = (bq <= a) ? sd.d[n++] : 0.0;
      }
      double w[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        double t = (a == lg) ? 1.0 : 0.0;
#pragma unroll
        for (int bq = 0; bq < a; ++bq) t -= dd[a][bq] * w[bq];
        w[a] = (a < lg) ? 0.0 : t * (1.0 / dd[a][a]);
      }
      const int i4 = l16 & 3;
      const double wmine = (i4 == 0) ? w[0] : (i4 == 1) ? w[1] : (i4 == 2) ? w[2] : w[3];
      d4 acc;
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = Xs[g * 8192 + (q0 + 4 * v + lg) * 16 + l16];
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const double fw = ((l16 >> 2) == s4) ? wmine : 0.0;
        const d4 z = __builtin_amdgcn_mfma_f64_16x16x4f64(fw, acc[s4], d4{0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
        acc[s4] = z[s4];
        const double fdv = (l16 >= 4 * s4 + 4) ? sd.fd[s4] : 0.0;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fdv, z[s4], acc, 0, 0, 2 /* neg B */);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) Xs[g * 8192 + (q0 + 4 * v + lg) * 16 + l16] = acc[v];
    }
    __syncthreads();
    // X^T[later column blocks] -= L[those rows, q0:q0+16] X^T[q0:q0+16] for both row groups
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int cb = rb + 1 + wave + 4 * t;
      if (cb < nblk) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          d4 acc;
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[v] = Xs[g * 8192 + (cb * 16 + 4 * v + lg) * 16 + l16];
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const double fx = Xs[g * 8192 + (q0 + kk * 4 + lg) * 16 + l16];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fl[t][kk], fx, acc, 0, 0, 2 /* neg B */);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) Xs[g * 8192 + (cb * 16 + 4 * v + lg) * 16 + l16] = acc[v];
        }
      }
    }
  };
  SolveData sa, sb;
  if (wave < 2) fetch_solve(rb0, sa);
  for (int rb = rb0; rb < nblk; rb += 2) {
    step(rb, sa, sb);
    if (rb + 1 < nblk) step(rb + 1, sb, sa);
  }
  __syncthreads();
  const int r = tid & 31, c0 = tid >> 5;
  if (r < S)
    for (int c = c0; c < mk; c += 8) st_dev(X + (int64_t)c * ldx + r, (TX)Xs[(r >> 4) * 8192 + c * 16 + (r & 15)]);
  if (Hs) {
    // runs of 4 columns (8 bytes per term): lane l of wavefront w takes row
    // 16 (w & 1) + l % 16 (consecutive rows: conflict-free reads of Xs) and
    // runs 4 u + l / 16 of its half of the columns (w / 2); a store
    // instruction then writes half of a 1 KB block
    const int hr = 16 * (wave & 1) + l16, half = mk >> 3;  // runs of 4 per half of the columns
    if (hr < S) {
#pragma unroll 1
      for (int u = 0; 4 * u + lg < half; ++u) {
        const int c0 = (wave >> 1) * (mk >> 1) + 4 * (4 * u + lg);
        uint64_t t0 = 0, t1 = 0, t2 = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t a0, a1, a2;
          split3(Xs[(hr >> 4) * 8192 + (c0 + e) * 16 + (hr & 15)], a0, a1, a2);
          t0 |= (uint64_t)a0 << (16 * e);
          t1 |= (uint64_t)a1 << (16 * e);
          t2 |= (uint64_t)a2 << (16 * e);
        }
        uint16_t* h = Hs + (int64_t)(wave & 1) * hgs + (int64_t)(c0 >> 5) * 512 + bw_slot(l16, (c0 >> 3) & 3) * 8 + (c0 & 7);
        st_dev(reinterpret_cast<uint64_t*>(h), t0);
        st_dev(reinterpret_cast<uint64_t*>(h + hterm), t1);
        st_dev(reinterpret_cast<uint64_t*>(h + 2 * hterm), t2);
      }
    }
  }
  if (REV == 2 && Qb != nullptr) {
    for (int idx = tid; idx < S * mk; idx += NT) {
      const int rr = idx / mk, c = idx - rr * mk;
      st_dev(Qb + (int64_t)rr * ldq + c, Xs[(rr >> 4) * 8192 + c * 16 + (rr & 15)]);
    }
  }
}

// ---------------------------------------------------------------------------
// TRSM work item through the diagonal tile's explicit inverse (FP64 launches
// that compute it, TRTRI(k) before TRSM(i, k)): rows of A_ik, X := X L_kk^{-T}
// = X (L_kk^{-1})^T, one 128-row block per item, as products with L_kk^{-1}
// (Linv, column-major, ld nb; entry (c, t) is zero for t > c) on the matrix
// cores.  Column block c of the result reads the columns of X up to the
// block's end, so the blocks go from the right to the left, each written
// after its own product has read it; no other item touches these rows.
template <int SEG>
__device__ __forceinline__ void trsm_inv_rows(double* __restrict__ X, int64_t ld, const double* __restrict__ Linv,
                                              int64_t nb, int M, int mk, double* lds) {
  for (int c0 = ((mk - 1) / GB) * GB; c0 >= 0; c0 -= GB) {
    const int N = imin(GB, mk - c0), K = c0 + N;
    gemm_tile<SEG>(X + (int64_t)c0 * ld, ld, X, ld, Linv + c0, nb, M, N, K, false, true, true, lds);
  }
}

// The same for a tile of order mk <= 128 (a multiple of 16): S <= 32 rows of
// A_ik, X := X L_kk^{-T}, small enough to hold every operand in registers.
// Wavefront w takes the 16-column blocks w and 7 - w of the result (together
// the same work for every wavefront: block c needs the 16 (c + 1) columns up
// to its own), requests all its fragments of L_kk^{-1} and X at once and
// stores after every wavefront has its part of X.  Bound by that one memory
// round trip and 72 products per wavefront: 14-17 us at mk = 128 (order
// 1024), against 21 of the substituting strip.
__device__ __forceinline__ void trsm_inv_strip(double* __restrict__ X, int64_t ld, const double* __restrict__ Linv,
                                               int64_t nb, int S, int mk) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int nblk = mk >> 4;
  const double* const Xl = X + (int64_t)lg * ld + imin(l16, S - 1);
  const int64_t r1 = imin(16 + l16, S - 1) - imin(l16, S - 1);
  const double* const Ll = Linv + (int64_t)lg * nb + l16;
  const int ca = wave, cz = 7 - wave;  // ca < cz
  double fa[16], fz[32], x[2][32];
  // k-steps 4 t .. 4 t + 3 are block column t of L_kk^{-1}
#pragma unroll
  for (int t = 0; t < 8; ++t)
    if (t < nblk && t <= (cz < nblk ? cz : ca)) {
#pragma unroll
      for (int k = 4 * t; k < 4 * t + 4; ++k) {
        x[0][k] = Xl[(int64_t)(4 * k) * ld];
        x[1][k] = Xl[(int64_t)(4 * k) * ld + r1];
        if (cz < nblk) fz[k] = Ll[(int64_t)(4 * k) * nb + cz * 16];
        if (t < 4 && t <= ca && ca < nblk) fa[k < 16 ? k : 0] = Ll[(int64_t)(4 * k) * nb + ca * 16];
      }
    }
  d4 acc[2][2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 2; ++g) acc[b][g] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    if (cz < nblk && t <= cz) {
#pragma unroll
      for (int k = 4 * t; k < 4 * t + 4; ++k) {
        acc[1][0] = mfma_f64(fz[k], x[0][k], acc[1][0]);
        acc[1][1] = mfma_f64(fz[k], x[1][k], acc[1][1]);
      }
    }
    if (t < 4 && ca < nblk && t <= ca) {
#pragma unroll
      for (int k = 4 * t; k < 4 * t + 4; ++k) {
        acc[0][0] = mfma_f64(fa[k < 16 ? k : 0], x[0][k], acc[0][0]);
        acc[0][1] = mfma_f64(fa[k < 16 ? k : 0], x[1][k], acc[0][1]);
      }
    }
  }
  // every wavefront's products must be done, so that its part of X has been read
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 2; ++g) asm volatile("" : : "v"(acc[b][g]));
  lds_barrier();
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int cb = b == 0 ? ca : cz;
    if (cb < nblk) {
      double* const Xs = X + ((int64_t)cb * 16 + lg) * ld + l16;
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (16 * g + l16 < S) {
#pragma unroll
          for (int i = 0; i < 4; ++i) st_dev(Xs + (int64_t)(4 * i) * ld + 16 * g, acc[b][g][i]);
        }
    }
  }
}

// C[M x N] -= Ap[M x K] Bp[N x K]^T for M, N <= 64, K <= 128 a multiple of 16:
// an update on the critical path of a factorization by small tiles.  Every
// fragment goes straight from memory to registers, all requested at once (a
// K this short does not repay stages in LDS); 2 x 2 wavefronts of 32 x 32.
// The products come in the order of gemm_tile's.  Bound by the memory round
// trip: 10-11 us at K = 128 (order 1024), against 24 of a 128 x 128 item.
// from_c: they are subtracted from C one after the other (potrf_columns' order
// of rounding) instead of summed first.
__device__ __forceinline__ void gemm_reg64(double* __restrict__ C, const double* __restrict__ Ap,
                                           const double* __restrict__ Bp, int64_t ld, int M, int N, int K,
                                           bool lower_only, bool from_c = false) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  if (wr >= M || wc >= N || (lower_only && wc > wr)) return;
  const double* A0[2];
  const double* B0[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    A0[g] = Ap + (int64_t)lg * ld + imin(wr + 16 * g + l16, M - 1);
    B0[g] = Bp + (int64_t)lg * ld + imin(wc + 16 * g + l16, N - 1);
  }
  double fa[2][32], fb[2][32];
  d4 acc[2][2], c0[2][2];
#pragma unroll
  for (int t = 0; t < 8; ++t)
    if (16 * t < K) {
#pragma unroll
      for (int k = 4 * t; k < 4 * t + 4; ++k)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          fa[g][k] = A0[g][(int64_t)(4 * k) * ld];
          fb[g][k] = B0[g][(int64_t)(4 * k) * ld];
        }
    }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wr + 16 * r + l16, col = wc + 16 * c + 4 * i + lg;
        const double v = C[(int64_t)imin(col, N - 1) * ld + imin(row, M - 1)];
        c0[r][c][i] = from_c ? 0.0 : v;
        acc[r][c][i] = from_c ? -v : 0.0;
      }
#pragma unroll
  for (int t = 0; t < 8; ++t)
    if (16 * t < K) {
#pragma unroll
      for (int k = 4 * t; k < 4 * t + 4; ++k)
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            acc[r][c] = mfma_f64(fb[c][k], fa[r][k], acc[r][c]);
    }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wr + 16 * r + l16, col = wc + 16 * c + 4 * i + lg;
        if (row < M && col < N && (!lower_only || row >= col)) st_dev(C + (int64_t)col * ld + row, c0[r][c][i] - acc[r][c][i]);
      }
}

// ---------------------------------------------------------------------------
// Solve work items.  Right-hand sides are processed 16 columns at a time
// (the N of an MFMA block).  MFMA layout used here: A operand = L fragment
// (rows of L on lanes % 16), B operand = right-hand-side fragment
// (right-hand sides on lanes % 16); a lane then holds rows 4i + lane/16 of
// one right-hand side (lane % 16) of the 16x16 result.

// Tile solves, register resident.  The tile's rows form blocks of 16
// (nblk <= 32); wavefront w owns blocks w, w + 4, ..., and keeps their
// right-hand sides in registers in the layout of an MFMA result: element v
// of lane l holds row 4v + l/16 of right-hand side l%16.  That is also the
// layout of the B operand of an MFMA's k-step v, so a solved block feeds the
// updates of the other blocks without leaving registers.
//
// Block rb is solved by its owner in four dependent 4-row sub-steps:
// y_s := W_s r_s with W_s the inverse of the s-th 4x4 diagonal block of L
// (one MFMA whose A operand is W_s in rows 4s..4s+3 and zero elsewhere),
// then the rows below lose L[rows, 4s..4s+3] y_s (one MFMA).  The 4x4
// inverses are formed once per task by substitution; a 4x4 inverse of an
// integer factor with power-of-two pivots is exact, so such systems are
// still solved exactly.  The solved block is published through LDS (two
// buffers, one barrier per block) and every wavefront subtracts its
// contribution from the blocks it owns; the owner of the next block
// updates and solves that block first.  The L fragments of block rb's
// updates are requested one block ahead.
//
// LDS: Fr[blk][s][f][64] the A-operand fragments of the sub-steps (f = 0:
// inverse, f = 1: update), then two 16 x 16 exchange buffers.
#define FR_SLOT(blk, s, f) ((((blk) * 4 + (s)) * 2 + (f)) * 64)
#define FR0_SLOT(blk, s) (((blk) * 4 + (s)) * 64)  // COMPACT: the inverses only

// Builds Fr for the forward (trans = false) or backward (trans = true)
// solve of the nblk diagonal 16-blocks of L_kk (m rows).  Rows and columns
// past m behave as the identity.  COMPACT: only the inverse fragments (the
// update fragments are read from L_kk by the solve).
template <bool COMPACT = false>
__device__ __forceinline__ void build_block_fragments(const double* __restrict__ Lkk, int64_t ld, int m,
                                                      bool trans, double* Fr) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int s = tid >> 6;  // wavefront w builds sub-step w of every block
  const int l16 = lane & 15, lg = lane >> 4;
  const int nblk = (m + 15) >> 4;
  auto slot0 = [](int blk, int s4) __attribute__((always_inline)) {
    return COMPACT ? FR0_SLOT(blk, s4) : FR_SLOT(blk, s4, 0);
  };
  if constexpr (COMPACT) {
    for (int blk = 0; blk < nblk; ++blk) Fr[FR0_SLOT(blk, s) + lane] = 0.0;
  } else {
    // update fragments (and zeros in the inverse slots): all 32 loads are
    // requested before any is used.  Forward: A[i][k] = L[r0+i][r0+4s+k] for
    // i >= 4s+4; backward: A[i][k] = L[r0+4s+k][r0+i] for i < 4s.
    const int row = trans ? 4 * s + lg : l16, col = trans ? l16 : 4 * s + lg;
    const bool live = trans ? (l16 < 4 * s) : (l16 >= 4 * s + 4);
    double v[32];
#pragma unroll
    for (int blk = 0; blk < 32; ++blk) {
      const int r0 = imin(blk, nblk - 1) * 16, bw = imin(16, m - r0);
      v[blk] = Lkk[(int64_t)(r0 + imin(col, bw - 1)) * ld + r0 + imin(row, bw - 1)];
    }
#pragma unroll
    for (int blk = 0; blk < 32; ++blk) {
      if (blk < nblk) {
        const int bw = imin(16, m - blk * 16);
        Fr[FR_SLOT(blk, s, 1) + lane] = (live & (row < bw) & (col < bw)) ? v[blk] : 0.0;
        Fr[FR_SLOT(blk, s, 0) + lane] = 0.0;
      }
    }
  }
  __syncthreads();
  // column c of the inverse of the 4x4 block (blk, s), by substitution; a
  // thread takes blocks tid/16 and tid/16 + 16
  {
    const int c = tid & 3, s4 = (tid >> 2) & 3;
    double d[2][4][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int blk = imin((tid >> 4) + 16 * h, nblk - 1);
      const int r0 = blk * 16 + 4 * s4, bw = imin(4, m - r0);  // bw may be <= 0: identity
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double x = Lkk[(int64_t)(imin(m - 1, r0 + j)) * ld + imin(m - 1, r0 + i)];
          d[h][i][j] = ((j <= i) & (i < bw) & (j < bw)) ? x : (i == j ? 1.0 : 0.0);
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int blk = (tid >> 4) + 16 * h;
      if (blk < nblk) {
        double w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          double t = (i == c) ? 1.0 : 0.0;
#pragma unroll
          for (int j = 0; j < i; ++j) t -= d[h][i][j] * w[j];
          w[i] = (i < c) ? 0.0 : t * (1.0 / d[h][i][i]);
        }
        // forward A[i'][k'] = W[i'-4s][k'] (i' in 4s..4s+3) -> lane k'*16 + i';
        // backward A[i'][k'] = W[k'][i'-4s] -> lane i*16 + 4s + c
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i >= c) Fr[slot0(blk, s4) + (trans ? i * 16 + 4 * s4 + c : c * 16 + 4 * s4 + i)] = w[i];
      }
    }
  }
  __syncthreads();
}

// Solves the owner's block in place (acc: the block's right-hand sides).
__device__ __forceinline__ void solve_block(d4& acc, const double* Fr, int blk, bool trans, int lane) {
#pragma unroll
  for (int ss = 0; ss < 4; ++ss) {
    const int s = trans ? 3 - ss : ss;
    const d4 z = __builtin_amdgcn_mfma_f64_16x16x4f64(Fr[FR_SLOT(blk, s, 0) + lane], acc[s], d4{0.0, 0.0, 0.0, 0.0},
                                                     0, 0, 0);
    acc[s] = z[s];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Fr[FR_SLOT(blk, s, 1) + lane], z[s], acc, 0, 0, 2 /* neg B */);
  }
}

// The same with the inverse fragments of the compact layout and the update
// fragments fu (sub-step order ss) read from L_kk: entry (row, col) of the
// block's sub-step s = trans ? 3 - ss : ss, zero outside its live part.
__device__ __forceinline__ void solve_block_c(d4& acc, const double* Fr, int blk, const double (&fu)[4], int m,
                                              bool trans, int lane) {
  const int l16 = lane & 15, lg = lane >> 4;
  const int bw = imin(16, m - blk * 16);
#pragma unroll
  for (int ss = 0; ss < 4; ++ss) {
    const int s = trans ? 3 - ss : ss;
    const int row = trans ? 4 * s + lg : l16, col = trans ? l16 : 4 * s + lg;
    const bool live = (trans ? (l16 < 4 * s) : (l16 >= 4 * s + 4)) & (row < bw) & (col < bw);
    const d4 z = __builtin_amdgcn_mfma_f64_16x16x4f64(Fr[FR0_SLOT(blk, s) + lane], acc[s], d4{0.0, 0.0, 0.0, 0.0},
                                                     0, 0, 0);
    acc[s] = z[s];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(live ? fu[ss] : 0.0, z[s], acc, 0, 0, 2 /* neg B */);
  }
}

// trans = false: Y_k := L_kk^{-1} B_k; trans = true: X_k := L_kk^{-T} Y_k.
// COMPACT (the compact instance, 69632 bytes of LDS, 256 registers): Fr
// holds only the blocks' inverse fragments, the update fragments of the
// block a step solves are loaded from L_kk one step ahead, and the step's
// update fragments at its start (one buffer instead of two: the other
// workgroup on the compute unit covers the wait).
template <bool COMPACT = false>
__device__ __forceinline__ void tile_solve(const double* __restrict__ Lkk, int64_t ld, double* Bk, int64_t ldb,
                                           int m, int nrhs, bool trans, double* lds) {
  double* Fr = lds;                                      // [nblk][4][2][64] (COMPACT: [nblk][4][64])
  double* Ex = lds + 32 * 4 * (COMPACT ? 1 : 2) * 64;  // [2][4][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int nblk = (m + 15) >> 4;
  build_block_fragments<COMPACT>(Lkk, ld, m, trans, Fr);
  // COMPACT: the raw entries behind block blk's update fragments (sub-step
  // order), clamped into the tile; solve_block_c masks them
  auto fetch_fu = [&](int blk, double (&fu)[4]) __attribute__((always_inline)) {
    const int r0 = imin(imax(blk, 0), nblk - 1) * 16, bw = imin(16, m - r0);
#pragma unroll
    for (int ss = 0; ss < 4; ++ss) {
      const int s = trans ? 3 - ss : ss;
      const int row = trans ? 4 * s + lg : l16, col = trans ? l16 : 4 * s + lg;
      fu[ss] = Lkk[(int64_t)(r0 + imin(col, bw - 1)) * ld + r0 + imin(row, bw - 1)];
    }
  };
  // fragments of the updates by solved block rb of the owned blocks ub = wave + 4t:
  // forward L[ub rows][rb cols], backward L[rb rows][ub cols]^T
  // Only the blocks the solved block rb still updates are fetched (forward:
  // ub > rb, backward: ub < rb): the same blocks that use the fragments.
  auto fetch = [&](int rb, double (&fl)[8][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int ub = wave + 4 * t;
      if (trans ? (ub < rb) : (ub > rb && ub < nblk)) {
        const int ur = imin(ub * 16 + l16, m - 1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int q = imin(rb * 16 + 4 * kk + lg, m - 1);
          fl[t][kk] = trans ? Lkk[(int64_t)ur * ld + q] : Lkk[(int64_t)q * ld + ur];
        }
      }
    }
  };
  for (int j0 = 0; j0 < nrhs; j0 += 16) {
    const int jn = imin(16, nrhs - j0);
    const int jc = imin(l16, jn - 1);
    d4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = (wave + 4 * t) * 16 + 4 * v + lg;
        const double x = Bk[(int64_t)(j0 + jc) * ldb + imin(row, m - 1)];
        acc[t][v] = (row < m) ? x : 0.0;
      }
    const int first = trans ? nblk - 1 : 0;
    double fla[8][4], flb[8][4];
    double fua[4], fub[4];  // COMPACT: update fragments of the block a step solves
    if constexpr (COMPACT)
      fetch_fu(first, fub);
    else
      fetch(first, fla);
    // the first block: solved by its owner, published in buffer 0
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (wave + 4 * t == first) {
        if constexpr (COMPACT)
          solve_block_c(acc[t], Fr, first, fub, m, trans, lane);
        else
          solve_block(acc[t], Fr, first, trans, lane);
#pragma unroll
        for (int v = 0; v < 4; ++v) Ex[v * 64 + lane] = acc[t][v];
      }
    if constexpr (COMPACT) fetch_fu(trans ? first - 1 : first + 1, fua);
    __syncthreads();
    // one step: block rb is solved and published in buffer (step & 1); its
    // contribution goes to every block still to be solved, the next block first
    auto step = [&](int step_i, const double (&fl)[8][4], double (&fln)[8][4], const double (&fu)[4],
                    double (&fun)[4]) __attribute__((always_inline)) {
      const int rb = trans ? nblk - 1 - step_i : step_i;
      const int nx = trans ? rb - 1 : rb + 1;
      const bool has_next = trans ? (rb > 0) : (rb + 1 < nblk);
      const double* ex = Ex + (step_i & 1) * 256;
      double* exn = Ex + ((step_i + 1) & 1) * 256;
      d4 yb;
#pragma unroll
      for (int v = 0; v < 4; ++v) yb[v] = ex[v * 64 + lane];
      if constexpr (COMPACT) {
        // one buffer (fl and fln are the same array): this step's fragments
        // now, the next solved block's update fragments one step ahead
        fetch(rb, fln);
        if (has_next) fetch_fu(trans ? nx - 1 : nx + 1, fun);
      } else if (has_next) {
        fetch(nx, fln);
      }
#pragma unroll
      for (int t = 0; t < 8; ++t)
        if (has_next && wave + 4 * t == nx) {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(fl[t][kk], yb[kk], acc[t], 0, 0, 2 /* neg B */);
          if constexpr (COMPACT)
            solve_block_c(acc[t], Fr, nx, fu, m, trans, lane);
          else
            solve_block(acc[t], Fr, nx, trans, lane);
#pragma unroll
          for (int v = 0; v < 4; ++v) exn[v * 64 + lane] = acc[t][v];
        }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int ub = wave + 4 * t;
        if ((trans ? ub < nx : (ub > nx && ub < nblk))) {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(fl[t][kk], yb[kk], acc[t], 0, 0, 2 /* neg B */);
        }
      }
      __syncthreads();
    };
    for (int si = 0; si < nblk; si += 2) {
      if constexpr (COMPACT) {
        step(si, fla, fla, fua, fub);
        if (si + 1 < nblk) step(si + 1, fla, fla, fub, fua);
      } else {
        step(si, fla, flb, fua, fub);
        if (si + 1 < nblk) step(si + 1, flb, fla, fub, fua);
      }
    }
    if (l16 < jn) {
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = (wave + 4 * t) * 16 + 4 * v + lg;
          if (row < m) st_dev(Bk + (int64_t)(j0 + l16) * ldb + row, acc[t][v]);
        }
    }
  }
}

// The strip update of gemv_strip with 16-byte transfers (two FP64 values,
// or two FP32 values in 8 bytes, per lane and load): half the load
// instructions.  K is taken in pairs of k-steps: step u of a wavefront
// covers K index kw + 8 (u / 2) + 2 (lane / 16) + u % 2, so that a lane's two
// consecutive indices sit in steps 2j and 2j + 1.  Without TRANS a lane's
// rows of L are paired instead: block t holds the strip's rows 2 m + t
// (m = lane % 16), both loaded by one transfer.  Needs a full strip of 32
// rows, a K range whose length is a multiple of 8 and starts even, even
// leading dimensions and 16-byte aligned L and X; then every step of every
// wavefront lies inside K and nothing is masked.
template <typename TL, bool TRANS, bool ASSIGN, class Late>
__device__ __forceinline__ void gemv_strip_wide(const TL* L, int64_t ld, double* Y, const double* X,
                                                int64_t ldb, int k0, int k1, int nrhs, double* lds, Late late) {
  typedef TL TL2 __attribute__((ext_vector_type(2)));
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) TL2 gTL2;
  double* Ps = lds;  // [wavefront][8][64]: the partial products
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int nsteps = (k1 - k0) >> 2;                // even
  const int qs = (((nsteps + 3) >> 2) + 1) & ~1;    // per wavefront, even, at most 32
  const int ns = imax(0, imin(qs, nsteps - wave * qs));  // even
  const int kw = k0 + 4 * wave * qs + 2 * lg;      // this lane's first K index
  gchar* const Lu = (gchar*)uniform_ptr(L);
  const uint32_t es = sizeof(TL), lds_b = (uint32_t)ld * es;
  double fa[32], fb[32];
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if (2 * j < ns) {
      const uint32_t c = (uint32_t)(kw + 8 * j);
      if (TRANS) {  // rows c, c + 1 of columns l16 and 16 + l16
        const TL2 va = *(gTL2*)(Lu + ((uint32_t)l16 * lds_b + c * es));
        const TL2 vb = *(gTL2*)(Lu + ((uint32_t)(16 + l16) * lds_b + c * es));
        fa[2 * j] = (double)va[0];
        fa[2 * j + 1] = (double)va[1];
        fb[2 * j] = (double)vb[0];
        fb[2 * j + 1] = (double)vb[1];
      } else {      // rows 2 l16, 2 l16 + 1 of columns c and c + 1
        const TL2 v0 = *(gTL2*)(Lu + (__umul24(c, lds_b) + (uint32_t)(2 * l16) * es));
        const TL2 v1 = *(gTL2*)(Lu + (__umul24(c + 1, lds_b) + (uint32_t)(2 * l16) * es));
        fa[2 * j] = (double)v0[0];
        fb[2 * j] = (double)v0[1];
        fa[2 * j + 1] = (double)v1[0];
        fb[2 * j + 1] = (double)v1[1];
      }
    }
  if (!late()) return;
  // output element (t, v) of a lane: strip row 2 (4 v + lg) + t (paired rows)
  // or 16 t + 4 v + lg (TRANS); this wavefront adds up two of the eight
  auto out_row = [&](int t, int v) __attribute__((always_inline)) {
    return TRANS ? 16 * t + 4 * v + lg : 2 * (4 * v + lg) + t;
  };
  const int ob = wave >> 1;
  for (int j0 = 0; j0 < nrhs; j0 += 16) {
    const int jn = imin(16, nrhs - j0);
    const int jc = j0 + imin(l16, jn - 1);
    const double* const Xj = X + (int64_t)jc * ldb + kw;
    double x[32];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (2 * j < ns) {
        typedef double dd2 __attribute__((ext_vector_type(2)));
        const dd2 v = *reinterpret_cast<const dd2*>(Xj + 8 * j);
        x[2 * j] = v[0];
        x[2 * j + 1] = v[1];
      }
    double y[2] = {0.0, 0.0};
    if (!ASSIGN)
#pragma unroll
      for (int h = 0; h < 2; ++h) y[h] = Y[(int64_t)jc * ldb + out_row(ob, 2 * (wave & 1) + h)];
    d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (2 * j < ns) {
#pragma unroll
        for (int u = 2 * j; u < 2 * j + 2; ++u) {
          acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u], x[u], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[u], x[u], acc[1], 0, 0, 0);
        }
      }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) Ps[(wave * 8 + 4 * t + v) * 64 + lane] = acc[t][v];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = 4 * ob + 2 * (wave & 1) + h;
      double s = ASSIGN ? Ps[e * 64 + lane] : y[h] - Ps[e * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) s = ASSIGN ? s + Ps[(w * 8 + e) * 64 + lane] : s - Ps[(w * 8 + e) * 64 + lane];
      if (l16 < jn) st_dev(Y + (int64_t)(j0 + l16) * ldb + out_row(ob, e & 3), s);
    }
    __syncthreads();
  }
}

// Solve update on one strip of at most 32 output rows:
//     Y := Y - op(L) X     or, ASSIGN,     Y := op(L) X
// with op(L) = L (output row r, K index c at L[c ld + r]: the forward
// update, and the diagonal steps that apply an explicit inverse) or, TRANS,
// L^T (output row r, K index c at L[r ld + c]: the backward update).  K runs
// over [k0, k1) (row c of X at X[c]); right-hand side j at column j (ld ldb).
// These items sit on the solve's dependency chain and move little data, so
// their time is memory latency: the four wavefronts take a quarter of K each
// and request all of their L fragments (two 16-row blocks, up to 32 k-steps
// of 4) and right-hand-side fragments before the first product, one round
// trip per item.  The quarters' partial products meet in LDS and are added
// in wavefront order, so the result does not depend on timing.  L in FP64
// or FP32 (the mixed-precision working copy); X and Y in FP64.
// late(), called by every wavefront once its fragments of L are requested,
// waits for X and Y (an item claimed before its predecessors are done, on an L
// that is final: its memory time then passes during the wait); false: give up.
template <typename TL, bool TRANS, bool ASSIGN, class Late>
__device__ __forceinline__ void gemv_strip(const TL* L, int64_t ld, double* Y, const double* X,
                                           int64_t ldb, int rows, int k0, int k1, int nrhs, double* lds, Late late) {
  if (rows == 32 && ((k1 - k0) & 7) == 0 && (k0 & 1) == 0 && ((ld | ldb) & 1) == 0 &&
      ((reinterpret_cast<uintptr_t>(L) | reinterpret_cast<uintptr_t>(X)) & 15) == 0) {
    gemv_strip_wide<TL, TRANS, ASSIGN>(L, ld, Y, X, ldb, k0, k1, nrhs, lds, late);
    return;
  }
  double* Ps = lds;  // [wavefront][8][64]: the partial products
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int nsteps = (k1 - k0 + 3) >> 2;  // k-steps of 4
  const int qs = (nsteps + 3) >> 2;       // per wavefront: at most 32 (K <= 512)
  const int ns = imax(0, imin(qs, nsteps - wave * qs));
  const int kw = k0 + 4 * wave * qs;
  const int kend = imin(k1, kw + 4 * ns);  // end of this wavefront's K
  const int ra = imin(l16, rows - 1), rb = imin(16 + l16, rows - 1);
  // L fragments by 32-bit byte offsets from a wave-uniform base (the item
  // spans less than 4 GB: at most 512 columns of at most 614400 rows), so
  // that a fragment's address costs a multiply-add instead of 64-bit
  // arithmetic.  Fragments of k-steps past this wavefront's quarter are
  // loaded (in bounds) but meet zeros in place of X, in groups of 8 k-steps.
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) TL gTL;
  gchar* const Lu = (gchar*)uniform_ptr(L);
  const uint32_t es = sizeof(TL), lds_b = (uint32_t)ld * es;
  const uint32_t offa = TRANS ? (uint32_t)ra * lds_b : (uint32_t)ra * es;
  const uint32_t offb = TRANS ? (uint32_t)rb * lds_b : (uint32_t)rb * es;
  double fa[32], fb[32];
#pragma unroll
  for (int g = 0; g < 4; ++g)
    if (8 * g < ns) {
#pragma unroll
      for (int u = 8 * g; u < 8 * g + 8; ++u) {
        const uint32_t c = (uint32_t)imin(kw + 4 * u + lg, k1 - 1);
        const uint32_t oc = TRANS ? c * es : __umul24(c, lds_b);
        fa[u] = (double)*(gTL*)(Lu + (offa + oc));
        fb[u] = (double)*(gTL*)(Lu + (offb + oc));
      }
    }
  if (!late()) return;
  // this wavefront's two outputs of the strip's eight per lane: block wave / 2,
  // rows 4 v + lg with v = 2 (wave % 2) + h
  const int ob = wave >> 1;
  for (int j0 = 0; j0 < nrhs; j0 += 16) {
    const int jn = imin(16, nrhs - j0);
    const int jc = j0 + imin(l16, jn - 1);
    const double* const Xj = X + (int64_t)jc * ldb;
    // loaded unconditionally (in bounds) and masked at their use: a select
    // between a loaded value and zero would be turned into a branch around
    // each load, with a wait for it at the join
    double x[32];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (8 * g < ns) {
#pragma unroll
        for (int u = 8 * g; u < 8 * g + 8; ++u) x[u] = Xj[imin(kw + 4 * u + lg, k1 - 1)];
      }
    double y[2] = {0.0, 0.0};
    if (!ASSIGN)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = 16 * ob + 4 * (2 * (wave & 1) + h) + lg;
        y[h] = Y[(int64_t)jc * ldb + imin(r, rows - 1)];
      }
    d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (8 * g < ns) {
#pragma unroll
        for (int u = 8 * g; u < 8 * g + 8; ++u) {
          const double xv = (kw + 4 * u + lg < kend) ? x[u] : 0.0;
          acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u], xv, acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[u], xv, acc[1], 0, 0, 0);
        }
      }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) Ps[(wave * 8 + 4 * t + v) * 64 + lane] = acc[t][v];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = 4 * ob + 2 * (wave & 1) + h;
      double s = ASSIGN ? Ps[e * 64 + lane] : y[h] - Ps[e * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) s = ASSIGN ? s + Ps[(w * 8 + e) * 64 + lane] : s - Ps[(w * 8 + e) * 64 + lane];
      const int r = 16 * ob + 4 * (e & 3) + lg;
      if (l16 < jn && r < rows) st_dev(Y + (int64_t)(j0 + l16) * ldb + r, s);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// POTRF of the mixed-precision factorization: the diagonal tiles live in
// FP64 in the workspace (Dk, ld nb) from the start (copied from A) and take
// their SYRK updates there, so the tile is factored in place by the FP64
// tile kernel.  Dk then holds L_kk for the TRSM strips of step k and the
// tile's inverses (TRTRI); the FP32 copy's diagonal tiles are never read.
template <bool BY_COLUMNS>
__device__ __forceinline__ int potrf_tile_mixed(double* __restrict__ Dk, int64_t ldd, int m, double* lds) {
  const int tid = threadIdx.x;
  int info;
  if (m > 128)
    info = potrf_tile<128>(Dk, ldd, m, lds);
  else if constexpr (BY_COLUMNS)
    info = potrf_columns(Dk, ldd, m, lds);
  else
    info = potrf_small(Dk, ldd, m, lds);
  info = __builtin_amdgcn_readfirstlane(info);
  // a ragged tile is padded to a multiple of 16 with the identity (for its
  // explicit inverse, which then holds L^{-1} in its leading m x m block)
  const int mpad = (m + 15) & ~15;
  for (int idx = tid; idx < mpad * mpad; idx += NT) {
    const int c = idx / mpad, r = idx - c * mpad;
    if (r >= c && (r >= m || c >= m)) st_dev(Dk + (int64_t)c * ldd + r, r == c ? 1.0 : 0.0);
  }
  return info;
}

// ---------------------------------------------------------------------------
// DRED work item: rows [r0, r0 + 16) of the diagonal tile's Lbar (ld) get
// the tile's partial products added, slot by slot in a fixed order (each slot
// holds -tril(P_ik^T L_ik), nb x nb at stride slot_stride, ld ldslot; only
// the lower triangle is read and written).  Eight entries per thread and
// four slots per round keep 32 loads in flight.  With LbT set, the strip's
// rows also go transposed into columns [r0, r0 + 16) of LbT (ld ldt), zero
// below the diagonal: Lbar_kk^T for the closed-form tile adjoint.
__device__ __forceinline__ void dred_strip(double* __restrict__ Bkk, int64_t ld, const double* __restrict__ slots,
                                           int64_t slot_stride, int nslots, int64_t ldslot, int m, int r0,
                                           double* __restrict__ LbT = nullptr, int64_t ldt = 0) {
  const int tid = threadIdx.x;
  const int ncol = imin(r0 + 16, m);          // columns that hold lower entries of these rows
  const int tot = 16 * ncol;                  // (row, column) pairs, rows fastest
  for (int base = 0; base < tot; base += 8 * NT) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = imin(base + u * NT + tid, tot - 1), c = idx >> 4, r = imin(r0 + (idx & 15), m - 1);
      v[u] = Bkk[(int64_t)c * ld + r];
    }
    for (int s0 = 0; s0 < nslots; s0 += 4) {
      double t[4][8];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int idx = imin(base + u * NT + tid, tot - 1), c = idx >> 4, r = imin(r0 + (idx & 15), m - 1);
          t[q][u] = (s0 + q < nslots) ? slots[(int64_t)(s0 + q) * slot_stride + (int64_t)c * ldslot + r] : 0.0;
        }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] += t[q][u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = base + u * NT + tid, c = idx >> 4, r = r0 + (idx & 15);
      if (idx < tot && r < m && r >= c) {
        st_dev(Bkk + (int64_t)c * ld + r, v[u]);
        if (LbT) st_dev(LbT + (int64_t)r * ldt + c, v[u]);
      }
      if (LbT && idx < tot && r < m && r < c) st_dev(LbT + (int64_t)r * ldt + c, 0.0);
    }
  }
  if (LbT) {  // the transposed rows below the strip's columns: zero
    const int rows = imin(r0 + 16, m) - r0, below = m - ncol;
    for (int idx = tid; idx < rows * below; idx += NT) {
      const int rr = idx / below, c = ncol + idx - rr * below;
      st_dev(LbT + (int64_t)(r0 + rr) * ldt + c, 0.0);
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint of the factorization of a diagonal tile.  In lower-parameter form
// (the derivative with respect to the entries the factorization reads, the
// lower triangle; Q = P + P^T is twice the symmetric adjoint), the reverse of
// a right-looking tile factorization with tiles of w has, per step k taken
// from the last to the first,
//   Lbar_ik -= sum_{j > k} Q_ij L_jk             (i > k)
//   P_ik     = Lbar_ik L_kk^{-1}                 (i > k)
//   Lbar_kk -= tril(sum_{i > k} P_ik^T L_ik)
//   P_kk     = the adjoint of the w x w factorization:
//              tril(G + G^T) - diag(G),  G = L_kk^{-T} Phi(L_kk^T Lbar_kk) L_kk^{-1}
//              (Phi: lower triangle with the diagonal halved).
// The tile's own adjoint applies this with w = 16 inside the tile, panels
// from the right: the matrix cores form the first line for the panel's rows
// below its diagonal block (Q of the tile as far as it is known, from the
// workspace), one thread per row solves the second, every thread takes one
// entry of the 16 x 16 third and fourth (the 16 x 16 inverse by substitution),
// and the panel's P is written to Q in both orientations and, halved off the
// diagonal (the symmetric adjoint), over Lbar.  Before the panels, the
// partial products of the tile's column are applied to Lbar_kk in a fixed
// order; each slot holds -tril(P_ik^T L_ik) (the tile product subtracts from
// a zero start), so they are added.  Lkk, Bkk: the factor and Lbar tiles (ld);
// LTkk, Qkk: the transposed factor and Q tiles (ldq, zero beyond the order).
__device__ __forceinline__ void prev_tile(const double* __restrict__ Lkk, const double* __restrict__ LTkk,
                                          double* __restrict__ Bkk, int64_t ld, double* __restrict__ Qkk, int64_t ldq,
                                          int m, const double* __restrict__ slots, int64_t slot_stride, int nslots,
                                          int64_t ldslot, double* lds) {
  const int tid = threadIdx.x;
  double* Ps = lds + P_STAGE_DOUBLES;  // [PW][PPLD] the panel's rows below its diagonal block
  double* Ls = Ps + PW * PPLD;         // [16][17] L of the diagonal block, identity-padded
  double* Bs = Ls + 16 * 17;           // [16][17] its Lbar
  double* Ms = Bs + 16 * 17;
  double* Is = Ms + 16 * 17;           // L^{-1} of the block
  double* Ys = Is + 16 * 17;
  double* Gs = Ys + 16 * 17;
  const int ta = tid >> 4, tb = tid & 15;  // the entry (row, column) a thread owns in 16 x 16 steps

  // Lbar_kk -= tril(P_ik^T L_ik), slot by slot (each slot holds the negated product)
  if (nslots > 0) {
    const int tot = m * m;
    for (int base = 0; base < tot; base += 16 * NT) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int idx = imin(base + u * NT + tid, tot - 1), c = idx / m, r = idx - c * m;
        v[u] = Bkk[(int64_t)c * ld + r];
      }
      for (int sl = 0; sl < nslots; ++sl) {
        const double* S0 = slots + (int64_t)sl * slot_stride;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int idx = imin(base + u * NT + tid, tot - 1), c = idx / m, r = idx - c * m;
          v[u] += (r >= c) ? S0[(int64_t)c * ldslot + r] : 0.0;
        }
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int idx = base + u * NT + tid, c = idx / m, r = idx - c * m;
        if (idx < tot && r >= c) st_dev(Bkk + (int64_t)c * ld + r, v[u]);
      }
    }
    wait_vmcnt<0>();
    __syncthreads();
  }
  const int mpad = (m + 15) & ~15;
  for (int c0 = ((m - 1) >> 4) << 4; c0 >= 0; c0 -= PW) {
    const int w = imin(PW, m - c0), R = m - c0;
    // (1) rows below the block: Lbar - Q L over the columns right of the panel, into LDS
    for (int s0 = 16; s0 < R; s0 += 256) {
      gemm_core<128, 256, PW, 8, 4, 4, 0>(Bkk + (int64_t)c0 * ld + c0 + s0, Qkk + (int64_t)(c0 + 16) * ldq + c0 + s0,
                                          LTkk + (int64_t)(c0 + 16) * ldq + c0, ldq, imin(256, R - s0), w,
                                          mpad - c0 - 16, lds, Ps + s0, PPLD, ld);
      __syncthreads();
    }
    {
      const bool in = ta < w && tb < w;
      Ls[ta * 17 + tb] = in ? (ta >= tb ? Lkk[(int64_t)(c0 + tb) * ld + c0 + ta] : 0.0) : (ta == tb ? 1.0 : 0.0);
      Bs[ta * 17 + tb] = (in && ta >= tb) ? Bkk[(int64_t)(c0 + tb) * ld + c0 + ta] : 0.0;
    }
    // the panel's L rows below the block, for the diagonal block's update (stage area is free)
    for (int idx = tid; idx < w * (R - 16); idx += NT) {
      const int c = idx / (R - 16), r = 16 + idx - c * (R - 16);
      lds[c * PPLD + r] = Lkk[(int64_t)(c0 + c) * ld + c0 + r];
    }
    __syncthreads();
    // (2) P rows := Lbar rows L_dd^{-1}: back substitution over the block's columns
    for (int r = 16 + tid; r < R; r += NT) {
      double y[PW];
#pragma unroll
      for (int c = 0; c < PW; ++c) y[c] = (c < w) ? Ps[c * PPLD + r] : 0.0;
#pragma unroll
      for (int c = PW - 1; c >= 0; --c) {
#pragma unroll
        for (int c2 = c + 1; c2 < PW; ++c2) y[c] -= y[c2] * Ls[c2 * 17 + c];
        y[c] = y[c] / Ls[c * 17 + c];
      }
#pragma unroll
      for (int c = 0; c < PW; ++c) Ps[c * PPLD + r] = y[c];
    }
    __syncthreads();
    // (3) Lbar_dd -= tril(P^T L) over the rows below the block
    if (ta >= tb && ta < w) {
      double acc = 0.0;
      for (int r = 16; r < R; ++r) acc += Ps[ta * PPLD + r] * lds[tb * PPLD + r];
      Bs[ta * 17 + tb] -= acc;
    }
    __syncthreads();
    // (4) the 16 x 16 adjoint
    {
      double acc = 0.0;
      if (ta >= tb)
        for (int t = ta; t < 16; ++t) acc += Ls[t * 17 + ta] * Bs[t * 17 + tb];
      Ms[ta * 17 + tb] = (ta == tb) ? 0.5 * acc : acc;
    }
    if (tid < 16) {
      const int c = tid;
      for (int r = 0; r < 16; ++r) {
        double v = (r == c) ? 1.0 : 0.0;
        for (int t = c; t < r; ++t) v -= Ls[r * 17 + t] * Is[t * 17 + c];
        Is[r * 17 + c] = (r < c) ? 0.0 : v / Ls[r * 17 + r];
      }
    }
    __syncthreads();
    {
      double acc = 0.0;
      for (int t = 0; t < 16; ++t) acc += Ms[ta * 17 + t] * Is[t * 17 + tb];
      Ys[ta * 17 + tb] = acc;
    }
    __syncthreads();
    {
      double acc = 0.0;
      for (int t = 0; t < 16; ++t) acc += Is[t * 17 + ta] * Ys[t * 17 + tb];
      Gs[ta * 17 + tb] = acc;
    }
    __syncthreads();
    // (5) write: Q (both orientations) and the symmetric adjoint over Lbar
    if (ta < w && tb < w) {
      const double g = Gs[ta * 17 + tb] + Gs[tb * 17 + ta];  // P_ab + P_ba off the diagonal, 2 P_aa on it
      st_dev(Qkk + (int64_t)(c0 + tb) * ldq + c0 + ta, g);
      if (ta >= tb) st_dev(Bkk + (int64_t)(c0 + tb) * ld + c0 + ta, (ta == tb) ? Gs[ta * 17 + ta] : 0.5 * g);
    }
    for (int idx = tid; idx < w * (R - 16); idx += NT) {
      const int c = idx / (R - 16), r = 16 + idx - c * (R - 16);
      const double v = Ps[c * PPLD + r];
      st_dev(Qkk + (int64_t)(c0 + c) * ldq + c0 + r, v);
      st_dev(Bkk + (int64_t)(c0 + c) * ld + c0 + r, 0.5 * v);
    }
    for (int idx = tid; idx < w * (R - 16); idx += NT) {
      const int r = 16 + idx / w, c = idx - (r - 16) * w;
      st_dev(Qkk + (int64_t)(c0 + r) * ldq + c0 + c, Ps[c * PPLD + r]);
    }
    wait_vmcnt<0>();
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Adjoint of a diagonal tile in closed form.  For the tile factorization
// L_kk L_kk^T = A_kk and the adjoint Lbar_kk of its factor (after the
// partial products of its column), the adjoint with respect to the tile is
// the symmetric matrix S / 2 with
//     S = L^{-T} (M + M^T) L^{-1} = L^{-T} Y + Y^T L^{-1},   Y = M L^{-1},
// M = Phi(L^T Lbar) (Phi: the lower triangle with its diagonal halved); in
// lower-parameter form P_kk = tril(S) - diag(S) / 2, so Q_kk = S, and the
// output over Lbar_kk is tril(S) / 2.
// This is the panel recursion of the tile's adjoint summed in closed form
// (the same linear map; only the rounding differs), and it turns the long
// chain of 16-column panels into three products over TCHOL_PRB-order blocks
// that many workgroups share:
//   PADJM: Mn = -M by lower blocks, from LT (L^T) and Lbar_kk^T (which
//          DRED(k) leaves in the Q_kk tile)
//   PADJY: Y^T = L^{-T} Mn^T negated, i.e. (M L^{-1})^T, by upper blocks
//   PADJS: S by lower blocks, stored to Q_kk in both orientations and,
//          halved, to the lower triangle of Lbar_kk
// L^{-T} comes from TRTRI(k) (upper triangular, exact zeros below).  Every
// product is C = -A B^T from a zero start (the matrix cores' primitive);
// the negated M absorbs the first sign, the second cancels it, and the
// third is undone at the store.  Zero regions: the products' K ranges
// skip the blocks that vanish by triangularity, and inside the diagonal
// blocks the stored zeros (of Mn above its diagonal, of L^{-T} below, of
// Lbar^T below) make the rest exact.
#define PRB TCHOL_PRB

// C = -(A0 B0^T [+ A1 B1^T]) for one PRB x PRB block (M, N <= PRB, K a multiple
// of 16; the A panels at ld, the B panels at ldb, default ld); with Cinit the
// products are subtracted from C (read at ldc) instead of from zero.
// epi(row, col, value) stores each entry.  SEG as for gemm_core (128 needs
// even leading dimensions and 16-byte aligned panels).
template <int SEG = 128, class Epi>
__device__ __forceinline__ void padj_block(const double* A0, const double* B0, const double* A1, const double* B1,
                                           int64_t ld, int M, int N, int K, double* lds, Epi epi, int64_t ldb = -1,
                                           const double* Cinit = nullptr, int64_t ldc = 0) {
  using S = GemmShape<PRB, PRB, 16, 2, 4, 0>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WGN, wn = wave % S::WGN;
  const int l16 = lane & 15, lg = lane >> 4;
  d4 acc[S::RB][S::CB];
#pragma unroll
  for (int rb = 0; rb < S::RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < S::CB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * S::WTM + rb * 16 + l16, col = wn * S::WTN + cb * 16 + 4 * i + lg;
        acc[rb][cb][i] = Cinit ? Cinit[(int64_t)imin(col, N - 1) * ldc + imin(row, M - 1)] : 0.0;
      }
  gemm_kloop<PRB, PRB, 16, 2, 4, 0, SEG>(acc, A0, B0, ld, M, N, K, lds, ldb);
  if (A1 != nullptr) {
    __syncthreads();  // the stages are refilled only after every wavefront's last reads
    gemm_kloop<PRB, PRB, 16, 2, 4, 0, SEG>(acc, A1, B1, ld, M, N, K, lds, ldb);
  }
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < S::RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < S::CB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * S::WTM + rb * 16 + l16, col = wn * S::WTN + cb * 16 + 4 * i + lg;
        if (row < M && col < N) epi(row, col, acc[rb][cb][i]);
      }
}

// TREV(i, k) work item through the tile's explicit inverse: rows r0 ..
// r0 + M - 1 of P_ik = Lbar_ik L_kk^{-1}, with L_kk^{-T} (IT, ld nb, upper
// triangular) from TRTRI(k).  Lb: those rows of Lbar_ik (ld); P(:, c) reads
// the columns of Lbar from c on, so the column blocks go left to right and
// each is written (P / 2 over Lbar, P into Q_ik at Qik and P^T into Q_ki at
// Qki, both ld ldq) after its own product has read it.  SEG = 128 needs Lb
// 16-byte aligned with an even ld; 32 serves the rest.
template <int SEG>
__device__ __forceinline__ void trev_rows(double* __restrict__ Lb, int64_t ld, const double* __restrict__ IT, int64_t nb,
                                          int M, int m, double* __restrict__ Qik, double* __restrict__ Qki,
                                          int64_t ldq, double* lds) {
  for (int c0 = 0; c0 < m; c0 += PRB) {
    padj_block<SEG>(Lb + (int64_t)c0 * ld, IT + (int64_t)c0 * nb + c0, nullptr, nullptr, ld, M, imin(PRB, m - c0),
                    m - c0, lds,
                    [&](int r, int c, double v) __attribute__((always_inline)) {
                      const double p = -v;
                      st_dev(Lb + (int64_t)(c0 + c) * ld + r, 0.5 * p);
                      st_dev(Qik + (int64_t)(c0 + c) * ldq + r, p);
                      st_dev(Qki + (int64_t)r * ldq + c0 + c, p);
                    },
                    nb);
  }
}

// Block (bi, bj), bi >= bj, of the lower triangle from a work item's part.
__device__ __forceinline__ void lower_block(int part, int& bi, int& bj) {
  bi = 0;
  while ((bi + 1) * (bi + 2) / 2 <= part) ++bi;
  bj = part - bi * (bi + 1) / 2;
}

// One work item of PADJM / PADJY / PADJS on tile k of order m (a multiple of
// 16).  LTkk, Qkk: the tile of L^T and of Q (ld ldq); Bkk: Lbar_kk (ld);
// IT: L_kk^{-T}, Mn and YT: the tile's scratch blocks (ld nb).
__device__ __forceinline__ void padj_item(int kind, int part, int m, const double* __restrict__ LTkk,
                                          double* __restrict__ Qkk, int64_t ldq, double* __restrict__ Bkk, int64_t ld,
                                          const double* __restrict__ IT, double* __restrict__ Mn,
                                          double* __restrict__ YT, int64_t nb, double* lds) {
  int bi, bj;
  lower_block(part, bi, bj);
  const int i0 = bi * PRB, j0 = bj * PRB;
  const int Mi = imin(PRB, m - i0), Nj = imin(PRB, m - j0);
  if (kind == TK_PADJM) {
    // Mn(i, j) = -sum_{t >= i} L^T(i, t) Lbar^T(j, t), diagonal halved, zero above it
    padj_block(LTkk + (int64_t)i0 * ldq + i0, Qkk + (int64_t)i0 * ldq + j0, nullptr, nullptr, ldq, Mi, Nj, m - i0,
               lds, [&](int r, int c, double v) __attribute__((always_inline)) {
                 if (bi == bj) v = r > c ? v : (r == c ? 0.5 * v : 0.0);
                 st_dev(Mn + (int64_t)(j0 + c) * nb + i0 + r, v);
               });
  } else if (kind == TK_PADJY) {
    // Y^T(j, i) = -sum_{j <= t <= i} L^{-T}(j, t) Mn(i, t), the block of rows j0 and columns i0
    const int kend = imin(i0 + PRB, m);
    padj_block(IT + (int64_t)j0 * nb + j0, Mn + (int64_t)j0 * nb + i0, nullptr, nullptr, nb, Nj, Mi, kend - j0, lds,
               [&](int r, int c, double v) __attribute__((always_inline)) {
                 st_dev(YT + (int64_t)(i0 + c) * nb + j0 + r, v);
               });
  } else {
    // S(i, j) = sum_{t >= i} L^{-T}(i, t) Y^T(j, t) + Y^T(i, t) L^{-T}(j, t), lower entries
    padj_block(IT + (int64_t)i0 * nb + i0, YT + (int64_t)i0 * nb + j0, YT + (int64_t)i0 * nb + i0,
               IT + (int64_t)i0 * nb + j0, nb, Mi, Nj, m - i0, lds,
               [&](int r, int c, double v) __attribute__((always_inline)) {
                 const int i = i0 + r, j = j0 + c;
                 if (i >= j) {
                   const double s = -v;
                   st_dev(Qkk + (int64_t)j * ldq + i, s);
                   st_dev(Qkk + (int64_t)i * ldq + j, s);
                   st_dev(Bkk + (int64_t)j * ld + i, 0.5 * s);
                 }
               });
  }
}

// Adjoint preparation: LT := L^T over the padded order np (LT(c, t) = L(t, c)
// at t * ldq + c, zero outside the lower triangle of the n x n factor), and
// the padding rows and columns of Q set to zero.  32 x 32 tiles through LDS.
__global__ void tchol_backward_prep(const double* __restrict__ L, int64_t n, double* __restrict__ LT,
                                    double* __restrict__ Q, int64_t ldq, int64_t np) {
  __shared__ double t32[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
  const int64_t c0 = (int64_t)blockIdx.x * 32, t0 = (int64_t)blockIdx.y * 32;
  // read L(t0 + j, c0 + i) for i = row of the transposed tile: columns c of L, rows t contiguous
  for (int i = ty; i < 32; i += 8) {
    const int64_t c = c0 + i, t = t0 + tx;
    t32[i][tx] = (c < n && t < n && t >= c) ? L[c * n + t] : 0.0;
  }
  __syncthreads();
  for (int j = ty; j < 32; j += 8) {
    const int64_t t = t0 + j, c = c0 + tx;
    if (t < np && c < np) LT[t * ldq + c] = t32[tx][j];
  }
  // Q padding: rows or columns at or past n
  for (int j = ty; j < 32; j += 8) {
    const int64_t t = t0 + j, r = c0 + tx;
    if (t < np && r < np && (t >= n || r >= n)) Q[t * ldq + r] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// scheduler
__device__ __forceinline__ int ld_relaxed(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int64_t tile_size(int64_t n, int64_t nb, int t) {
  const int64_t r = n - (int64_t)t * nb;
  return r < nb ? r : nb;
}

__device__ __forceinline__ int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Executed by a whole wavefront with every decision made wave-uniform
// (readfirstlane), so the compiler keeps the control flow scalar: a barrier
// must never end up inside lane-masked loop structure.  Waits until the
// task's counter reaches zero; false when the run is being aborted or the
// wait exceeded its bound.
// one (not null): a single-matrix launch's failure word, read along with the
// first look (and again after a wait) into failed.  early(), asked when the
// first look finds the task not ready: true to go on without waiting (the work
// item then waits itself).
template <class Early>
__device__ __forceinline__ bool wait_ready(const KArgs& a, int task, int lane, const int32_t* one, int& failed,
                                           Early early) {
  const int dep0 = ld_relaxed(&a.dep[task]), abort0 = ld_relaxed(&a.hdr[HDR_ABORT]);  // all in flight at once
  const int f0 = one ? ld_relaxed(one) : 0;
  failed = uniform_i(f0);
  if (uniform_i(dep0) == 0) return uniform_i(abort0) == 0;
  if (uniform_i(abort0) == 0 && early()) return true;
  const uint64_t t0 = wall_clock64();
  for (int poll = 0;; ++poll) {
    __builtin_amdgcn_s_sleep(2);
    // the counter and the failure word in flight together: one round trip per
    // poll; the abort flag, in a line that every waiting worker would read and
    // the tickets are drawn from, on every eighth (a task that is ready may run)
    const int d = ld_relaxed(&a.dep[task]), f = one ? ld_relaxed(one) : 0;
    failed = uniform_i(f);
    if (uniform_i(d) == 0) return true;
    if ((poll & 7) != 7) continue;
    if (uniform_i(ld_relaxed(&a.hdr[HDR_ABORT])) != 0) return false;
    if ((int64_t)(wall_clock64() - t0) > a.wait_limit) {
      if (lane == 0) {
        __hip_atomic_store(&a.hdr[HDR_ERROR], DEV_ERR_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.hdr[HDR_ABORT], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      }
      return false;
    }
  }
}

// Stops every worker with a runtime error code (the first one is kept).
__device__ __forceinline__ void raise_error(const KArgs& a, int code) {
  if (threadIdx.x == 0) {
    int expected = 0;
    __hip_atomic_compare_exchange_strong(&a.hdr[HDR_ERROR], &expected, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a.hdr[HDR_ABORT], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------------------------
// POTRF split over several workgroups.  A diagonal tile of order m > 128 is
// factored as its own small tile Cholesky DAG over 128 x 128 sub-blocks
// (T2 = ceil(m / 128) per side):
//   P(b)        chol of sub-block (b, b)                  (potrf_small)
//   S(r, b, s)  32-row strip s of sub-block (r, b) := . L_bb^{-T}, r > b   (trsm_strip)
//   U(r, c, b, s)  64 x 64 block s of sub-block (r, c) -= L_rb L_cb^T, r >= c > b  (gemm_reg64:
//               10 us where a whole 128 x 128 sub-block takes gemm_tile 24)
// The POTRF task has several work items; each one that starts joins the
// tile's pool: the worker takes the next sub-unit from a counter in the
// workspace, waits for that unit's predecessors through per-sub-block
// counters, runs it through the same tile bodies as whole tasks and
// publishes it (write-through stores, then the counter), until no unit is
// left; then its work item is done.  Units are handed out in a topological order, so the oldest
// unfinished unit always has its predecessors finished or running, and a
// single work item drains the pool alone if no other joins: no workgroup
// ever waits for one that has not started.  Updates of a sub-block are
// applied in order of b, so the factor does not depend on which workgroup
// runs what.
#define PSB 128        // sub-block order
#define PL_NEXT 0      // next unit to hand out
#define PL_P 2         // + b: P(b) done
#define PL_S 8         // + 4 r + b: strips of S(r, b) done
#define PL_U 24        // + 4 r + c: blocks of updates applied to sub-block (r, c)
#define PL_INV 44      // items of the tile's TRTRI done
// A unit that failed, or was skipped in a launch in which a failing system
// stops only its own work, adds PL_FAILED to its counter as well: the units that
// wait for it find out with the wait, and are skipped too.
#define PL_FAILED 0x10000

struct PoolUnit {
  int type, b, r, c, s;  // type 0: P(b); 1: S(r, b, s); 2: U(r, c, b, s); -1: none left
};

__device__ __forceinline__ int psb_size(int m, int i) { return imin(PSB, m - i * PSB); }
__device__ __forceinline__ int psb_strips(int m, int i) { return (psb_size(m, i) + TS - 1) / TS; }

// Blocks of an update of sub-block (r, c), r >= c: 64 x 64, of a diagonal
// one the lower blocks, row by row.
__device__ __forceinline__ int psb_blocks(int m, int r, int c) {
  const int nr = psb_size(m, r) > 64 ? 2 : 1, nc = psb_size(m, c) > 64 ? 2 : 1;
  return r == c ? nr * (nr + 1) / 2 : nr * nc;
}
// Unit u of the sub-DAG in claim order: step by step, P(b), then the strips
// of each sub-block row below it, then its updates column by column (the
// next diagonal sub-block's first: it leads to P(b + 1)).
__device__ __forceinline__ PoolUnit pool_unit(int m, int u) {
  const int T2 = (m + PSB - 1) / PSB;
  for (int b = 0; b < T2; ++b) {
    if (u == 0) return {0, b, b, b, 0};
    --u;
    for (int r = b + 1; r < T2; ++r) {
      const int ns = psb_strips(m, r);
      if (u < ns) return {1, b, r, b, u};
      u -= ns;
    }
    for (int c = b + 1; c < T2; ++c)
      for (int r = c; r < T2; ++r) {
        const int nu = psb_blocks(m, r, c);
        if (u < nu) return {2, b, r, c, u};
        u -= nu;
      }
  }
  return {-1, 0, 0, 0, 0};
}

// Wavefront 0: waits until pool[q0] >= v0, pool[q1] >= v1 and pool[q2] >= v2
// (agent-scope loads, s_sleep back-off); false on abort or when the wait
// exceeds its bound (which then raises TCHOL_E_TIMEOUT like a task wait).
// failed: set when a unit counted there was one (PL_FAILED).
__device__ __forceinline__ bool pool_wait(const KArgs& a, const int32_t* pool, int q0, int v0, int q1, int v1, int q2,
                                          int v2, int lane, int& failed) {
  // the three counters and the abort flag in flight together: one round trip per poll
  int ab = 0;
  auto met = [&]() __attribute__((always_inline)) {
    const int x0 = ld_relaxed(pool + q0), x1 = ld_relaxed(pool + q1), x2 = ld_relaxed(pool + q2);
    ab = uniform_i(ld_relaxed(&a.hdr[HDR_ABORT]));
    constexpr int count = PL_FAILED - 1;
    const bool all = uniform_i(((x0 & count) >= v0) & ((x1 & count) >= v1) & ((x2 & count) >= v2)) != 0;
    if (all && uniform_i(x0 | x1 | x2) >= PL_FAILED) failed = 1;
    return all;
  };
  if (met()) return ab == 0;
  const uint64_t t0 = wall_clock64();
  for (;;) {
    __builtin_amdgcn_s_sleep(2);
    if (met()) return ab == 0;
    if (ab != 0) return false;
    if ((int64_t)(wall_clock64() - t0) > a.wait_limit) {
      if (lane == 0) {
        __hip_atomic_store(&a.hdr[HDR_ERROR], DEV_ERR_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.hdr[HDR_ABORT], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      }
      return false;
    }
  }
}

// Wavefront 0: waits for the predecessors of pool unit pu of a tile of order m.
__device__ __forceinline__ bool pool_wait_unit(const KArgs& a, const int32_t* pool, int m, const PoolUnit& pu,
                                               int lane, int& failed) {
  // sub-block (r, c) updated b times (c = b for P and S)
  const int nu = pu.b * psb_blocks(m, pu.r, pu.c);
  if (pu.type == 0)  // P(b): the diagonal sub-block has taken its b updates
    return pool_wait(a, pool, PL_U + 5 * pu.b, nu, PL_U + 5 * pu.b, nu, PL_U + 5 * pu.b, nu, lane, failed);
  if (pu.type == 1)  // S(r, b, s): L_bb factored, sub-block (r, b) updated b times
    return pool_wait(a, pool, PL_P + pu.b, 1, PL_U + 4 * pu.r + pu.b, nu, PL_P + pu.b, 1, lane, failed);
  // U(r, c, b): every strip of (r, b) and (c, b) solved, (r, c) updated b times
  return pool_wait(a, pool, PL_S + 4 * pu.r + pu.b, psb_strips(m, pu.r), PL_S + 4 * pu.c + pu.b,
                   psb_strips(m, pu.c), PL_U + 4 * pu.r + pu.c, nu, lane, failed);
}

// SEG = 128: the launch guarantees even leading dimensions, 16-byte aligned
// matrices and, for odd orders, a leading dimension above the order, so
// every panel the updates stream is 16-byte transferable; SEG = 32 serves
// every other case.  One transfer width per kernel instance keeps the
// update loops free of per-item branches.
// MODE 4: the batched FP32 launch: the mixed-precision factor kinds and
// the solve kinds with substitution against the FP64 diagonal tiles (one
// solve of a few right-hand sides does not repay explicit inverses).
// MODE 0: FP64 factorization and solve.  MODE 1 / 2: the mixed-precision
// factorization / its solves: the matrix is the FP32 working copy (a.A points
// to it), factored with FP32 MFMA updates and FP64 diagonal tiles kept in
// a.D; solves run in FP64 reading L in FP32 off the diagonal and in FP64 on
// it.  MODE 5: the mixed-precision factorization with BF16 updates: as
// MODE 1, with the TRSM strips also storing their results as three BF16
// terms (a.H) and the GEMM items running on the BF16 matrix cores over them.
// A mixed launch runs only its own task kinds (keeping each instance small)
// and is always a 16-byte one.
template <int SEG, int MODE>
__global__ void __launch_bounds__(NT, MODE >= 6 ? 2 : 1) tchol_persistent(KArgs a) {
  constexpr bool MIXED = MODE == 1 || MODE == 2 || MODE == 4 || MODE == 5;
  constexpr bool FACTOR_KINDS = MODE == 0 || MODE == 1 || MODE == 4 || MODE == 5;
  constexpr bool SOLVE_KINDS = MODE == 0 || MODE == 2 || MODE == 4;
  constexpr bool ADJOINT_KINDS = MODE == 3;
  // The FP64 and mixed-precision factorizations split large POTRF tasks
  // over their work items (the tile's pool of sub-units; the mixed one on
  // its FP64 diagonal tile); the batched FP32 instance factors each diagonal
  // tile on one workgroup (only part 0 of a POTRF task works)
  constexpr bool POOLED = MODE == 0 || MODE == 1 || MODE == 5;
  // MODE 6 (batched systems of one tile each): the compact POTRF and tile
  // solves only, in half the LDS, two workgroups per compute unit; MODE 7 the
  // same with each system's matrix read from and L written to FP32 storage
  // (A32, the FP64 tile in A for the products and the solves)
  static_assert(FRB_COMPACT_DOUBLES <= LDS_COMPACT_DOUBLES && PT_LDS_COMPACT <= LDS_COMPACT_DOUBLES, "compact LDS budget");
  constexpr bool COMPACT = MODE == 6 || MODE == 7;
  __shared__ double lds[COMPACT ? LDS_COMPACT_DOUBLES : LDS_DOUBLES];
  __shared__ int s_claim[6];
  // what wavefront 0 finds out after the claim: whether the item's system has
  // failed, the outcome of a late wait (the claim's words stay as they were claimed)
  __shared__ int s_word;
  __shared__ int32_t s_desc[DESC_WORDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform_i(tid >> 6);
  // wavefront 0's record of the work item it ran last, published at the
  // start of the next claim, and of the items this worker completed
  int p_task = -1, p_ticket = 0, p_parts = 0, p_e0 = 0, p_e1 = 0, ndone = 0;
  bool p_fwd = false;  // it was an item of the last FTRSV
  uint64_t p_end = 0;
  // wavefront 0: the POTRF pool this worker serves (pl_task < 0: none) and
  // the POTRF work item's record, published when the pool has run dry
  int pl_task = -1, pl_m = 0, pl_ticket = 0, pl_parts = 0, pl_e0 = 0, pl_e1 = 0;
  int pl_failed = 0;  // the system had failed when this worker joined the pool
  int32_t* pl_pool = nullptr;
  // a launch of one matrix (nsys <= 2: its factor's and its solve's tile size)
  // keeps the system records in LDS and has one failure word, which the claim
  // reads along with the task's counter: fewer round trips before an item starts
  __shared__ int64_t s_sys[2 * SYS_WORDS];
  const bool one_matrix = !COMPACT && a.nsys <= 2 && (a.nsys == 1 || a.batched == 2);
  if (one_matrix && tid < a.nsys * SYS_WORDS) s_sys[tid] = a.sys[tid];
  const int32_t* const one_failed = one_matrix && a.batched ? a.sinfo : nullptr;
  for (;;) {
    // publish + claim: wavefront 0 marks the previous item done and takes the
    // next ticket in the same round trip, then waits for the new task while
    // its descriptor is fetched.  A worker in a POTRF pool takes the pool's
    // next sub-unit instead, and returns to the tickets when none is left.
    if (wave == 0) {
      int task = -1, part = 0, unit = -1, t = 0, failed = 0, early = 0;
      bool claimed = false;
      uint64_t tw = 0;
      if (POOLED && pl_task >= 0) {
        int u = 0;
        if (lane == 0) u = __hip_atomic_fetch_add(pl_pool + PL_NEXT, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        u = uniform_i(u);
        const PoolUnit pu = pool_unit(pl_m, u);
        if (pu.type >= 0) {
          claimed = true;
          task = pl_task;
          t = pl_ticket;
          unit = u;
          failed = pl_failed;
          if (!pool_wait_unit(a, pl_pool, pl_m, pu, lane, failed)) task = -1;
        } else {
          // the pool has run dry: this worker's POTRF work item is complete
          p_task = pl_task;
          p_ticket = pl_ticket;
          p_parts = pl_parts;
          p_e0 = pl_e0;
          p_e1 = pl_e1;
          if (a.trace) p_end = wall_clock64();
          pl_task = -1;
        }
      }
      if (!claimed) {
        int prev = 0;
        if (lane == 0) {
          if (p_task >= 0)
            prev = __hip_atomic_fetch_add(&a.done[p_task], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          t = __hip_atomic_fetch_add(&a.hdr[HDR_TICKET], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (p_task >= 0) {
          // the last work item of a task activates its successors
          if (uniform_i(prev) == p_parts - 1) {
            for (int e = p_e0 + lane; e < p_e1; e += 64)
              __hip_atomic_fetch_sub(&a.dep[a.succ[e]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (SOLVE_KINDS && p_fwd && lane == 0)
              __hip_atomic_store(&a.hdr[HDR_FWD], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          ++ndone;
          if (a.trace && lane == 0) {
            a.trace[4 * (int64_t)p_ticket + 2] = p_end;
            a.trace[4 * (int64_t)p_ticket + 3] = (uint64_t)(uint32_t)p_task | ((uint64_t)(uint32_t)blockIdx.x << 32);
          }
          p_task = -1;
        }
        t = uniform_i(t);
        if (t < a.nitem) {
          task = uniform_i(a.items[2 * t]);
          part = uniform_i(a.items[2 * t + 1]);
          if (a.trace) tw = wall_clock64();
          const int dv = lane < DESC_WORDS ? a.desc[DESC_WORDS * (int64_t)task + lane] : 0;
          // A strip of the solve whose L (or inverse) is already final starts
          // before its right-hand sides are: it requests L, then waits.  L is
          // final from the start in a launch that only solves, and everywhere once
          // the last FTRSV is done (HDR_FWD); a diagonal tile's inverse once
          // its TRTRI items have counted up its pool word.  Faster at every tile
          // size: a solve alone takes, without / with it, 156 / 141 us at n = 300 and
          // tiles of 64, 247 / 212 us at 1024 and 128, 631 / 475 us at 4096 and 256,
          // 2.27 / 1.73 ms at 16384 and 512; merged at n = 300 and 64 247 us both ways.
          auto early_ok = [&]() __attribute__((always_inline)) {
            if constexpr (!SOLVE_KINDS || MODE == 4) return false;
            if (!one_matrix) return false;
            const int kd = uniform_i(__builtin_amdgcn_readlane(dv, 0)), pd = uniform_i(__builtin_amdgcn_readlane(dv, 4));
            bool ok = false;
            if (kd == TK_FGEMV) {
              ok = a.lfinal != 0;
            } else if (kd == TK_BGEMV) {
              ok = a.lfinal != 0 || uniform_i(ld_relaxed(&a.hdr[HDR_FWD])) != 0;
            } else if ((kd == TK_FTRSV || kd == TK_BTRSV) && pd > 1) {  // by strips, with the tile's inverse
              if (MODE == 2) {
                ok = true;
              } else {
                const int tkd = uniform_i(__builtin_amdgcn_readlane(dv, 3)), sd = uniform_i(__builtin_amdgcn_readlane(dv, 7));
                const int64_t* srd = s_sys + SYS_WORDS * sd;
                const int m = (int)tile_size(srd[2], srd[3], tkd);
                ok = uniform_i(ld_relaxed(a.pool + POOL_WORDS * (srd[6] + tkd) + PL_INV)) ==
                     uniform_i((m + a.trsm_rows - 1) / a.trsm_rows);
              }
            }
            early = ok ? 1 : 0;
            return ok;
          };
          if (!wait_ready(a, task, lane, one_failed, failed, early_ok)) task = -1;
          if (lane < DESC_WORDS) s_desc[lane] = dv;
          const int kd = uniform_i(__builtin_amdgcn_readlane(dv, 0)), pd = uniform_i(__builtin_amdgcn_readlane(dv, 4));
          if (POOLED && task >= 0 && kd == TK_POTRF && pd > 1) {
            // a work item of a split POTRF: join the tile's pool
            const int tkd = uniform_i(__builtin_amdgcn_readlane(dv, 3)), sd = uniform_i(__builtin_amdgcn_readlane(dv, 7));
            const int64_t* srd = a.sys + SYS_WORDS * (int64_t)sd;
            pl_task = task;
            pl_m = (int)tile_size(srd[2], srd[3], tkd);
            pl_pool = a.pool + POOL_WORDS * (srd[6] + tkd);
            pl_ticket = t;
            pl_parts = pd;
            pl_failed = failed;
            pl_e0 = uniform_i(__builtin_amdgcn_readlane(dv, 5));
            pl_e1 = uniform_i(__builtin_amdgcn_readlane(dv, 6));
            int u = 0;
            if (lane == 0) u = __hip_atomic_fetch_add(pl_pool + PL_NEXT, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            u = uniform_i(u);
            const PoolUnit pu = pool_unit(pl_m, u);
            if (pu.type >= 0) {
              unit = u;
              if (!pool_wait_unit(a, pl_pool, pl_m, pu, lane, failed)) task = -1;
            } else {
              unit = -2;  // the pool ran dry before this item started: nothing to do
              pl_task = -1;
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (lane == 0) {
        s_claim[0] = task;
        s_claim[1] = part;
        s_claim[2] = t;
        s_claim[3] = unit;
        s_claim[4] = failed;
        s_claim[5] = early;
        if (a.trace && task >= 0 && !claimed) {
          a.trace[4 * (int64_t)t + 0] = tw;
          a.trace[4 * (int64_t)t + 1] = wall_clock64();
        }
        // the completed-item count, added once per worker
        if (task < 0 && ndone > 0)
          __hip_atomic_fetch_add(&a.hdr[HDR_DONE], ndone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __syncthreads();
    const int task = uniform_i(s_claim[0]), part = uniform_i(s_claim[1]), ticket = uniform_i(s_claim[2]);
    const int unit = uniform_i(s_claim[3]);
    if (task < 0) break;
    const int kind = uniform_i(s_desc[0]), ti = uniform_i(s_desc[1]), tj = uniform_i(s_desc[2]),
              tk = uniform_i(s_desc[3]);
    const int d_parts = uniform_i(s_desc[4]), d_e0 = uniform_i(s_desc[5]), d_e1 = uniform_i(s_desc[6]);
    // the task's system: base pointers, order, tile size, leading dimension
    const int sid = uniform_i(s_desc[7]);
    int64_t sr[SYS_WORDS];
    if (one_matrix) {
#pragma unroll
      for (int i = 0; i < SYS_WORDS; ++i) {
        const int64_t v = s_sys[SYS_WORDS * sid + i];
        sr[i] = ((int64_t)uniform_i((int)(v >> 32)) << 32) | (int64_t)(uint32_t)uniform_i((int)v);
      }
    } else {
#pragma unroll
      for (int i = 0; i < SYS_WORDS; ++i) sr[i] = a.sys[SYS_WORDS * (int64_t)sid + i];
    }
    using E = typename std::conditional<MIXED, float, double>::type;
    E* const Abase = reinterpret_cast<E*>(a.A) + sr[0];
    double* const Bbase = a.B + sr[1];
    const int64_t sn = sr[2], nb = sr[3], ld = sr[4], ldb = sn;
    // mixed precision: the system's FP64 diagonal tiles and their inverses
    double* const Dsys = a.D + (MIXED ? sr[5] : 0);
    double* const DinvSys = a.Dinv + sr[5];
    double* const DinvTSys = a.DinvT + sr[5];
    auto tsz = [&](int t) __attribute__((always_inline)) { return (int)tile_size(sn, nb, t); };
    // the solve's diagonal step on tile t applies explicit inverses (and keeps
    // y in the scratch vector): always in the mixed-precision solves; in the
    // FP64 solve of a launch that computes them (their tiles' orders are
    // multiples of 16), else substitution in place
    auto inv_tile = [&](int t) __attribute__((always_inline)) {
      return MODE == 2 || (MODE == 0 && a.inv != 0 && (tsz(t) & 15) == 0);
    };
    // in a batched launch a system whose factorization failed only passes
    // its remaining tasks on, so that the DAG drains
    // (one read for the whole workgroup, whose wavefronts must agree while
    // another one may be storing the word: a single matrix's came with the
    // claim.  In the compact instance a system's tasks follow one another, and
    // every wavefront that loads the word finds the same.)
    bool skip;
    if (COMPACT) {
      skip = uniform_i(ld_relaxed(&a.sinfo[sid])) != 0;
    } else if (one_matrix) {
      skip = uniform_i(s_claim[4]) != 0;
    } else {
      if (wave == 0) {
        const int f = ld_relaxed(&a.sinfo[sid]);
        if (lane == 0) s_word = f;
      }
      lds_barrier();
      skip = uniform_i(s_word) != 0;
    }
    int ok = 1;
    // the wait of a strip that was claimed early (all wavefronts): false when the run is being aborted
    const bool was_early = uniform_i(s_claim[5]) != 0;
    auto late = [&]() __attribute__((always_inline)) {
      if (!was_early) return true;
      if (wave == 0) {
        int f;
        const bool go = wait_ready(a, task, lane, nullptr, f, []() __attribute__((always_inline)) { return false; });
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (lane == 0) {
          s_word = go;
          if (a.trace) a.trace[4 * (int64_t)ticket + 1] = wall_clock64();
        }
      }
      lds_barrier();
      const bool go = uniform_i(s_word) != 0;
      if (!go) ok = 0;
      return go;
    };
    int unit_failed = skip;
    int count_inv = 0;  // a TRTRI item of an FP64 launch counts up its tile's pool word
    // A unit of a POTRF pool runs the POTRF, TRSM or GEMM body on sub-blocks
    // of the diagonal tile (tk, tk): po_* give the sub-block offsets (rows,
    // columns, panel columns) and sizes; whole tasks take the tile's.
    int body = kind;
    int po_r = 0, po_c = 0, po_k = 0, po_m = 0, po_n = 0, po_kk = 0, po_s = 0;
    PoolUnit pu = {-1, 0, 0, 0, 0};
    if (POOLED && unit >= 0) {
      const int m = tsz(tk);
      pu = pool_unit(m, unit);
      body = pu.type == 0 ? TK_POTRF : (pu.type == 1 ? TK_TRSM : TK_GEMM);
      po_r = pu.r * PSB;
      po_c = pu.c * PSB;
      po_k = pu.b * PSB;
      po_m = psb_size(m, pu.r);
      po_n = psb_size(m, pu.c);
      po_kk = psb_size(m, pu.b);
      po_s = pu.s;
    } else if (POOLED && unit == -2) {
      body = -1;
    }
    if constexpr (COMPACT) {
      const bool fuse_fwd = a.nrhs > 0 && a.nrhs <= PT_FWD;
      if (skip) {
      } else if (kind == TK_POTRF) {
        // up to PT_FWD right-hand sides: the forward solve rides along (its FTRSV task only passes the completion on)
        // MODE 7: the system's FP32 matrix at A32 + sr[5], leading dimension sr[7]
        const int info = uniform_i(potrf_slabs<MODE == 7>(
            Abase + (tk * nb) * ld + tk * nb, ld, tsz(tk), lds, fuse_fwd ? Bbase + tk * nb : nullptr, ldb,
            (int)a.nrhs, MODE == 7 ? a.A32 + sr[5] + (tk * nb) * sr[7] + tk * nb : nullptr, sr[7]));
        if (info != 0 && tid == 0)
          __hip_atomic_store(&a.sinfo[sid], (int)(tk * nb) + info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (kind == TK_BTRSV || (kind == TK_FTRSV && !fuse_fwd)) {
        tile_solve<true>(Abase + (tk * nb) * ld + tk * nb, ld, Bbase + tk * nb, ldb, tsz(tk), (int)a.nrhs,
                         kind == TK_BTRSV, lds);
      } else if (kind != TK_FTRSV) {
        ok = 0;
      }
    } else switch (skip ? -1 : body) {
      case -1:
        break;
      case TK_POTRF: {
        if constexpr (!FACTOR_KINDS) {
          ok = 0;
          break;
        }
        // tiles of order <= 128 are factored by one workgroup in LDS; larger
        // ones through the tile's pool of sub-units when the task has several
        // work items (the plan's choice), else by the one-workgroup kernel
        int info;
        if constexpr (MIXED) {
          double* const Dk = Dsys + (int64_t)tk * nb * nb;
          if (POOLED && unit >= 0) {
            // P(b) on the FP64 diagonal tile; the last one pads a ragged tile
            // to a multiple of 16 with the identity (for its inverse)
            double* const Db = Dk + (int64_t)po_k * nb + po_k;
            if constexpr (MODE == 5)
              info = uniform_i(potrf_columns(Db, nb, po_m, lds));
            else
              info = uniform_i(potrf_small(Db, nb, po_m, lds));
            if (info != 0) {
              info += po_k;
            } else if (po_k + po_m == tsz(tk)) {
              const int m = tsz(tk), mpad = (m + 15) & ~15;
              for (int idx = tid; idx < mpad * mpad; idx += NT) {
                const int c = idx / mpad, r = idx - c * mpad;
                if (r >= c && (r >= m || c >= m)) st_dev(Dk + (int64_t)c * nb + r, r == c ? 1.0 : 0.0);
              }
            }
          } else {
            if (part > 0) break;  // one workgroup factors the tile
            info = uniform_i(potrf_tile_mixed<MODE == 5>(Dk, nb, tsz(tk), lds));
          }
        } else {
          const bool sub = unit >= 0;
          const int m = sub ? po_m : tsz(tk);
          E* Akk = Abase + (tk * nb + po_k) * ld + tk * nb + po_k;
          // a whole tile's inverse comes along when the launch's TRSMs apply it
          if (m <= PSB)
            info = uniform_i(potrf_small(Akk, ld, m, lds, a.finv != 0 && !sub ? DinvSys + (int64_t)tk * nb * nb : nullptr, nb));
          else
            info = uniform_i(potrf_tile<SEG>(Akk, ld, m, lds));
          if (info != 0) info += po_k;
        }
        if (info != 0 && tid == 0) {
          if (a.batched) {
            // (the first failure stays: a later tile may be reached before it is seen there)
            int none = 0;
            __hip_atomic_compare_exchange_strong(&a.sinfo[sid], &none, (int)(tk * nb) + info, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          } else {
            __hip_atomic_store(&a.hdr[HDR_INFO], (int)(tk * nb) + info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.hdr[HDR_ABORT], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
        if (info != 0 && !a.batched) ok = 0;
        if (info != 0 && a.batched) unit_failed = 1;
        break;
      }
      case TK_TRSM: {
        if constexpr (!FACTOR_KINDS) {
          ok = 0;
          break;
        }
        if constexpr (MIXED) {
          double* const Dk = Dsys + (int64_t)tk * nb * nb;
          if (POOLED && unit >= 0) {
            // strip of sub-block (r, b) of the FP64 diagonal tile
            const int r0 = po_s * TS;
            trsm_strip(Dk + (int64_t)po_k * nb + po_r + r0, nb, Dk + (int64_t)po_k * nb + po_k, nb,
                       imin(TS, po_m - r0), po_kk, lds);
          } else {
            const int r0 = part * a.trsm_rows;
            const int S = imin(a.trsm_rows, tsz(ti) - r0);
            if constexpr (MODE == 5)  // the strip also as BF16 terms, for the BF16 updates (whole 32-column blocks)
              trsm_strip(Abase + (tk * nb) * ld + ti * nb + r0, ld, Dk, nb, S, tsz(tk), lds, nullptr, 0,
                         nb % 32 == 0 ? a.H + ((int64_t)tk * a.hrows + (int64_t)ti * nb + r0) * nb : nullptr, 16 * nb,
                         (int64_t)a.T * a.hrows * nb);
            else
              trsm_strip(Abase + (tk * nb) * ld + ti * nb + r0, ld, Dk, nb, S, tsz(tk), lds);
          }
        } else if (a.inv != 0 && unit < 0) {
          // a block of inv_rows rows of A_ik through L_kk^{-1} (from POTRF(k) with
          // finv, else from the launch's TRTRI(k))
          const int r0 = part * a.inv_rows, M = imin(a.inv_rows, tsz(ti) - r0);
          E* const Xr = Abase + (tk * nb) * ld + ti * nb + r0;
          const double* const Li = DinvSys + (int64_t)tk * nb * nb;
          if (tsz(tk) <= PSB)
            for (int r = 0; r < M; r += TS) trsm_inv_strip(Xr + r, ld, Li, nb, imin(TS, M - r), tsz(tk));
          else
            trsm_inv_rows<SEG>(Xr, ld, Li, nb, M, tsz(tk), lds);
        } else {
          // a strip of A_ik, or of sub-block (r, b) of the diagonal tile for a pool unit
          const bool sub = unit >= 0;
          const int rs = sub ? TS : a.trsm_rows;
          const int r0 = (sub ? po_s : part) * rs;
          const int64_t row0 = sub ? (int64_t)tk * nb + po_r + r0 : (int64_t)ti * nb + r0;
          const int S = imin(rs, (sub ? po_m : tsz(ti)) - r0);
          const int64_t col0 = (int64_t)tk * nb + po_k;
          trsm_strip(Abase + col0 * ld + row0, ld, Abase + col0 * ld + col0, ld, S, sub ? po_kk : tsz(tk), lds);
        }
        break;
      }
      case TK_SYRK:
      case TK_GEMM:
      case TK_GEMM2:
      case TK_GEMM4: {
        if constexpr (!FACTOR_KINDS) {
          ok = 0;
          break;
        }
        // the work item's output sub-tile: row block si of bm rows, column block sj of bn
        int si, sj, bm, bn;
        if (kind == TK_SYRK) {
          si = 0;
          while ((si + 1) * (si + 2) / 2 <= part) ++si;
          sj = part - si * (si + 1) / 2;
          bm = bn = a.syrk_b;
        } else {
          bm = kind == TK_GEMM ? a.gemm1_m : a.gemm_m;
          bn = kind == TK_GEMM ? a.gemm1_n : a.gemm_n;
          const int ncj = (tsz(tj) + bn - 1) / bn;
          si = part / ncj;
          sj = part % ncj;
        }
        int M = imin(bm, tsz(ti) - si * bm);
        int N = imin(bn, tsz(tj) - sj * bn);
        // a merged update streams the panel columns of its two or four steps,
        // which are adjacent in the matrix: one product with K = 2 nb or 4 nb
        int K = tsz(tk) * (kind == TK_GEMM2 ? 2 : kind == TK_GEMM4 ? 4 : 1);
        bool lower = kind == TK_SYRK && si == sj;
        int64_t crow = (int64_t)ti * nb + si * bm, ccol = (int64_t)tj * nb + sj * bn, kcol = (int64_t)tk * nb;
        int64_t brow = (int64_t)tj * nb + sj * bn;
        if (POOLED && unit >= 0) {
          // block (bi, bj) of sub-block (r, c) of the diagonal tile -= L_rb L_cb^T
          const int nc = po_n > 64 ? 2 : 1;
          const int bi = po_r == po_c ? (po_s + 1) >> 1 : po_s / nc, bj = po_r == po_c ? po_s >> 1 : po_s % nc;
          lower = po_r == po_c && bi == bj;
          po_r += 64 * bi;
          po_c += 64 * bj;
          bm = 64;
          M = imin(64, po_m - 64 * bi);
          N = imin(64, po_n - 64 * bj);
          K = po_kk;
          crow = (int64_t)tk * nb + po_r;
          ccol = (int64_t)tk * nb + po_c;
          kcol = (int64_t)tk * nb + po_k;
          brow = ccol;
        }
        E* C = Abase + ccol * ld + crow;
        const E* Ap = Abase + kcol * ld + crow;
        const E* Bp = Abase + kcol * ld + brow;
        const bool misaligned = ((reinterpret_cast<uintptr_t>(Ap) | reinterpret_cast<uintptr_t>(Bp)) & 15) != 0;
        if constexpr (MIXED) {
          if (POOLED && unit >= 0) {
            // the block on the FP64 diagonal tile, in FP64
            double* const Dk = Dsys + (int64_t)tk * nb * nb;
            double* const Cu = Dk + (int64_t)po_c * nb + po_r;
            const double* const Au = Dk + (int64_t)po_k * nb + po_r;
            const double* const Bu = Dk + (int64_t)po_k * nb + po_c;
            gemm_reg64(Cu, Au, Bu, nb, M, N, K, lower, MODE == 5);
            break;
          }
          // four rows per 16-byte lane: ld a multiple of 4 and three rows after the order
          if ((((int)ld & 3) != 0) || ld < sn + 3 || misaligned) {
            raise_error(a, DEV_ERR_LAYOUT);  // unreachable when the host honours the launch contract
            ok = 0;
            break;
          }
          if (kind == TK_SYRK)
            gemm_nt_f32_d(Dsys + (int64_t)ti * nb * nb + (int64_t)(sj * bn) * nb + si * bm, nb, Ap, Bp, ld, M, N,
                          tsz(tk), si == sj, lds);
          else if (MODE == 5 && bm == 256 && bn == 128 && tsz(tk) % 32 == 0)
            gemm_bf16x6_wide(C, ld, (const char*)(a.H + ((int64_t)tk * a.hrows + crow) * nb),
                             (const char*)(a.H + ((int64_t)tk * a.hrows + brow) * nb), 32 * nb,
                             2 * (int64_t)a.T * a.hrows * nb, 2 * a.hrows * nb, (int)nb / 32, M, N, K, lds);
          else if (bm == 256 && bn == 128 && tsz(tk) % 32 == 0)
            gemm_f32_wide<32, 3>(C, Ap, Bp, ld, M, N, K, lds);
          else  // 128-row products (a 256-row item whose K is not a multiple of 32 takes two)
            for (int r0 = 0; r0 < M; r0 += 128)
              gemm_nt_f32(C + r0, Ap + r0, Bp, ld, imin(128, M - r0), N, K, false, lds);
        } else {
          if (SEG == 128 && (((int)ld & 1) != 0 || (((M | N) & 1) != 0 && ld <= sn) || misaligned)) {
            raise_error(a, DEV_ERR_LAYOUT);  // unreachable when the host honours the launch contract
            ok = 0;
            break;
          }
          if (bm == 64 && K <= PSB)
            gemm_reg64(C, Ap, Bp, ld, M, N, K, lower);
          else
            gemm_nt<SEG>(C, Ap, Bp, ld, M, N, K, lower, lds);
        }
        break;
      }
      case TK_FTRSV:
      case TK_BTRSV:
        if constexpr (!SOLVE_KINDS) {
          ok = 0;
        } else if constexpr (MODE == 4) {
          // batched FP32 systems: substitution against the FP64 diagonal tile, in place
          tile_solve(Dsys + (int64_t)tk * nb * nb, nb, Bbase + tk * nb, ldb, tsz(tk), (int)a.nrhs, kind == TK_BTRSV,
                     lds);
        } else if (inv_tile(tk)) {
          // explicit inverses, by row strips: forward y_k := L_kk^{-1} b_k into
          // the scratch vector (its rows r0.. need columns up to r0 + rows), backward
          // x_k := L_kk^{-T} y_k back into B (rows r0.. need columns from r0)
          const int m = tsz(tk);
          const int r0 = part * a.gemv_rows;
          const int rows = imin(a.gemv_rows, m - r0);
          double* const Sbase = a.S + sr[1];
          if (kind == TK_FTRSV && MODE == 0)  // L_kk^{-1} = (L_kk^{-T})^T: rows of it are columns of DinvT
            gemv_strip<double, true, true>(DinvTSys + (int64_t)tk * nb * nb + (int64_t)r0 * nb, nb,
                                           Sbase + tk * nb + r0, Bbase + tk * nb, ldb, rows, 0, imin(m, r0 + rows),
                                           (int)a.nrhs, lds, late);
          else if (kind == TK_FTRSV)
            gemv_strip<double, false, true>(DinvSys + (int64_t)tk * nb * nb + r0, nb, Sbase + tk * nb + r0,
                                            Bbase + tk * nb, ldb, rows, 0, imin(m, r0 + rows), (int)a.nrhs, lds, late);
          else
            gemv_strip<double, false, true>(DinvTSys + (int64_t)tk * nb * nb + r0, nb, Bbase + tk * nb + r0,
                                            Sbase + tk * nb, ldb, rows, r0, m, (int)a.nrhs, lds, late);
        } else if constexpr (MODE == 0) {
          // substitution against L_kk, in place (batched systems; an order not a multiple of 16)
          tile_solve(Abase + (tk * nb) * ld + tk * nb, ld, Bbase + tk * nb, ldb, tsz(tk), (int)a.nrhs,
                     kind == TK_BTRSV, lds);
        } else {
          ok = 0;
        }
        break;
      case TK_FGEMV: {
        if constexpr (!SOLVE_KINDS) {
          ok = 0;
          break;
        }
        const int r0 = part * a.gemv_rows;
        const int rows = imin(a.gemv_rows, tsz(ti) - r0);
        // y_k is in the scratch vector when the diagonal step applied an inverse
        const double* Yk = inv_tile(tk) ? a.S + sr[1] + tk * nb : Bbase + tk * nb;
        gemv_strip<E, false, false>(Abase + (tk * nb) * ld + ti * nb + r0, ld, Bbase + ti * nb + r0, Yk, ldb, rows,
                                    0, tsz(tk), (int)a.nrhs, lds, late);
        break;
      }
      case TK_BGEMV: {
        if constexpr (!SOLVE_KINDS) {
          ok = 0;
          break;
        }
        const int c0 = part * a.gemv_rows;
        const int cols = imin(a.gemv_rows, tsz(ti) - c0);
        double* Yi = inv_tile(ti) ? a.S + sr[1] + ti * nb + c0 : Bbase + ti * nb + c0;
        gemv_strip<E, true, false>(Abase + (ti * nb + c0) * ld + tk * nb, ld, Yi, Bbase + tk * nb, ldb, cols, 0,
                                   tsz(tk), (int)a.nrhs, lds, late);
        break;
      }
      case TK_TRTRI: {
        if constexpr (MODE != 0 && MODE != 1 && MODE != 3 && MODE != 5) {
          ok = 0;
        } else {
          // L_kk^{-T} by 32-row strips: identity rows solved in place (into DinvT, ld nb).
          // The mixed-precision factorization reads its FP64 diagonal tile,
          // identity-padded when ragged, and also stores the transposes as
          // L_kk^{-1} (Dinv); the FP64 launches read L_kk in A (its order is
          // then a multiple of 16) and keep L_kk^{-1} as well (for the TRSM
          // items), the adjoint L_kk^{-T} only.
          const int mpad = (tsz(tk) + 15) & ~15;
          const int r0 = part * a.trsm_rows;
          const int S = imin(a.trsm_rows, mpad - r0);
          double* X = DinvTSys + (int64_t)tk * nb * nb + r0;
          for (int idx = tid; idx < S * mpad; idx += NT) {
            const int c = idx / S, r = idx - c * S;
            st_dev(X + (int64_t)c * nb + r, (r0 + r == c) ? 1.0 : 0.0);
          }
          wait_vmcnt<0>();
          __syncthreads();
          if constexpr (MODE == 0)  // with L_kk^{-1} too (Dinv), if the TRSM items apply it (and not POTRF(k)'s)
            trsm_strip<double, 2>(X, nb, Abase + (tk * nb) * ld + tk * nb, ld, S, mpad, lds,
                                  a.finv ? nullptr : DinvSys + (int64_t)tk * nb * nb + (int64_t)r0 * nb, nb, nullptr, 0,
                                  0, r0 >> 4);
          else if constexpr (MODE == 3)  // the adjoint: L (its A) is the factor
            trsm_strip<double>(X, nb, Abase + (tk * nb) * ld + tk * nb, ld, S, mpad, lds, nullptr, 0, nullptr, 0, 0,
                               r0 >> 4);
          else
            trsm_strip<double, 2>(X, nb, Dsys + (int64_t)tk * nb * nb, nb, S, mpad, lds,
                                  DinvSys + (int64_t)tk * nb * nb + (int64_t)r0 * nb, nb, nullptr, 0, 0, r0 >> 4);
          count_inv = MODE == 0 ? 1 : 0;
        }
        break;
      }
      case TK_GREV:
      case TK_GREV2:
      case TK_TREV:
      case TK_DPART:
      case TK_DRED:
      case TK_PREV:
      case TK_PADJM:
      case TK_PADJY:
      case TK_PADJS: {
        if constexpr (!ADJOINT_KINDS) {
          ok = 0;
        } else {
          // A = L, B = Lbar (both at ld); Q and LT at ldq, zero past the order
          // (padded to a multiple of 16, so every K below is one)
          const int64_t ldq = a.ldq;
          const int T = (int)((sn + nb - 1) / nb);
          const int64_t np = (sn + 15) & ~(int64_t)15;
          if ((ldq & 1) != 0 || ldq < np) {
            raise_error(a, DEV_ERR_LAYOUT);  // unreachable when the host honours the launch contract
            ok = 0;
            break;
          }
          // partial-product slots, column k after column k - 1: S_ik at base(k) + i - k - 1
          auto slot = [&](int i, int k) __attribute__((always_inline)) {
            return (int64_t)k * (T - 1) - (int64_t)k * (k - 1) / 2 + (i - k - 1);
          };
          if (kind == TK_GREV) {
            // a single link (the last of its chain, on the critical path): 64 x 64 blocks
            const int ncj = (tsz(tk) + PRB - 1) / PRB;
            const int si = part / ncj, sj = part % ncj;
            const int M = imin(PRB, tsz(ti) - si * PRB), N = imin(PRB, tsz(tk) - sj * PRB);
            const int K = (int)(np - (int64_t)tj * nb < nb ? np - (int64_t)tj * nb : nb);
            double* C = Bbase + (tk * nb + sj * PRB) * ld + ti * nb + si * PRB;
            padj_block(a.Q + (tj * nb) * ldq + ti * nb + si * PRB, a.LT + (tj * nb) * ldq + tk * nb + sj * PRB, nullptr,
                       nullptr, ldq, M, N, K, lds,
                       [&](int r, int c, double v) __attribute__((always_inline)) {
                         st_dev(C + (int64_t)c * ld + r, v);
                       },
                       -1, C, ld);
          } else if (kind == TK_GREV2) {
            // the links j = tj and tj + 1 as one product over their
            // consecutive columns of Q and L^T (K = 2 nb, less at the padded end)
            const int ncj = (tsz(tk) + a.gemm_n - 1) / a.gemm_n;
            const int si = part / ncj, sj = part % ncj;
            const int M = imin(a.gemm_m, tsz(ti) - si * a.gemm_m);
            const int N = imin(a.gemm_n, tsz(tk) - sj * a.gemm_n);
            const int64_t kw = 2 * nb;
            const int K = (int)(np - (int64_t)tj * nb < kw ? np - (int64_t)tj * nb : kw);
            gemm_nt_ex(Bbase + (tk * nb + sj * a.gemm_n) * ld + ti * nb + si * a.gemm_m, ld,
                       a.Q + (tj * nb) * ldq + ti * nb + si * a.gemm_m, a.LT + (tj * nb) * ldq + tk * nb + sj * a.gemm_n,
                       ldq, M, N, K, false, false, lds);
          } else if (kind == TK_TREV) {
            // 64-row blocks of P_ik through L_kk^{-T} from TRTRI(k) (tile k is
            // never the ragged last one, so its order is a multiple of 16)
            const int r0 = part * PRB;
            double* Lb = Bbase + (tk * nb) * ld + ti * nb + r0;
            const int M = imin(PRB, tsz(ti) - r0);
            double* Qik = a.Q + (tk * nb) * ldq + ti * nb + r0;
            double* Qki = a.Q + (ti * nb + r0) * ldq + tk * nb;
            const double* IT = DinvTSys + (int64_t)tk * nb * nb;
            if ((ld & 1) == 0 && (reinterpret_cast<uintptr_t>(Bbase) & 15) == 0)
              trev_rows<128>(Lb, ld, IT, nb, M, tsz(tk), Qik, Qki, ldq, lds);
            else
              trev_rows<32>(Lb, ld, IT, nb, M, tsz(tk), Qik, Qki, ldq, lds);
          } else if (kind == TK_DPART) {
            // 64 x 64 block (bi, bj) of the lower triangle of the slot, -(P_ik^T L_ik)
            int bi, bj;
            lower_block(part, bi, bj);
            const int M = imin(PRB, tsz(tk) - bi * PRB), N = imin(PRB, tsz(tk) - bj * PRB);
            const int K = (int)(np - (int64_t)ti * nb < nb ? np - (int64_t)ti * nb : nb);
            double* Sk = a.D + slot(ti, tk) * nb * nb + (int64_t)(bj * PRB) * nb + bi * PRB;
            padj_block(a.Q + (ti * nb) * ldq + tk * nb + bi * PRB, a.LT + (ti * nb) * ldq + tk * nb + bj * PRB, nullptr,
                       nullptr, ldq, M, N, K, lds, [&](int r, int c, double v) __attribute__((always_inline)) {
                         if (bi != bj || r >= c) st_dev(Sk + (int64_t)c * nb + r, v);
                       });
          } else if (kind == TK_DRED) {
            // a tile whose order is a multiple of 16 takes the closed-form adjoint,
            // which reads Lbar_kk^T from the Q_kk tile
            const bool closed = (tsz(tk) & 15) == 0;
            dred_strip(Bbase + (tk * nb) * ld + tk * nb, ld, a.D + slot(tk + 1, tk) * nb * nb, nb * nb, T - 1 - tk, nb,
                       tsz(tk), part * 16, closed ? a.Q + (tk * nb) * ldq + tk * nb : nullptr, ldq);
          } else if (kind != TK_PREV) {
            // the closed-form tile adjoint: L_kk^{-T} in DinvT, two scratch
            // blocks (Mn, Y^T) per diagonal tile in Dinv
            const int64_t nb2 = nb * nb;
            padj_item(kind, part, tsz(tk), a.LT + (tk * nb) * ldq + tk * nb, a.Q + (tk * nb) * ldq + tk * nb, ldq,
                      Bbase + (tk * nb) * ld + tk * nb, ld, DinvTSys + tk * nb2, DinvSys + 2 * tk * nb2,
                      DinvSys + (2 * tk + 1) * nb2, nb, lds);
          } else {
            // the partial products were applied by DRED(k)
            prev_tile(Abase + (tk * nb) * ld + tk * nb, a.LT + (tk * nb) * ldq + tk * nb,
                      Bbase + (tk * nb) * ld + tk * nb, ld, a.Q + (tk * nb) * ldq + tk * nb, ldq, tsz(tk), a.D,
                      nb * nb, 0, nb, lds);
          }
        }
        break;
      }
      default:
        ok = 0;
        break;
    }
    // Publish.  Every global store of a work item is a device-scope store
    // (st_dev), written through to the device's point of coherence; once
    // each wavefront has seen its stores complete (vmcnt 0) the item's
    // results are visible to any CU that invalidates its caches before
    // reading them (the acquire after each wait).  This replaces an
    // agent-scope release fence, whose L2 write-back costs tens of
    // microseconds per work item on this part.  The completion counter is
    // incremented at the start of the next claim.
    wait_vmcnt<0>();
    __syncthreads();
    if (POOLED && unit >= 0) {
      // a pool unit: its sub-block counter tells the units that wait for it
      if (tid == 0) {
        const int ctr = pu.type == 0 ? PL_P + pu.b : (pu.type == 1 ? PL_S + 4 * pu.r + pu.b : PL_U + 4 * pu.r + pu.c);
        __hip_atomic_fetch_add(a.pool + POOL_WORDS * (sr[6] + tk) + ctr, unit_failed ? 1 + PL_FAILED : 1,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else if (wave == 0) {
      if (count_inv && lane == 0)
        __hip_atomic_fetch_add(a.pool + POOL_WORDS * (sr[6] + tk) + PL_INV, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      p_fwd = kind == TK_FTRSV && (int64_t)(tk + 1) * nb >= sn;
      p_task = ok ? task : -1;
      p_ticket = ticket;
      p_parts = d_parts;
      p_e0 = d_e0;
      p_e1 = d_e1;
      if (a.trace) p_end = wall_clock64();
    }
  }
}

// Clears the header and the per-task completion counters and copies the
// initial dependency counters; the plan's constant part is copied by the host.
__global__ void tchol_reset(int32_t* hdr, int32_t* dep, int32_t* done, const int32_t* dep0, int32_t ntask,
                            int32_t* sinfo, int32_t nsys, int32_t* pool, int64_t npool) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < HDR_WORDS) hdr[i] = 0;
  if (i < ntask) {
    dep[i] = dep0[i];
    done[i] = 0;
  }
  if (i < nsys) sinfo[i] = 0;
  if (i < npool) pool[i] = 0;
}

// wide: every panel the launch streams is 16-byte transferable (even
// leading dimensions, 16-byte aligned matrices), decided by the host.
// npool: words of the POTRF pools (all zeroed by the reset kernel).
extern "C" hipError_t tchol_dev_launch(const KArgs* a, int32_t ntask, const int32_t* dep0, int64_t npool, int grid,
                                       int wide, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  const int rb = 256;
  int64_t cover = ntask > HDR_WORDS ? ntask : HDR_WORDS;
  if (a->nsys > cover) cover = a->nsys;
  if (npool > cover) cover = npool;
  hipLaunchKernelGGL(tchol_reset, dim3((unsigned)((cover + rb - 1) / rb)), dim3(rb), 0, stream, a->hdr, a->dep,
                     a->done, dep0, ntask, a->sinfo, a->nsys, a->pool, npool);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev0) {
    e = hipEventRecord(ev0, stream);
    if (e != hipSuccess) return e;
  }
  if (a->mixed == 5)
    hipLaunchKernelGGL((tchol_persistent<128, 5>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (a->mixed == 4)
    hipLaunchKernelGGL((tchol_persistent<128, 4>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (a->mixed == 3)
    hipLaunchKernelGGL((tchol_persistent<128, 3>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (a->mixed == 1)
    hipLaunchKernelGGL((tchol_persistent<128, 1>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (a->mixed == 2)
    hipLaunchKernelGGL((tchol_persistent<128, 2>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (a->mixed == 6)
    hipLaunchKernelGGL((tchol_persistent<128, 6>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (a->mixed == 7)
    hipLaunchKernelGGL((tchol_persistent<128, 7>), dim3(grid), dim3(NT), 0, stream, *a);
  else if (wide)
    hipLaunchKernelGGL((tchol_persistent<128, 0>), dim3(grid), dim3(NT), 0, stream, *a);
  else
    hipLaunchKernelGGL((tchol_persistent<32, 0>), dim3(grid), dim3(NT), 0, stream, *a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev1) e = hipEventRecord(ev1, stream);
  return e;
}

// The adjoint's preparation (LT and the padding of Q), before its persistent launch.
extern "C" hipError_t tchol_dev_backward_prep(const double* L, int64_t n, double* LT, double* Q, int64_t ldq,
                                              int64_t np, hipStream_t stream) {
  if (np == 0) return hipSuccess;
  const unsigned g = (unsigned)((np + 31) / 32);
  hipLaunchKernelGGL(tchol_backward_prep, dim3(g, g), dim3(256), 0, stream, L, n, LT, Q, ldq, np);
  return hipGetLastError();
}

// Workgroups of the compact instance (batched systems of one tile each) that
// the device holds at once.
extern "C" hipError_t tchol_dev_compact_grid(int device, int* grid) {
  int cus = 0, occ = 0;
  hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, tchol_persistent<128, 6>, NT, 0);
  if (e != hipSuccess) return e;
  int occ7 = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ7, tchol_persistent<128, 7>, NT, 0);
  if (e != hipSuccess) return e;
  occ = occ < occ7 ? occ : occ7;
  *grid = cus * (occ > 0 ? occ : 1);
  return hipSuccess;
}

extern "C" hipError_t tchol_dev_max_grid(int device, int* grid) {
  int cus = 0, occ = 0;
  hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  if (e != hipSuccess) return e;
  // both instances share the LDS size and launch bounds; take the smaller occupancy
  int occ32 = 0;
  int occm = 0, occs = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, tchol_persistent<128, 0>, NT, 0);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ32, tchol_persistent<32, 0>, NT, 0);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occm, tchol_persistent<128, 1>, NT, 0);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occs, tchol_persistent<128, 2>, NT, 0);
  if (e != hipSuccess) return e;
  int occa = 0, occb = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occa, tchol_persistent<128, 3>, NT, 0);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occb, tchol_persistent<128, 4>, NT, 0);
  if (e != hipSuccess) return e;
  int occf = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occf, tchol_persistent<128, 5>, NT, 0);
  if (e != hipSuccess) return e;
  occ = occ < occf ? occ : occf;
  occ = occ < occa ? occ : occa;
  occ = occ < occb ? occ : occb;
  occ = occ < occ32 ? occ : occ32;
  occ = occ < occm ? occ : occm;
  occ = occ < occs ? occ : occs;
  *grid = cus * (occ > 0 ? occ : 1);
  return hipSuccess;
}
