// FP8 GEMM for the three products of the split linear (gfx950 MFMA).
//
// §3.2 of the paper: F computes Y = X W^T, dI computes dX = dY W, and the
// deferred dW computes dW = dY^T X, each on FP8-quantized operands.  With the
// quantizer writing every operand both row-wise and transposed, all three are
// the same "TN" product with both operands contiguous along the reduction:
//     D[i][j] = 2^(ea + eb) * sum_r A[i][r] B[j][r]
// where 2^ea, 2^eb are the operands' scale inverses (powers of two, so the
// rescale is one exact ldexp).  The epilogue stores D (FP32 or BF16), or adds
// it to an FP32 destination in place: the direct placement of dW into its
// slice of the flat main-gradient buffer (§3.4), with no staging copy.
//
// gemm_tn_w4_kernel serves the large tiles, 256 x 256 x 128 (and 256 x 224,
// 256 x 192, 192 x 256); gemm_ring.hip the small ones.  Every shape uses
// v_mfma_f32_16x16x128_f8f6f4 with the same assignment of reduction bytes to
// lanes and accumulates each output element in the same order, so all give the
// same bits.  Four waves (one per SIMD) on a 2 x 2 grid, each a 128 x 128
// sub-tile of 8 x 8 MFMA blocks.  A K tile's 64 MFMAs run in two phases; every
// fragment read or LDS-bound load is issued right after an MFMA, in a fixed
// order (sched_barrier), so the MFMA pipe stays busy in the single wave, and
// the LDS-bound loads are branch-free (two instructions each) because a single
// wave issues at most one instruction per four cycles, eight per MFMA.  The K
// loop is rotated so that its back-edge sits at the stage barrier, where all
// LDS reads have completed; the compiler can then wait for fragment reads one
// by one instead of draining them at the loop head.  The epilogue goes through
// LDS so every store instruction writes whole row runs (512-byte FP32 runs;
// BF16 values are rounded first and go as 256-byte runs).
// Operand formats (E4M3 or E5M2) are chosen per call.  K tiles are
// double-buffered in LDS and filled by LDS-bound global loads
// (global_load_lds_dwordx4: no register staging, no LDS store instructions)
// issued a K tile ahead; each wave waits for its own loads and a barrier
// publishes the stage.  The 4-wave kernel splits a K tile's loads: the B part
// goes into a stage's B half as soon as every wave holds the B fragments of
// the tile that stage held (during phase A, a K step and a half before it is
// read), the A part in the first half of phase B; a second barrier per K step
// marks the B half free.  (Measured on MI355X: against all loads spread over
// phase B, the Llama-3-70B stage's GEMMs 4% faster, products whose operands
// stream from HBM up to 8%.)  LDS rows are 128 bytes, their 16-byte chunks
// XOR-swizzled by row (row_swizzle) so that a fragment read meets no bank
// conflict, and since fragments start on multiples of 16 rows, every fragment
// of a wave is one base address plus a constant.  The LDS-bound loads are inline
// assembly: the compiler's own form makes it wait for them before every LDS
// read, serialising the loads with the MFMA work.  Rows past M / N are
// clamped to the last row (their results are never stored), so only the last,
// partial K tile needs masking; it goes through registers.
//
// MFMA operand order: the B fragment is passed as source A and the A fragment
// as source B, so each lane ends up holding four consecutive output columns of
// one output row and the epilogue stores 16 bytes per lane.  Within a lane the
// 32 reduction bytes of a fragment come from the same positions for A and B,
// so any fixed assignment of reduction indices to MFMA slots gives the same
// dot products.
//
// Determinism: no atomics and no split reduction; the same inputs produce the
// same bits, which the split-vs-full-backward check relies on.
#include "gemm_util.h"
#include "scale_update.h"

namespace qe {
namespace {

// 256 x 256 x 128 tile (also 256 x 224, 256 x 192 and 192 x 256), four waves
// (one per SIMD) on a 2 x 2 grid, each wave a TM x TN sub-tile of 16 x 16 blocks of
// v_mfma_f32_16x16x128_f8f6f4, one MFMA per block per K tile.  (On random FP8
// operands this MFMA sustains about a third more throughput than the 32 x 32 x
// 64 one on MI355X, which draws more power per FLOP; with constant operands
// the two are equal.)
// A K tile's MFMAs run in two phases of I/2 block rows each:
//   phase A (block rows 0 .. I/2-1, column-major): uses A fragments
//     0 .. I/2-1 and every B fragment; reads A fragments I/2 .. I-1 of the
//     same tile; issues the B part of the LDS-bound loads of the tile two K
//     tiles ahead into this stage's B half;
//   phase B (block rows I/2 .. I-1, column-major): each B fragment's last use
//     is followed by the read of the next tile's B fragment into the same
//     registers, and the next tile's A fragments 0 .. I/2-1 are read too; the
//     A part of the loads of the tile after next is issued in its first half.
// So all of tile t is read by the end of its phase A, where the stage barrier
// sits: it frees tile t's A half for the A part of tile t+2 and publishes tile
// t+1.  A second barrier, after phase B, marks the B half of tile t+1's stage
// free once every wave holds tile t+1's B fragments, so phase A of tile t+1
// loads tile t+3's B part there: a K step and a half of latency budget for
// the B part, about a phase for the A part.  Fragment registers: I + J
// fragments of 8 VGPRs, no second set.  The K loop is rotated (phase B of tile t, then phase A of tile t+1)
// so its back-edge sits at the barrier, where every LDS read has completed;
// the waits for fragment reads inside an iteration can then be partial.
template <int FA, int FB, int OUT, int BM, int BN>
__global__ __launch_bounds__(256) void gemm_tn_w4_kernel(GemmParams g, int tiles_m, int tiles_n, int vec_ok,
                                                         UpdateParams upd) {
  static_assert((BM == 256 || BM == 192) && (BN == 256 || BN == 224 || BN == 192), "tile sizes");
  constexpr int NW = 4, TM = BM / 2, TN = BN / 2;
  constexpr int I = TM / 16, J = TN / 16;    // 16 x 16 MFMA blocks per wave sub-tile
  constexpr int IA = I / 2, IB = I - IA;     // block rows of phase A and phase B
  constexpr int QA = IA * J, QB = IB * J;    // MFMAs per phase
  constexpr int CHA = BM / 32, CHB = BN / 32;  // 16-byte LDS-bound loads per lane per K tile
  constexpr int ND = CHA + CHB;              // LDS-bound loads per K tile
  constexpr int STAGE = (BM + BN) * BK;
  constexpr int EP = TN + 4;                 // epilogue staging row, in floats (padded)
  static_assert(NW * 32 * EP * 4 <= 2 * STAGE, "epilogue staging fits in the stages");
  static_assert(CHA * NW * 1024 == BM * BK, "LDS-bound load d of a tile lands at stage + 4096 d");
  // two K stages, then one 1 KB block per wave that absorbs the loads issued
  // past the last full K tile (so the loop issues them unconditionally)
  __shared__ __attribute__((aligned(16))) uint8_t smem[2 * STAGE + NW * 1024];
  static_assert(sizeof(smem) >= (kMaxHistory + kUpdateThreads / 64) * 4, "history staging fits in the stages");

  // Workgroups past the tiles (dispatched last) run the delayed scale update
  // of the action's roles beside the tiles: the tiles read the scale_inv
  // snapshots, never the live scales this update writes.
  if (int(blockIdx.x) >= tiles_m * tiles_n) {
    const int r = int(blockIdx.x) - tiles_m * tiles_n;
    uint32_t *hs = reinterpret_cast<uint32_t *>(smem);
    scale_update_role(upd.m[r], r == 0 ? upd.token : nullptr, hs, hs + kMaxHistory);
    return;
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  const int pid = xcd_remap(blockIdx.x, tiles_m * tiles_n);
  const int in_group = kGroupM * tiles_n;
  const int group = pid / in_group;
  const int first_m = group * kGroupM;
  const int gsize = min(tiles_m - first_m, kGroupM);
  const int tm = first_m + (pid % in_group) % gsize;
  const int tn = (pid % in_group) / gsize;
  const int64_t m0 = int64_t(tm) * BM, n0 = int64_t(tn) * BN;

  const int64_t M = g.m, N = g.n, K = g.k;
  const int KT = int(K / BK);
  const int64_t ktail = K - int64_t(KT) * BK;
  const int T = KT + (ktail > 0 ? 1 : 0);

  const int lrow = lane >> 3;
  uint32_t oa[CHA], ob[CHB];
#pragma unroll
  for (int c = 0; c < CHA; ++c) {
    const int row = 8 * (wave + NW * c) + lrow;
    const int lch = (lane & 7) ^ row_swizzle(row);
    oa[c] = chunk_offset(min(m0 + row, M - 1), g.lda, lch, K);
  }
#pragma unroll
  for (int c = 0; c < CHB; ++c) {
    const int row = 8 * (wave + NW * c) + lrow;
    const int lch = (lane & 7) ^ row_swizzle(row);
    ob[c] = chunk_offset(min(n0 + row, N - 1), g.ldb, lch, K);
  }
  const uint32_t lds_base = uint32_t(reinterpret_cast<uintptr_t>(smem));
  const uint32_t wblk = __builtin_amdgcn_readfirstlane(lds_base + uint32_t(wave) * 1024u);
  const uint32_t wdummy = __builtin_amdgcn_readfirstlane(lds_base + uint32_t(2 * STAGE) + uint32_t(wave) * 1024u);

  auto issue = [&](int kt, int buf) {
    if (kt < KT) {
      const uint8_t *ga = g.a + int64_t(kt) * BK;
      const uint8_t *gb = g.b + int64_t(kt) * BK;
      const uint32_t sa = wblk + uint32_t(buf * STAGE);
      const uint32_t sb = sa + uint32_t(BM * BK);
#pragma unroll
      for (int c = 0; c < CHA; ++c)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(oa[c]), "s"(ga),
                     "s"(sa + uint32_t(c * NW * 1024)) : "memory", "m0");
#pragma unroll
      for (int c = 0; c < CHB; ++c)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(ob[c]), "s"(gb),
                     "s"(sb + uint32_t(c * NW * 1024)) : "memory", "m0");
    } else {  // the last, partial K tile, through registers: bytes at or past K are zero
      uint8_t *dA = smem + buf * STAGE;
      uint8_t *dB = dA + BM * BK;
      const uint32_t k0 = uint32_t(KT) * BK;
#pragma unroll
      for (int c = 0; c < CHA; ++c) {
        const int row = 8 * (wave + NW * c) + lrow;
        const int64_t gk = int64_t(k0) + ((lane & 7) ^ row_swizzle(row)) * 16;
        const uint4 va = gk < K ? mask_tail(*reinterpret_cast<const uint4 *>(g.a + (oa[c] + k0)), K - gk) : make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4 *>(dA + (wave + NW * c) * 1024 + lane * 16) = va;
      }
#pragma unroll
      for (int c = 0; c < CHB; ++c) {
        const int row = 8 * (wave + NW * c) + lrow;
        const int64_t gk = int64_t(k0) + ((lane & 7) ^ row_swizzle(row)) * 16;
        const uint4 vb = gk < K ? mask_tail(*reinterpret_cast<const uint4 *>(g.b + (ob[c] + k0)), K - gk) : make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4 *>(dB + (wave + NW * c) * 1024 + lane * 16) = vb;
      }
    }
  };

  // 16-row fragments: lane l reads row (l & 15), the 32 bytes 32 (l >> 4) .. +31
  // of the K tile, i.e. logical chunks 2 (l >> 4) and the next.  The swizzle
  // term depends on (l & 15) only, so every fragment is base + constant.
  const int fr = lane & 15, fq = lane >> 4;
  const uint32_t f_lo = uint32_t(fr) * BK + uint32_t((2 * fq) ^ row_swizzle(fr)) * 16;
  const uint32_t f_hi = uint32_t(fr) * BK + uint32_t((2 * fq + 1) ^ row_swizzle(fr)) * 16;
  auto frag = [&](const uint8_t *base) -> v8i {
    const uint4 lo = *reinterpret_cast<const uint4 *>(base + f_lo);
    const uint4 hi = *reinterpret_cast<const uint4 *>(base + f_hi);
    return v8i{int(lo.x), int(lo.y), int(lo.z), int(lo.w), int(hi.x), int(hi.y), int(hi.z), int(hi.w)};
  };
  auto read_a = [&](int buf, int i, v8i (&fa)[I]) { fa[i] = frag(smem + buf * STAGE + (wm * TM + i * 16) * BK); };
  auto read_b = [&](int buf, int j, v8i (&fb)[J]) {
    fb[j] = frag(smem + buf * STAGE + (BM + wn * TN + j * 16) * BK);
  };

  v4f acc[I][J];
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  auto mfma = [&](int i, int j, const v8i (&fa)[I], const v8i (&fb)[J]) {
    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fb[j], fa[i], acc[i][j], FB, FA, 0, 0, 0, 0);
  };
  // LDS-bound loads inside the K loop, two instructions each: load d of a K
  // tile lands at stage + 4096 d, so M0 steps by a uniform stride, and the
  // step is issued before an MFMA and the load after it (the MFMA is the wait
  // state M0 needs).  Past the last full K tile the loads still run, from
  // tile 0 into the wave's dummy block with stride 0: no branch per load (and
  // no byte past a row of less than 128, see chunk_offset).
  auto dma_m0 = [&](int d, uint32_t base, uint32_t stride) {
    if (d == 0)
      asm volatile("s_mov_b32 m0, %0" ::"s"(base) : "m0");
    else
      asm volatile("s_add_u32 m0, m0, %0" ::"s"(stride) : "m0", "scc");
  };
  auto dma_load = [&](int d, const uint8_t *ga, const uint8_t *gb) {
    if (d < CHA)
      asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(oa[d]), "s"(ga) : "memory");
    else
      asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(ob[d - CHA]), "s"(gb) : "memory");
  };

  // Phase A of a tile from stage `buf`: column-major MFMAs over block rows
  // 0 .. IA-1 (B fragment j is first needed at MFMA j * IA, so the fragments
  // read last in the previous phase B are needed last); A fragments IA .. I-1
  // of the same tile are read after the first MFMAs (one per even slot), long
  // before phase B needs them.  The tile's B fragments are all in registers
  // by now, so the same stage's B half already takes the B part of the tile
  // two K tiles ahead (`kt3`), spread over the phase: a K step and a half
  // before it is read.
  auto b_slot = [](int q, int k) { return (k * QA) / CHB + 1 == q; };
  auto phase_a = [&](int buf, bool dmab, int kt3, v8i (&fa)[I], v8i (&fb)[J]) {
    const uint8_t *gb = dmab ? g.b + int64_t(kt3) * BK : g.b;
    const uint32_t base = dmab ? wblk + uint32_t(buf * STAGE + BM * BK) : wdummy;
    const uint32_t stride = dmab ? uint32_t(NW * 1024) : 0u;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      int d = -1;  // the B-part load of this slot (folds to a constant once unrolled)
#pragma unroll
      for (int k = 0; k < CHB; ++k) d = b_slot(q, k) ? k : d;
      __builtin_amdgcn_sched_barrier(0);
      if (d >= 0) dma_m0(d, base, stride);
      __builtin_amdgcn_sched_barrier(0);
      mfma(q % IA, q / IA, fa, fb);
      __builtin_amdgcn_sched_barrier(0);
      if (d >= 0) dma_load(CHA + d, g.a, gb);
      if (q % 2 == 0 && q / 2 < IB) read_a(buf, IA + q / 2, fa);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Phase B of a tile: column-major MFMAs over block rows IA .. I-1.  After
  // the last use of B fragment j, the next tile's B fragment j is read from
  // stage `nbuf` into the same registers; the next tile's A fragments
  // 0 .. IA-1 are read in the first slots (their registers are free since
  // phase A).  `dma` issues the A part of tile `kt2` into stage `buf`.
  // Slots of phase B, one kind of memory instruction each where possible: the
  // next tile's A fragments after MFMAs 0, 4, 8, ..; LDS-bound loads after
  // MFMAs q = 1, 2 (mod 4), so the A part is issued in the first half of the
  // phase; B fragments after the last use of each (q = 3 (mod 4) when IB =
  // 4).  Loads that do not fit go to the latest q = 0 (mod 4) slots past the A
  // reads.  (Measured: the A part spread over all of phase B instead, equal;
  // the B part packed into the first half of phase A, 0.5% slower.)
  auto load_slot = [](int q) -> bool {
    constexpr int n12 = (QB / 4) * 2;
    if (q % 4 == 1 || q % 4 == 2) return (q / 4) * 2 + (q % 4 - 1) < CHA;
    if (q % 4 == 0 && CHA > n12) return q / 4 >= IA && QB / 4 - 1 - q / 4 < CHA - n12;
    return false;
  };
  auto phase_b = [&](int nbuf, bool dma, int kt2, int buf, v8i (&fa)[I], v8i (&fb)[J]) {
    static_assert(QB % 4 == 0, "phase B slots come in fours");
    const uint8_t *ga = dma ? g.a + int64_t(kt2) * BK : g.a;
    const uint8_t *gb = dma ? g.b + int64_t(kt2) * BK : g.b;
    const uint32_t base = dma ? wblk + uint32_t(buf * STAGE) : wdummy;
    const uint32_t stride = dma ? uint32_t(NW * 1024) : 0u;
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int j = q / IB, i = IA + q % IB;
      const bool ld = load_slot(q);
      int d = 0;  // loads in earlier slots (folds to a constant once unrolled)
#pragma unroll
      for (int r = 0; r < q; ++r) d += load_slot(r) ? 1 : 0;
      __builtin_amdgcn_sched_barrier(0);
      if (ld) dma_m0(d, base, stride);
      __builtin_amdgcn_sched_barrier(0);  // M0 is written before the MFMA, never next to the load
      mfma(i, j, fa, fb);
      __builtin_amdgcn_sched_barrier(0);
      if (ld) dma_load(d, ga, gb);
      if (q % 4 == 0 && q / 4 < IA) read_a(nbuf, q / 4, fa);
      if (q % IB == IB - 1) read_b(nbuf, j, fb);  // last use of B fragment j was this MFMA
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  if (T > 0) {
    v8i fa[I], fb[J];
    issue(0, 0);
    if (KT > 1) {
      // both first K tiles are full: tile 1's LDS-bound loads stay in flight
      // while the wave waits for its tile-0 loads (the ND most recent ones
      // are tile 1's; the counter completes in order)
      issue(1, 1);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ND) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j) read_b(0, j, fb);
#pragma unroll
    for (int i = 0; i < IA; ++i) read_a(0, i, fa);
    if (T > 1 && KT <= 1) issue(1, 1);  // tile 1 is the partial tail: through registers
    __syncthreads();                       // every wave holds tile 0's B fragments: stage 0's B half is free
    phase_a(0, 2 < KT, 2, fa, fb);         // and takes tile 2's B part
    // tile 1 complete; the CHB most recent loads (tile 2's B part) may still
    // be in flight: the counter completes in order
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CHB) : "memory");
    __syncthreads();                       // tile 1 published; tile 0 fully read
    for (int t = 0; t < T; ++t) {
      const int buf = t & 1;
      const bool dma = t + 2 < KT;
      if (t + 2 < T && !dma) issue(t + 2, buf);
      // phase B of tile t, with tile t+2's A part; reads of tile t+1 (in the
      // last iteration they read a stale stage that is never used: always in
      // bounds, and branch-free here)
      phase_b(buf ^ 1, dma, t + 2, buf, fa, fb);
      if (t + 1 < T) {
        __syncthreads();                   // tile t+1's B fragments read by every wave
        phase_a(buf ^ 1, t + 3 < KT, t + 3, fa, fb);  // with tile t+3's B part
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CHB) : "memory");
        __syncthreads();                   // tile t+2 published; tile t+1 fully read
      }
    }
  }

  // Epilogue through LDS: the MFMA layout gives each lane one row and a column
  // quad per 16 x 16 block, so store instructions would touch 16 rows x 64 B.
  // Each wave instead writes one 32-row block of its sub-tile (32 x TN FP32,
  // rows padded to TN + 4 floats) into LDS, then reads it back row-contiguous:
  // 32 lanes x 16 B cover one 512-byte output row run per store instruction.
  __syncthreads();  // every wave is done reading the last stage
  float *ep = reinterpret_cast<float *>(smem) + wave * 32 * EP;
  const int e = pow2_exponent(g.a_scale_inv) + pow2_exponent(g.b_scale_inv);
  const bool nfull = n0 + BN <= N;
  // Full tile with a vector-aligned destination (the common case): no bounds
  // checks, every store address is a uniform row base (scalar registers) plus
  // one per-lane offset, and LDS addresses are one base plus immediates.  With
  // one wave per SIMD the epilogue runs at instruction latency, so its
  // instruction count is its time.  Other tiles take the checked path.
  constexpr int ES = OUT == 1 ? 2 : 4;  // output element bytes
  // (buffer instructions: the row offset is a scalar operand; every offset of
  // the wave's TM x TN block stays below 2^31)
  const bool fast = vec_ok && nfull && m0 + BM <= M && g.ldc * ES * (TM + 2) < (int64_t(1) << 31);
  const bool has_col = (lane & 31) * 4 < TN;  // TN = 112 or 96: 28 or 24 of each 32 lanes hold a column quad
  const int wu = __builtin_amdgcn_readfirstlane(wave);
  const uint32_t voff = uint32_t((lane >> 5) * g.ldc + (lane & 31) * 4) * uint32_t(ES);
  char *cbase = static_cast<char *>(g.c) + ((m0 + (wu >> 1) * TM) * g.ldc + n0 + (wu & 1) * TN) * ES;
  const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(cbase, short(0), 0x7fffffff, 0x00020000);
  const int rstep = int(g.ldc) * ES;  // bytes per output row
  float *ew = ep + (lane & 15) * EP + 4 * (lane >> 4);
  const float *er = ep + (lane >> 5) * EP + (lane & 31) * 4;
#pragma unroll
  for (int i = 0; i < TM / 32; ++i) {
    // accumulate: read this block's destination first, so the loads are in
    // flight during the LDS round trip instead of one dependent load per row
    float4 pre[16];
    if constexpr (OUT == 2) {
      if (fast) {
#pragma unroll
        for (int it = 0; it < 16; ++it)
          if (has_col) pre[it] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(crs, voff, (i * 32 + 2 * it) * rstep, kNT));
      } else {
#pragma unroll
        for (int it = 0; it < 16; ++it) {
          const int64_t row = m0 + wm * TM + i * 32 + 2 * it + (lane >> 5);
          const int64_t col = n0 + wn * TN + (lane & 31) * 4;
          pre[it] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (has_col && row < M && (nfull || col + 4 <= N)) {
            const v4f_out w = *reinterpret_cast<const v4f_out *>(static_cast<const float *>(g.c) + row * g.ldc + col);
            pre[it] = make_float4(w[0], w[1], w[2], w[3]);
          }
        }
      }
    }
    if constexpr (OUT == 1) {
      if (fast) {
        // BF16 output: rounded before the LDS round trip, which then moves
        // half the bytes (rows of TN values padded to TN + 8), and every store
        // instruction writes four 2 * TN-byte row runs, 16 bytes per lane.
        // The same round-to-nearest-even of the same FP32 value, so the same
        // bits; measured 0.3-0.5% faster per stage step on MI355X.
        constexpr int EPH = TN + 8;
        uint16_t *eh = reinterpret_cast<uint16_t *>(ep);
        uint16_t *ehw = eh + (lane & 15) * EPH + 4 * (lane >> 4);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const v4f a = acc[2 * i + h][j];
            *reinterpret_cast<uint2 *>(ehw + h * 16 * EPH + j * 16) =
                make_uint2(bf16x2_bits(__builtin_ldexpf(a[0], e), __builtin_ldexpf(a[1], e)),
                           bf16x2_bits(__builtin_ldexpf(a[2], e), __builtin_ldexpf(a[3], e)));
          }
        const uint16_t *ehr = eh + (lane >> 4) * EPH + (lane & 15) * 8;
        const uint32_t voffh = uint32_t((lane >> 4) * g.ldc + (lane & 15) * 8) * 2u;
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          if ((lane & 15) * 8 >= TN) continue;
          const uint4 v = *reinterpret_cast<const uint4 *>(ehr + it * 4 * EPH);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), crs, voffh, (i * 32 + 4 * it) * rstep, kNT);
        }
        continue;
      }
    }
    // block rows 2i and 2i+1: lane holds row (lane & 15) of each, four
    // consecutive columns 16 j + 4 (lane >> 4) .. +3 of every column block j
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < J; ++j)
        *reinterpret_cast<float4 *>(ew + h * 16 * EP + j * 16) =
            make_float4(__builtin_ldexpf(acc[2 * i + h][j][0], e), __builtin_ldexpf(acc[2 * i + h][j][1], e),
                        __builtin_ldexpf(acc[2 * i + h][j][2], e), __builtin_ldexpf(acc[2 * i + h][j][3], e));
    // same wave writes then reads its own LDS rows: LDS operations of one wave
    // complete in order
    if (fast) {
#pragma unroll
      for (int it = 0; it < 16; ++it) {
        if (!has_col) continue;
        const float4 v4 = *reinterpret_cast<const float4 *>(er + it * 2 * EP);
        const int so = (i * 32 + 2 * it) * rstep;
        if constexpr (OUT == 0) {
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v4), crs, voff, so, kNT);
        } else if constexpr (OUT == 1) {
          const v2i w = {int(bf16x2_bits(v4.x, v4.y)), int(bf16x2_bits(v4.z, v4.w))};
          __builtin_amdgcn_raw_buffer_store_b64(w, crs, voff, so, kNT);
        } else {
          const float4 o = pre[it];
          const float4 r = make_float4(o.x + v4.x, o.y + v4.y, o.z + v4.z, o.w + v4.w);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, r), crs, voff, so, kNT);
        }
      }
      continue;
    }
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      const int r = 2 * it + (lane >> 5);
      const int64_t row = m0 + wm * TM + i * 32 + r;
      const int cl = (lane & 31) * 4;
      const int64_t col = n0 + wn * TN + cl;
      if (!has_col) continue;
      const float4 v4 = *reinterpret_cast<const float4 *>(ep + r * EP + cl);
      if (row >= M) continue;
      const float v[4] = {v4.x, v4.y, v4.z, v4.w};
      if (nfull || col + 4 <= N) {  // at any alignment
        if constexpr (OUT == 0) {
          *reinterpret_cast<v4f_out *>(static_cast<float *>(g.c) + row * g.ldc + col) = v4f_out{v[0], v[1], v[2], v[3]};
        } else if constexpr (OUT == 1) {
          const uint32_t lo = bf16x2_bits(v[0], v[1]);
          const uint32_t hi = bf16x2_bits(v[2], v[3]);
          *reinterpret_cast<v2i_out *>(static_cast<uint16_t *>(g.c) + row * g.ldc + col) = v2i_out{int(lo), int(hi)};
        } else {
          const float4 o = pre[it];
          *reinterpret_cast<v4f_out *>(static_cast<float *>(g.c) + row * g.ldc + col) =
              v4f_out{o.x + v[0], o.y + v[1], o.z + v[2], o.w + v[3]};
        }
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (col + t >= N) break;
          if constexpr (OUT == 0) {
            static_cast<float *>(g.c)[row * g.ldc + col + t] = v[t];
          } else if constexpr (OUT == 1) {
            static_cast<uint16_t *>(g.c)[row * g.ldc + col + t] = bf16_bits(v[t]);
          } else {
            float *dst = static_cast<float *>(g.c) + row * g.ldc + col + t;
            *dst = *dst + v[t];
          }
        }
      }
    }
  }
}

template <int FA, int FB, int BM, int BN>
hipError_t launch_w4(const GemmParams &g, hipStream_t s, const UpdateParams &u) {
  const int tiles_m = int((g.m + BM - 1) / BM), tiles_n = int((g.n + BN - 1) / BN);
  const int vec_ok = gemm_vec_ok(g);
  const dim3 grid(unsigned(tiles_m) * unsigned(tiles_n) + unsigned(u.n)), block(256);
  switch (g.out) {
    case 0: return klaunch(gemm_tn_w4_kernel<FA, FB, 0, BM, BN>, grid, block, 0, s, g, tiles_m, tiles_n, vec_ok, u);
    case 1: return klaunch(gemm_tn_w4_kernel<FA, FB, 1, BM, BN>, grid, block, 0, s, g, tiles_m, tiles_n, vec_ok, u);
    default: return klaunch(gemm_tn_w4_kernel<FA, FB, 2, BM, BN>, grid, block, 0, s, g, tiles_m, tiles_n, vec_ok, u);
  }
}

template <int BM, int BN>
hipError_t launch_w4_fmts(const GemmParams &g, hipStream_t s, const UpdateParams &u) {
  if (g.fmt_a == 0 && g.fmt_b == 0) return launch_w4<0, 0, BM, BN>(g, s, u);
  if (g.fmt_a == 1 && g.fmt_b == 0) return launch_w4<1, 0, BM, BN>(g, s, u);
  if (g.fmt_a == 0 && g.fmt_b == 1) return launch_w4<0, 1, BM, BN>(g, s, u);
  return launch_w4<1, 1, BM, BN>(g, s, u);
}

}  // namespace

hipError_t launch_gemm_large(int tile, const GemmParams &g, hipStream_t s, const UpdateParams &u) {
  switch (tile) {
    case kTile256x192: return launch_w4_fmts<256, 192>(g, s, u);
    case kTile192x256: return launch_w4_fmts<192, 256>(g, s, u);
    case kTile256x224: return launch_w4_fmts<256, 224>(g, s, u);
    default: return launch_w4_fmts<256, 256>(g, s, u);
  }
}

}  // namespace qe
