// FP8 GEMM for products whose grid of 256-row tiles leaves the chip idle
// (small microbatches, small layers), with the same result bits as the large
// tiles of gemm_fp8.hip.
//
// One workgroup of four waves (2 x 2) per BM x BN tile; each wave owns a
// BM/2 x BN/2 sub-tile of 16 x 16 blocks of v_mfma_f32_16x16x128_f8f6f4, with
// the same reduction bytes per lane and the same order along K as the large
// tiles, so every shape rounds every element alike.
//
// What bounds a small tile is latency, not the MFMAs: a K tile is 128 (64 x 64)
// to 512 (128 x 128) MFMA cycles per SIMD, against about 2000 cycles from an
// LDS-bound load's issue to its data.  So K tiles go through a ring of S LDS
// stages, loaded S tiles ahead (global_load_lds, no staging registers), and
// fragments are double-buffered in registers: step t multiplies tile t from
// registers while tile t + 1's fragments are read from LDS.  One barrier per
// step publishes tile t + 1 and frees tile t's stage, whose next loads (tile
// t + S) are issued right behind it.  The last, partial K tile is loaded the
// same way (chunks past the row's last 16 bytes re-read that chunk) and masked
// in the fragments.
//
// The epilogue stages 64 output rows at a time in LDS and stores whole row
// runs, four columns per lane at any alignment.  (Rows that are not
// vector-aligned went one element per lane before; MI355X, us: 4100 x 4100 x
// 1040 into rows of 4103, BF16 46 -> 34, FP32 46 -> 39, accumulated 60 -> 49;
// 8191 x 8191 x 2049 FP32 219 -> 181, accumulated 254 -> 216.)
#include "gemm_util.h"
#include "scale_update.h"

namespace qe {
namespace {

// Bytes [0, valid) of a 32-byte fragment kept, the rest zeroed.
__device__ __forceinline__ v8i mask_frag(v8i f, int valid) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int nb = valid - 4 * q;
    const int k = nb <= 0 ? 0 : (nb >= 4 ? 4 : nb);
    f[q] &= int(uint32_t((uint64_t(1) << (8 * k)) - 1u));
  }
  return f;
}

// Two workgroups per compute unit where the LDS holds two.  Their 256 registers
// per lane then suffice without a spill, the 128 x 128 tile with 224, as long as
// the compiler is kept from packed FP32 instructions: with them the same source
// takes 256 and spills 70, and every reload in the K loop would wait for the
// LDS-bound loads in flight.  test_kernel_resources.py checks the built library.
template <int FA, int FB, int BM, int BN, int S>
__global__ __launch_bounds__(256, (BM + BN) * BK * S > 81920 ? 1 : 2) void gemm_tn_ring_kernel(
    GemmParams g, int tiles_m, int tiles_n, int nt, UpdateParams upd) {
  static_assert(BM % 64 == 0 && BN % 64 == 0 && S >= 2, "tile sizes");
  constexpr int NW = 4, TM = BM / 2, TN = BN / 2;
  constexpr int I = TM / 16, J = TN / 16;
  constexpr int CHA = BM / 32, CHB = BN / 32;  // LDS-bound loads per lane per K tile
  constexpr int L = CHA + CHB;
  constexpr int Q = I * J;                     // MFMAs per wave and K tile
  constexpr int STAGE = (BM + BN) * BK;
  constexpr int ER = 64;                       // output rows staged at a time
  constexpr int EP = BN + 4;                   // staging row, in floats (padded)
  static_assert(ER * EP * 4 <= S * STAGE, "epilogue staging fits in the stages");
  static_assert((S - 1) * L < 64, "the load counter holds 63");
  __shared__ __attribute__((aligned(16))) uint8_t smem[S * STAGE];
  static_assert(sizeof(smem) >= (kMaxHistory + kUpdateThreads / 64) * 4, "history staging fits in the stages");

  // Workgroups past the tiles run the delayed scale update of the action's
  // roles beside them (the tiles read only scale_inv snapshots).
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

  const int64_t M = g.m, N = g.n;
  const int K = int(g.k);
  const int ktail = K % BK;
  const int T = K / BK + (ktail > 0 ? 1 : 0);

  // Load c of a wave fills 8 rows x 128 bytes; lane l fetches the chunk that
  // the swizzle puts at row 8 b + l / 8, physical chunk l % 8.
  const int lrow = lane >> 3;
  uint32_t oa[CHA], ob[CHB];
#pragma unroll
  for (int c = 0; c < CHA; ++c) {
    const int row = 8 * (wave + NW * c) + lrow;
    oa[c] = uint32_t(min(m0 + row, M - 1) * g.lda) + ((lane & 7) ^ row_swizzle(row)) * 16;
  }
#pragma unroll
  for (int c = 0; c < CHB; ++c) {
    const int row = 8 * (wave + NW * c) + lrow;
    ob[c] = uint32_t(min(n0 + row, N - 1) * g.ldb) + ((lane & 7) ^ row_swizzle(row)) * 16;
  }
  const uint32_t lds_base = uint32_t(reinterpret_cast<uintptr_t>(smem));
  const uint32_t wblk = __builtin_amdgcn_readfirstlane(lds_base + uint32_t(wave) * 1024u);

  auto load16 = [](uint32_t off, const uint8_t *base, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds)
                 : "memory", "m0");
  };
  auto issue = [&](int t, uint32_t stage) {
    const uint8_t *ga = g.a + int64_t(t) * BK;
    const uint8_t *gb = g.b + int64_t(t) * BK;
    const uint32_t sa = wblk + stage, sb = sa + uint32_t(BM * BK);
    if (ktail == 0 || t + 1 < T) {
#pragma unroll
      for (int c = 0; c < CHA; ++c) load16(oa[c], ga, sa + uint32_t(c * NW * 1024));
#pragma unroll
      for (int c = 0; c < CHB; ++c) load16(ob[c], gb, sb + uint32_t(c * NW * 1024));
    } else {  // chunks past the row's last 16 bytes re-read its last chunk; the fragments mask them
      const int last = (ktail - 1) >> 4;
#pragma unroll
      for (int c = 0; c < CHA; ++c) {
        const int row = 8 * (wave + NW * c) + lrow;
        const int ch = (lane & 7) ^ row_swizzle(row);
        load16(oa[c] - uint32_t(max(ch - last, 0) * 16), ga, sa + uint32_t(c * NW * 1024));
      }
#pragma unroll
      for (int c = 0; c < CHB; ++c) {
        const int row = 8 * (wave + NW * c) + lrow;
        const int ch = (lane & 7) ^ row_swizzle(row);
        load16(ob[c] - uint32_t(max(ch - last, 0) * 16), gb, sb + uint32_t(c * NW * 1024));
      }
    }
  };

  // 16-row fragments: lane l holds row (l & 15), bytes 32 (l >> 4) .. +31 of
  // the K tile (the layout of the large tiles).
  const int fr = lane & 15, fq = lane >> 4;
  const uint32_t f_lo = uint32_t(fr) * BK + uint32_t((2 * fq) ^ row_swizzle(fr)) * 16;
  const uint32_t f_hi = uint32_t(fr) * BK + uint32_t((2 * fq + 1) ^ row_swizzle(fr)) * 16;
  auto frag = [&](uint32_t base) -> v8i {
    const uint4 lo = *reinterpret_cast<const uint4 *>(smem + base + f_lo);
    const uint4 hi = *reinterpret_cast<const uint4 *>(smem + base + f_hi);
    return v8i{int(lo.x), int(lo.y), int(lo.z), int(lo.w), int(hi.x), int(hi.y), int(hi.z), int(hi.w)};
  };
  struct Frags {
    v8i a[I], b[J];
  };
  auto read = [&](uint32_t stage, Frags &f) {
#pragma unroll
    for (int i = 0; i < I; ++i) f.a[i] = frag(stage + uint32_t((wm * TM + i * 16) * BK));
#pragma unroll
    for (int j = 0; j < J; ++j) f.b[j] = frag(stage + uint32_t((BM + wn * TN + j * 16) * BK));
  };
  auto mask = [&](Frags &f) {
    const int valid = ktail - 32 * fq;
#pragma unroll
    for (int i = 0; i < I; ++i) f.a[i] = mask_frag(f.a[i], valid);
#pragma unroll
    for (int j = 0; j < J; ++j) f.b[j] = mask_frag(f.b[j], valid);
  };

  v4f acc[I][J];
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  auto mfma = [&](int i, int j, const Frags &f) {
    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f.b[j], f.a[i], acc[i][j], FB, FA, 0, 0, 0, 0);
  };
  uint32_t rd = 0;  // stage of tile t
  // Step t: fragments of tile t are in `cur`; tile t + 1's are read into `nxt`.
  // main_step (tile t + S exists and is full): after each MFMA, in a fixed
  // order, one LDS-bound load and one fragment read where they are due, so the
  // three pipes (MFMA, LDS, address) work side by side in a single wave.
  auto main_step = [&](int t, const Frags &cur, Frags &nxt) {
    // tile t + 1 complete: of the tiles issued so far, t + 2 .. t + S - 1 may
    // still be in flight (the counter completes in order)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * L) : "memory");
    __syncthreads();  // tile t + 1 published; every wave holds tile t's fragments
    const uint8_t *ga = g.a + int64_t(t + S) * BK;
    const uint8_t *gb = g.b + int64_t(t + S) * BK;
    const uint32_t sa = wblk + rd;  // tile t's stage takes tile t + S; load d lands at sa + 4096 d
    rd = rd + STAGE == uint32_t(S * STAGE) ? 0u : rd + STAGE;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < L; ++d)
        if (d * Q / L == q) {
          if (d == 0)
            asm volatile("s_mov_b32 m0, %0" ::"s"(sa) : "m0");
          else
            asm volatile("s_add_u32 m0, m0, %0" ::"n"(NW * 1024) : "m0", "scc");
        }
      __builtin_amdgcn_sched_barrier(0);  // M0 is written before the MFMA, never next to the load
      mfma(q / J, q % J, cur);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < L; ++d)
        if (d * Q / L == q) {
          if (d < CHA)
            asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(oa[d]), "s"(ga) : "memory");
          else
            asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(ob[d - CHA]), "s"(gb) : "memory");
        }
#pragma unroll
      for (int r = 0; r < I + J; ++r)
        if (r * Q / (I + J) == q) {
          if (r < I)
            nxt.a[r] = frag(rd + uint32_t((wm * TM + r * 16) * BK));
          else
            nxt.b[r - I] = frag(rd + uint32_t((BM + wn * TN + (r - I) * 16) * BK));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // The last steps: no tile, or the partial one, left to issue.  (Past the last
  // tile a stale stage is read and never used, so that the reads stay
  // branch-free and the compiler can wait for them one by one.)
  auto last_step = [&](int t, const Frags &cur, Frags &nxt) {
    if (t + S <= T)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * L) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const uint32_t freed = rd;
    rd = rd + STAGE == uint32_t(S * STAGE) ? 0u : rd + STAGE;
    read(rd, nxt);
    __builtin_amdgcn_sched_barrier(0);
    if (t + S < T) issue(t + S, freed);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < Q; ++q) mfma(q / J, q % J, cur);
    __builtin_amdgcn_sched_barrier(0);
    if (t + 2 == T && ktail != 0) mask(nxt);
  };

  if (T > 0) {
    Frags f0, f1;
#pragma unroll
    for (int t = 0; t < S; ++t)
      if (t < T) issue(t, uint32_t(t * STAGE));
    if (T >= S)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * L) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    read(0, f0);
    if (T == 1 && ktail != 0) mask(f0);
    int t = 0;
    for (; t + 1 + S < K / BK; t += 2) {
      main_step(t, f0, f1);
      main_step(t + 1, f1, f0);
    }
    for (; t + 1 < T; t += 2) {
      last_step(t, f0, f1);
      last_step(t + 1, f1, f0);
    }
    if (t < T) {
#pragma unroll
      for (int q = 0; q < Q; ++q) mfma(q / J, q % J, f0);
    }
  }

  // Epilogue: BM / 64 passes of 64 rows through LDS.  Accumulating, a pass
  // reads its destination before it stages its rows, all loads in flight.
  // Accesses are non-temporal, as in the large tiles, unless launch_ring says
  // otherwise.
  const int e = pow2_exponent(g.a_scale_inv) + pow2_exponent(g.b_scale_inv);
  float *ep = reinterpret_cast<float *>(smem);
  constexpr int RW = ER < TM ? ER : TM;  // rows a wave stages per pass
  constexpr int NQ = ER * BN / 4 / 256;  // column quads per lane and pass
  const int cols = int(min(int64_t(BN), N - n0));
  // lane's first column quad of a pass and its step in rows
  const int rv = tid / (BN / 4), cv = (tid % (BN / 4)) * 4;
  constexpr int DV = 1024 / BN;
#pragma unroll
  for (int p = 0; p < BM / ER; ++p) {
    const int64_t r0 = m0 + p * ER;
    const int rows = int(min(int64_t(ER), M - r0));
    const int64_t ov = (r0 + rv) * g.ldc + n0 + cv;
    v4f pre[NQ];
    if (g.out == 2) {
      const float *d = static_cast<const float *>(g.c) + ov;
#pragma unroll
      for (int it = 0; it < NQ; ++it) {
        pre[it] = v4f{0.f, 0.f, 0.f, 0.f};
        if (rv + it * DV < rows && cv + 4 <= cols)
          pre[it] = nt ? __builtin_nontemporal_load(reinterpret_cast<const v4f_out *>(d + it * (DV * g.ldc)))
                       : v4f(*reinterpret_cast<const v4f_out *>(d + it * (DV * g.ldc)));
      }
    }
    __syncthreads();  // the last reads of the stages (or of the previous pass) are done
    if (TM < ER || wm == p * ER / TM) {
#pragma unroll
      for (int i = 0; i < RW / 16; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const v4f a = acc[TM < ER ? i : (p * ER % TM) / 16 + i][j];
          *reinterpret_cast<float4 *>(ep + ((TM < ER ? wm * TM : 0) + i * 16 + fr) * EP + wn * TN + j * 16 + 4 * fq) =
              make_float4(__builtin_ldexpf(a[0], e), __builtin_ldexpf(a[1], e), __builtin_ldexpf(a[2], e),
                          __builtin_ldexpf(a[3], e));
        }
    }
    __syncthreads();
    const float *lv = ep + rv * EP + cv;
#pragma unroll
    for (int it = 0; it < NQ; ++it) {
      if (rv + it * DV >= rows || cv >= cols) continue;
      v4f v = *reinterpret_cast<const v4f *>(lv + it * DV * EP);
      const int64_t o = ov + it * (DV * g.ldc);
      if (cv + 4 <= cols) {
        if (g.out == 1) {
          const v2i w = {int(bf16x2_bits(v[0], v[1])), int(bf16x2_bits(v[2], v[3]))};
          uint16_t *dst = static_cast<uint16_t *>(g.c) + o;
          if (nt)
            __builtin_nontemporal_store(w, reinterpret_cast<v2i_out *>(dst));
          else
            *reinterpret_cast<v2i_out *>(dst) = w;
        } else {
          if (g.out == 2) v += pre[it];
          float *dst = static_cast<float *>(g.c) + o;
          if (nt)
            __builtin_nontemporal_store(v, reinterpret_cast<v4f_out *>(dst));
          else
            *reinterpret_cast<v4f_out *>(dst) = v;
        }
      } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          if (cv + k >= cols) break;
          if (g.out == 1)
            static_cast<uint16_t *>(g.c)[o + k] = bf16_bits(v[k]);
          else if (g.out == 2)
            static_cast<float *>(g.c)[o + k] += v[k];
          else
            static_cast<float *>(g.c)[o + k] = v[k];
        }
      }
    }
  }
}

template <int BM, int BN, int S>
hipError_t launch_ring(const GemmParams &g, hipStream_t s, const UpdateParams &u) {
  const int tiles_m = int((g.m + BM - 1) / BM), tiles_n = int((g.n + BN - 1) / BN);
  // Accumulating into rows that are not vector-aligned, lanes and workgroups
  // share cache lines; while the destination is small enough to stay in the
  // 256 MB memory-side cache, ordinary accesses merge them there.  Measured on
  // MI355X (us, non-temporal / ordinary): 4100 x 4100 x 1040 accumulated 53.5 /
  // 45.7, 2730 x 1365 x 1000 17.6 / 14.1, but 8191 x 8191 x 2049 217 / 243; FP32
  // stores of the last 174 / 208.
  const int nt = g.out != 2 || gemm_vec_ok(g) || g.m * g.n > (int64_t(32) << 20);
  const dim3 grid(unsigned(tiles_m) * unsigned(tiles_n) + unsigned(u.n)), block(256);
  if (g.fmt_a == 0 && g.fmt_b == 0) return klaunch(gemm_tn_ring_kernel<0, 0, BM, BN, S>, grid, block, 0, s, g, tiles_m, tiles_n, nt, u);
  if (g.fmt_a == 1 && g.fmt_b == 0) return klaunch(gemm_tn_ring_kernel<1, 0, BM, BN, S>, grid, block, 0, s, g, tiles_m, tiles_n, nt, u);
  if (g.fmt_a == 0 && g.fmt_b == 1) return klaunch(gemm_tn_ring_kernel<0, 1, BM, BN, S>, grid, block, 0, s, g, tiles_m, tiles_n, nt, u);
  return klaunch(gemm_tn_ring_kernel<1, 1, BM, BN, S>, grid, block, 0, s, g, tiles_m, tiles_n, nt, u);
}

}  // namespace

hipError_t launch_gemm_ring(int tile, const GemmParams &g, hipStream_t s, const UpdateParams &u) {
  switch (tile) {
    case kTile256x128: return launch_ring<256, 128, 3>(g, s, u);
    case kTile64x64: return launch_ring<64, 64, 4>(g, s, u);
    case kTile128x64: return launch_ring<128, 64, 3>(g, s, u);
    case kTile128x64Deep: return launch_ring<128, 64, 6>(g, s, u);
    case kTile64x128: return launch_ring<64, 128, 3>(g, s, u);
    case kTile64x128Deep: return launch_ring<64, 128, 6>(g, s, u);
    case kTile128x128: return launch_ring<128, 128, 2>(g, s, u);
    default: return launch_ring<128, 128, 4>(g, s, u);
  }
}

}  // namespace qe
