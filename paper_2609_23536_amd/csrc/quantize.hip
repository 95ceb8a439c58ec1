// FP8 quantization with fused transpose and amax recording (gfx950).
//
// Delayed scaling (§2.1 of the paper): a tensor is cast with the scale the
// previous update produced, and its amax is recorded for later updates.  The
// split backward (§3.2) needs each operand both row-wise (for F / dI) and
// column-wise (for the deferred dW), so one pass writes both:
//   q_row[r][c] = Q(x[r][c] * scale),  q_col[c][r] = the same code,
//   history[0]  = max(history[0], max |x|)      (unscaled, NaN propagates)
// Q rounds to nearest even and saturates to +-fmax; NaN becomes 0x7F with the
// input's sign bit.  Formats: OCP E4M3 (max 448) and E5M2 (max 57344).
//
// Layout: one workgroup of 256 lanes per tile of 128 rows (64 for small tensors)
// x 128 columns.  Phase 1: every load
// instruction is one contiguous 16-byte piece per lane along a row (16 lanes
// per bf16 row, 32 per fp32 row); each lane converts its 8 (or 4) values and
// stores the codes row-wise and into an LDS tile whose 16-byte chunks are
// XOR-swizzled by row block.
// Phase 2: each lane gathers a 16-row (8-row) x 4-column block of codes from LDS
// and writes four 16-byte (8-byte) column segments; eight consecutive lanes
// complete one 128-byte (64-byte) run of a transposed row.  amax: a max over the |x| bit patterns
// (which order like the values, NaN above inf) per lane, a wave shuffle
// reduction, then one atomicMax per workgroup into one of the 64 lines of the
// role's amax accumulator (same-line atomics serialise).  HBM-bound: per element it
// moves 2 or 4 bytes in and 2 bytes out.
//
// Rows need no alignment beyond the element's: the global accesses are the same
// single 16-, 8- and 4-byte instructions at any address (unaligned access is
// the normal mode of the device), and a tile at the tensor's edge guards each
// of them instead of falling back to single elements.  Measured on MI355X, one
// step of a 1365 x 2730 layer with two 1000-token microbatches (no row 16-byte
// aligned): 236 us with single elements, 151 us so; 1500 x 4099 fp32 current
// cast, with the scale derived in the cast (CurrentParams): 46 -> 19 us.
#include "scale_update.h"

#include <type_traits>

namespace qe {
namespace {

constexpr int kTile = 128;
constexpr int kThreads = 256;

// Vectors at element (input) and byte (code) alignment.
typedef unsigned int u32x4_in __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int u32x4_out __attribute__((ext_vector_type(4), aligned(1)));
typedef unsigned int u32x2_out __attribute__((ext_vector_type(2), aligned(1)));
typedef unsigned int u32_out __attribute__((aligned(1)));

// Four scaled values -> four FP8 codes, byte i = value i.  The hardware
// conversion rounds to nearest even but neither saturates (it overflows to
// NaN / inf) nor keeps the sign of a NaN, so values are clamped first with
// med3, which maps NaN to -fmax; NaN inputs are repaired separately.
template <int FMT>
__device__ __forceinline__ uint32_t enc4(float a, float b, float c, float d) {
  constexpr float fm = FMT == 0 ? 448.0f : 57344.0f;
  const float ca = __builtin_amdgcn_fmed3f(a, -fm, fm);
  const float cb = __builtin_amdgcn_fmed3f(b, -fm, fm);
  const float cc = __builtin_amdgcn_fmed3f(c, -fm, fm);
  const float cd = __builtin_amdgcn_fmed3f(d, -fm, fm);
  int r;
  if constexpr (FMT == 0) {
    r = __builtin_amdgcn_cvt_pk_fp8_f32(ca, cb, 0, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(cc, cd, r, true);
  } else {
    r = __builtin_amdgcn_cvt_pk_bf8_f32(ca, cb, 0, false);
    r = __builtin_amdgcn_cvt_pk_bf8_f32(cc, cd, r, true);
  }
  return uint32_t(r);
}

// NaN -> 0x7F with the input's sign bit, for the rare thread that saw one.
__device__ __forceinline__ uint32_t nan_fix(uint32_t u, int byte, float v) {
  if (v != v) {
    const uint32_t code = 0x7fu | ((__float_as_uint(v) >> 24) & 0x80u);
    u = (u & ~(0xffu << (8 * byte))) | (code << (8 * byte));
  }
  return u;
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

__device__ __forceinline__ uint32_t abs_bits(float v) { return __float_as_uint(v) & 0x7fffffffu; }

// A lane of phase 2 reads RPL consecutive rows; the swizzle follows its block.
template <int RPL>
__device__ __forceinline__ uint32_t lds_chunk_offset(int row, int chunk) {
  return uint32_t(row) * kTile + (uint32_t((chunk ^ (row / RPL)) & 7) << 4);
}

__device__ __forceinline__ uint32_t byte_of(uint32_t w, int j) { return (w >> (8 * j)) & 0xffu; }

// E values of one 16-byte input load (8 bf16 or 4 fp32), as floats
template <bool BF16>
__device__ __forceinline__ void unpack16(const uint4 &v, float *f) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  if constexpr (BF16) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = bf16_to_f32(w[e] & 0xffffu);
      f[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(w[e]);
  }
}

// One launch casts one tensor, or two independent ones (the forward's weight
// refresh and input cast) whose tiles follow each other in one grid, so the
// second tensor's tiles fill the first one's tail instead of a second launch
// ramping up after it.
struct QuantJob {
  QuantParams p;
  int64_t tiles, tiles_c;
};
struct QuantPair {
  QuantJob j[2];
  int32_t n, pad;
};

// CUR: the cast of a current-scaling role derives its own scale (see scale_of).
template <bool BF16, int FMT, bool CUR, int ROWS>
__device__ __forceinline__ void quantize_body(const QuantPair &pp, const CurrentParams &cp) {
  __shared__ __attribute__((aligned(16))) uint8_t tile[ROWS * kTile];
  __shared__ uint32_t red[kThreads / 64];
  // Phase 1 mapping: one 16-byte load per lane per step, consecutive lanes on
  // consecutive 16 bytes of a row (LPR lanes per 128-element row).
  constexpr int EPL = BF16 ? 8 : 4;          // elements per load
  constexpr int LPR = kTile / EPL;           // lanes per tile row
  constexpr int NLD = ROWS * kTile / (EPL * kThreads);  // loads per lane
  constexpr int RPL = ROWS / 8;              // rows per lane in phase 2
  const int tid = threadIdx.x;
  const bool second = pp.n > 1 && int64_t(blockIdx.x) >= pp.j[0].tiles;  // uniform per workgroup
  const QuantJob &job = second ? pp.j[1] : pp.j[0];
  const QuantParams &p = job.p;
  const int64_t tiles_c = job.tiles_c;
  const int64_t t = second ? int64_t(blockIdx.x) - pp.j[0].tiles : int64_t(blockIdx.x);
  const int64_t r0 = (t / tiles_c) * ROWS;
  const int64_t c0 = (t % tiles_c) * kTile;
  // The scale.  Under CUR every workgroup reduces the amax pass's partial
  // maxima (at most kMaxPartials floats, from the L2) instead of waiting for
  // an update kernel; the first one stores the role's new state, which the
  // others never read: they read the live scale only where the amax leaves it
  // as it is.
  auto scale_of = [&]() -> float {
    if constexpr (!CUR) {
      if (t == 0 && tid == 0 && p.snapshot != nullptr) *p.snapshot = *p.scale_inv;
      return *p.scale;
    } else {
      uint32_t a = 0;
#pragma unroll
      for (int k = 0; k < kMaxPartials / kThreads; ++k)
        if (k * kThreads + tid < cp.n) {
          const uint32_t b = __float_as_uint(cp.partials[k * kThreads + tid]);
          a = b > a ? b : a;
        }
      a = update_wave_max(a);
      if ((tid & 63) == 0) red[tid >> 6] = a;
      __syncthreads();
      a = red[0];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) a = red[w] > a ? red[w] : a;
      int e;
      const bool valid = update_exponent(a, cp.m.fmt, cp.m.margin, &e);
      const float sc = valid ? __uint_as_float(uint32_t(e + 127) << 23) : *p.scale;
      if (t == 0 && tid == 0) {
        const float inv = valid ? __uint_as_float(uint32_t(127 - e) << 23) : *p.scale_inv;
        if (valid) {
          *cp.m.scale = sc;
          *cp.m.scale_inv = inv;
        }
        cp.m.hist[0] = 0.0f;
        if (p.snapshot != nullptr) *p.snapshot = inv;
        if (cp.token != nullptr) __hip_atomic_fetch_add(cp.token, 1ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      return sc;
    }
  };
  const float scale = scale_of();
  const bool full = r0 + ROWS <= p.rows && c0 + kTile <= p.cols;
  uint32_t amax = 0;

  // Phase 1, for whole tiles (EDGE false) and tiles at the tensor's edge: a
  // lane's elements past the last column or row count as zero and are not
  // stored.  Edge tiles take their steps in two groups; both paths share one
  // register allocation (128 rows: bf16 145 VGPRs and 26 scalars kept in VGPR
  // lanes, fp32 134, three waves per SIMD).  Four groups take bf16 to 144 and
  // no such scalars, which whole tiles do not notice (4096 x 4096 15.3 us
  // either way) and edge tiles do (8192 x 8208 57.3 -> 58.7, 5000 x 4099 21.5
  // -> 22.1); fp32 held to 128 VGPRs for a fourth wave is slower (4096 x 4096
  // 22.5 -> 23.0, with its scale update).
  auto cast_tile = [&](auto edge) {
    constexpr bool EDGE = decltype(edge)::value;
    // valid elements of the lane's piece of step `it`
    auto valid = [&](int it) -> int {
      const int q = it * kThreads + tid;
      const int64_t left = r0 + q / LPR < p.rows ? p.cols - (c0 + q % LPR * EPL) : 0;
      return left <= 0 ? 0 : (left >= EPL ? EPL : int(left));
    };
    constexpr int G = EDGE ? NLD / 2 : NLD;
#pragma unroll 1
    for (int g = 0; g < NLD; g += G) {
      uint4 raw[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int q = (g + u) * kThreads + tid, row = q / LPR, cl = q % LPR;
        const int64_t eoff = (r0 + row) * p.cols + c0 + cl * EPL;
        const char *src = static_cast<const char *>(p.in) + eoff * (BF16 ? 2 : 4);
        if constexpr (!EDGE) {
          const u32x4_in x = __builtin_nontemporal_load(reinterpret_cast<const u32x4_in *>(src));
          raw[u] = make_uint4(x.x, x.y, x.z, x.w);
        } else {
          const int n = valid(g + u);
          raw[u] = make_uint4(0u, 0u, 0u, 0u);
          if (n > 0) {
            if (eoff + EPL <= p.rows * p.cols) {  // may run into the next row; masked below
              const u32x4_in x = *reinterpret_cast<const u32x4_in *>(src);
              raw[u] = make_uint4(x.x, x.y, x.z, x.w);
            } else {  // the tensor's last elements
              uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
              for (int e = 0; e < EPL; ++e) {
                if (e >= n) break;
                if constexpr (BF16)
                  w[e / 2] |= uint32_t(reinterpret_cast<const uint16_t *>(src)[e]) << (16 * (e % 2));
                else
                  w[e] = reinterpret_cast<const uint32_t *>(src)[e];
              }
              raw[u] = make_uint4(w[0], w[1], w[2], w[3]);
            }
          }
        }
      }
      auto values = [&](int u, float *f) {
        unpack16<BF16>(raw[u], f);
        if constexpr (EDGE) {
          const int n = valid(g + u);
#pragma unroll
          for (int e = 0; e < EPL; ++e) f[e] = e < n ? f[e] : 0.0f;
        }
      };
      uint32_t codes[G][EPL / 4];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        float f[EPL];
        values(u, f);
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const uint32_t b = abs_bits(f[e]);
          amax = b > amax ? b : amax;
        }
#pragma unroll
        for (int w = 0; w < EPL / 4; ++w)
          codes[u][w] = enc4<FMT>(f[4 * w] * scale, f[4 * w + 1] * scale, f[4 * w + 2] * scale, f[4 * w + 3] * scale);
      }
      if (__builtin_expect(amax > 0x7f800000u, 0)) {  // this lane saw a NaN
#pragma unroll
        for (int u = 0; u < G; ++u) {
          float f[EPL];
          values(u, f);
#pragma unroll
          for (int e = 0; e < EPL; ++e) codes[u][e / 4] = nan_fix(codes[u][e / 4], e % 4, f[e]);
        }
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int q = (g + u) * kThreads + tid, row = q / LPR, cl = q % LPR;
        const int col = cl * EPL;
        uint8_t *lds = tile + lds_chunk_offset<RPL>(row, col >> 4) + (col & 15);
        if constexpr (BF16)
          *reinterpret_cast<uint2 *>(lds) = make_uint2(codes[u][0], codes[u][1]);
        else
          *reinterpret_cast<uint32_t *>(lds) = codes[u][0];
        if (p.q_row == nullptr) continue;
        uint8_t *dst = p.q_row + (r0 + row) * p.ld_row + c0 + col;
        const int n = EDGE ? valid(g + u) : EPL;
        if (!EDGE || n == EPL) {
          if constexpr (BF16)
            *reinterpret_cast<u32x2_out *>(dst) = u32x2_out{codes[u][0], codes[u][1]};
          else
            *reinterpret_cast<u32_out *>(dst) = codes[u][0];
        } else {
#pragma unroll
          for (int e = 0; e < EPL; ++e)
            if (e < n) dst[e] = uint8_t(byte_of(codes[u][e / 4], e % 4));
        }
      }
    }
  };
  if (full)
    cast_tile(std::false_type{});
  else
    cast_tile(std::true_type{});

  // amax: wave shuffle reduction, then one atomic per workgroup
  if constexpr (CUR) {
    __syncthreads();
  } else {
    amax = update_wave_max(amax);
    if ((tid & 63) == 0) red[tid >> 6] = amax;
    __syncthreads();
    if (tid == 0) {
      uint32_t a = red[0];
      for (int w = 1; w < kThreads / 64; ++w) a = red[w] > a ? red[w] : a;
      fold_amax(p.amax_accum, p.amax_slot, a);
    }
  }

  if (p.q_col == nullptr) return;
  // Phase 2: lane (rb, cq) transposes RPL rows from rb*RPL x columns 4cq..4cq+3.
  // Whole tiles have a loop of their own, without the guards (bf16 4096 x 4096,
  // in one run with a common loop: 15.35 -> 15.00 us, fp32 8192 x 8192 65.4 -> 65.2).
  const int rb = tid & 7, cq = tid >> 3;
  uint32_t d[RPL];
#pragma unroll
  for (int i = 0; i < RPL; ++i) {
    const int R = rb * RPL + i;
    d[i] = *reinterpret_cast<const uint32_t *>(tile + lds_chunk_offset<RPL>(R, cq >> 2) + ((cq & 3) << 2));
  }
  auto segment = [&](int j, uint32_t *w) -> uint8_t * {
#pragma unroll
    for (int q = 0; q < RPL / 4; ++q)
      w[q] = byte_of(d[4 * q], j) | (byte_of(d[4 * q + 1], j) << 8) | (byte_of(d[4 * q + 2], j) << 16) |
             (byte_of(d[4 * q + 3], j) << 24);
    return p.q_col + (c0 + 4 * cq + j) * p.ld_col + r0 + rb * RPL;
  };
  auto store = [](uint8_t *dst, const uint32_t *w) {
    if constexpr (RPL == 16)
      *reinterpret_cast<u32x4_out *>(dst) = u32x4_out{w[0], w[1], w[2], w[3]};
    else
      *reinterpret_cast<u32x2_out *>(dst) = u32x2_out{w[0], w[1]};
  };
  if (full) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t w[RPL / 4];
      uint8_t *dst = segment(j, w);
      store(dst, w);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t w[RPL / 4];
    uint8_t *dst = segment(j, w);
    if (c0 + 4 * cq + j >= p.cols) continue;
    const int64_t n = p.rows - (r0 + rb * RPL);
    if (n >= RPL) {
      store(dst, w);
    } else {  // the last rows: whole words, then bytes
#pragma unroll
      for (int q = 0; q < RPL / 4; ++q) {
        if (4 * q + 4 <= n) {
          *reinterpret_cast<u32_out *>(dst + 4 * q) = w[q];
        } else {
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (4 * q + e < n) dst[4 * q + e] = uint8_t(byte_of(w[q], e));
        }
      }
    }
  }
}

template <bool BF16, int FMT, int ROWS>
__global__ __launch_bounds__(kThreads) void quantize_kernel(QuantPair pp) {
  quantize_body<BF16, FMT, false, ROWS>(pp, CurrentParams{});
}

template <bool BF16, int FMT, int ROWS>
__global__ __launch_bounds__(kThreads) void quantize_current_kernel(QuantPair pp, CurrentParams cp) {
  quantize_body<BF16, FMT, true, ROWS>(pp, cp);
}

int64_t tiles_of(const QuantParams &p, int rows) {
  const int64_t n = ((p.rows + rows - 1) / rows) * ((p.cols + kTile - 1) / kTile);
  return n < 1 ? 1 : n;  // an empty tensor still writes the scale_inv snapshot
}

QuantJob make_job(const QuantParams &p, int rows) {
  QuantJob j;
  memset(&j, 0, sizeof(j));  // padding too: recorded launches are compared bytewise
  j.p = p;
  const int64_t tiles_c = (p.cols + kTile - 1) / kTile;
  j.tiles = tiles_of(p, rows);
  j.tiles_c = tiles_c < 1 ? 1 : tiles_c;
  return j;
}

template <int ROWS>
hipError_t launch_rows(const QuantParams *p, int n, const CurrentParams *cp, hipStream_t s) {
  QuantPair pp;
  memset(&pp, 0, sizeof(pp));
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    pp.j[i] = make_job(p[i], ROWS);
    tiles += pp.j[i].tiles;
  }
  pp.n = n;
  const dim3 grid{unsigned(tiles)}, block(kThreads);
  const bool e4m3 = p[0].fmt == 0;
  if (cp != nullptr) {
    if (p[0].in_bf16)
      return e4m3 ? klaunch(quantize_current_kernel<true, 0, ROWS>, grid, block, 0, s, pp, *cp)
                  : klaunch(quantize_current_kernel<true, 1, ROWS>, grid, block, 0, s, pp, *cp);
    return e4m3 ? klaunch(quantize_current_kernel<false, 0, ROWS>, grid, block, 0, s, pp, *cp)
                : klaunch(quantize_current_kernel<false, 1, ROWS>, grid, block, 0, s, pp, *cp);
  }
  if (p[0].in_bf16)
    return e4m3 ? klaunch(quantize_kernel<true, 0, ROWS>, grid, block, 0, s, pp)
                : klaunch(quantize_kernel<true, 1, ROWS>, grid, block, 0, s, pp);
  return e4m3 ? klaunch(quantize_kernel<false, 0, ROWS>, grid, block, 0, s, pp)
              : klaunch(quantize_kernel<false, 1, ROWS>, grid, block, 0, s, pp);
}

// Up to two 128-row tiles per compute unit the tiles take 64 rows: twice the
// workgroups, half the chain of loads and edge guards in each.  Measured on
// MI355X (us, 128 rows -> 64): fp32 1000 x 2730 10.3 -> 7.6, 1500 x 4099 12.8 ->
// 11.8, 2048 x 4096 (512 tiles) 11.7 -> 11.0; bf16 1000 x 2730 8.5 -> 7.7,
// 2048 x 4096 level; one step of the 1365 x 2730 layer above 141 -> 131.
// Beyond, the 64-byte runs of the transposed codes cost more: bf16 4096 x
// 14336 46 -> 50, 57344 x 8192 321 -> 335, fp32 495 -> 554.
constexpr int64_t kSmallTiles = 512;

hipError_t launch_casts(const QuantParams *p, int n, const CurrentParams *cp, hipStream_t s) {
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) tiles += tiles_of(p[i], kTile);
  return tiles <= kSmallTiles ? launch_rows<64>(p, n, cp, s) : launch_rows<kTile>(p, n, cp, s);
}

}  // namespace

hipError_t launch_quantize(const QuantParams &p, hipStream_t s) { return launch_casts(&p, 1, nullptr, s); }

hipError_t launch_quantize_current(const AmaxParams &a, const QuantParams &q, const MetaRef &m, long long *token,
                                   float *partials, hipStream_t s) {
  if (q.rows * q.cols == 0 || amax_blocks(a) > kMaxPartials) return hipErrorInvalidValue;
  AmaxParams ap = a;
  ap.partials = partials;
  CurrentParams cp;
  memset(&cp, 0, sizeof(cp));
  cp.m = m;
  cp.partials = partials;
  cp.n = amax_blocks(ap);
  cp.token = token;
  const hipError_t e = launch_amax(ap, s);
  return e != hipSuccess ? e : launch_casts(&q, 1, &cp, s);
}

hipError_t launch_quantize_pair(const QuantParams &a, const QuantParams &b, hipStream_t s) {
  if (a.in_bf16 != b.in_bf16 || a.fmt != b.fmt) {  // different kernel instances: two launches
    const hipError_t e = launch_quantize(a, s);
    return e != hipSuccess ? e : launch_quantize(b, s);
  }
  const QuantParams p[2] = {a, b};
  return launch_casts(p, 2, nullptr, s);
}

}  // namespace qe
