// gfx950 (CDNA4) kernels of the batched Muon step.
//
// Per chunk of same-shape matrices (Sec. 6.6 shape fusion):
//   k_prologue   momentum update in place, per-tile sums of u^2, and X~ = u
//                (unscaled), transpose-first, cast; writes X~ and X~^T (HBM-bound)
//   k_finalize   r = 1 / (||u||_F + eps) per matrix (fixed-order sum)
//   k_rescale    X0 = r*u for the rare matrices whose r the first products
//                cannot apply (see k_finalize); others exit at once
//   k_gemm_tile  the three contractions of Eq. (1) on MFMA, 256 x 256 or
//                128 x 128 tiles (bf16, or fp32 as three bf16 planes):
//                  A  = X X^T          (Gram, upper-triangle tiles only)
//                  B  = b A + c A A    (A is symmetric, so A A = A A^T)
//                  X' = a X + B X      (X read K-major by transposing LDS reads)
//                the last step's epilogue applies the update to W directly;
//   k_gemm_nt    the same on 128 x 128 tiles for rows past the tile kernel's
//                offsets (writes mirrored A and B and reads X^T);
//   k_slice_*    short sides up to 128 in column slices; k_ns_small the
//                smallest of them in one launch;
//   k_apply_x0   the update from X0 when K = 0;
//   k_adamw      AdamW for the parameters Muon does not take.
//
// All workspace buffers are zero-padded to multiples of 128 in both extents,
// so the contraction kernels never test bounds; zero padding is preserved by
// every step (padded rows/columns of X, A and B stay exactly zero).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>
#include <utility>

#include "muon_internal.h"

namespace muon {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// bfloat16 storage: uint16 bit patterns.  Widening is exact; narrowing is
// the hardware conversion (v_cvt_pk_bf16_f32): round to nearest, ties to
// even, NaN stays NaN, overflow to infinity.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}
// lo | hi << 16, both rounded as above, in one instruction
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ uint16_t from_f32<uint16_t>(float v) { return f32_to_bf16(v); }

__device__ __forceinline__ float load_as_f32(const void* p, int64_t i, int dt) {
  return dt == DT_BF16 ? bf16_to_f32(static_cast<const uint16_t*>(p)[i])
                       : static_cast<const float*>(p)[i];
}
__device__ __forceinline__ void store_from_f32(void* p, int64_t i, int dt, float v) {
  if (dt == DT_BF16) static_cast<uint16_t*>(p)[i] = f32_to_bf16(v);
  else static_cast<float*>(p)[i] = v;
}

// 8 consecutive elements at base + i (16-byte aligned) as fp32, and back
// (bf16 rounded to nearest even).
template <typename T>
__device__ __forceinline__ void load8(const T* base, int64_t i, float out[8]) {
  if constexpr (sizeof(T) == 2) {
    const u32x4_t raw = *reinterpret_cast<const u32x4_t*>(base + i);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      out[2 * q] = __uint_as_float(raw[q] << 16);
      out[2 * q + 1] = __uint_as_float(raw[q] & 0xffff0000u);
    }
  } else {
    const float4 a = *reinterpret_cast<const float4*>(base + i);
    const float4 b = *reinterpret_cast<const float4*>(base + i + 4);
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
    out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
  }
}

template <typename T>
__device__ __forceinline__ void store8(T* base, int64_t i, const float in[8]) {
  if constexpr (sizeof(T) == 2) {
    u32x4_t raw;
#pragma unroll
    for (int q = 0; q < 4; ++q) raw[q] = pack_bf16x2(in[2 * q], in[2 * q + 1]);
    *reinterpret_cast<u32x4_t*>(base + i) = raw;
  } else {
    *reinterpret_cast<float4*>(base + i) = make_float4(in[0], in[1], in[2], in[3]);
    *reinterpret_cast<float4*>(base + i + 4) = make_float4(in[4], in[5], in[6], in[7]);
  }
}

// An fp32 value kept as three bfloat16 planes, x = h + m + l: h is x rounded,
// m the rest rounded, l what then remains (at most 8 bits of x's 24, so the
// sum is exact unless l falls below bfloat16's range).  The fp32
// Newton-Schulz products on the tile kernel take their operands in this form.
struct Split3 {};
// How an iterate is stored: element type, planes, and the type its tiles take
// in the prologue's LDS transpose.
template <typename XT> struct Store { using E = XT; using L = XT; static constexpr int planes = 1; };
template <> struct Store<Split3> { using E = uint16_t; using L = float; static constexpr int planes = 3; };

template <typename XT>
__device__ __forceinline__ void store8x(typename Store<XT>::E* base, int64_t i, int64_t plane, const float in[8]) {
  if constexpr (std::is_same<XT, Split3>::value) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = in[q];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      u32x4_t raw;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        raw[q] = pack_bf16x2(v[2 * q], v[2 * q + 1]);
        v[2 * q] -= __uint_as_float(raw[q] << 16);
        v[2 * q + 1] -= __uint_as_float(raw[q] & 0xffff0000u);
      }
      *reinterpret_cast<u32x4_t*>(base + p * plane + i) = raw;
    }
  } else {
    store8(base, i, in);
  }
}

// Fixed-order sum over a 256-thread block: butterfly within each 64-lane
// wavefront, then the four wave sums in wave order.  Deterministic.  In fp64:
// the sums of u^2 stay finite for every finite u (|u| < 2^128 and at most
// 2^62 elements), where binary32 would overflow once |u| passes 2^64.
__device__ __forceinline__ double block_sum_256(double v, double* red4) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red4[wave] = v;
  __syncthreads();
  return ((red4[0] + red4[1]) + red4[2]) + red4[3];
}

// The factor r = 1 / (||u|| + eps) as two binary32 factors whose product is r
// (rounded once), each a normal number: r itself when it is one, else a power
// of two 2^-64 or 2^64 times the rest, for norms beyond 2^126 or below 2^-126.
__device__ __forceinline__ void split_scale(double r, float& s1, float& s2) {
  if (r < 0x1p-126 && r > 0.0) {
    s1 = 0x1p-64f;
    s2 = static_cast<float>(r * 0x1p64);
  } else if (r > 0x1p126) {
    s1 = 0x1p64f;
    s2 = static_cast<float>(r * 0x1p-64);
  } else {
    s1 = 1.0f;
    s2 = static_cast<float>(r);
  }
}

// ---------------------------------------------------------------------------
// Prologue, one pass over g and the momentum.  X0 = u / (||u|| + eps) needs
// the norm of all of u before any element of X0 can be formed; rather than
// reading g and the momentum a second time, this pass writes X~ = u unscaled
// (cast to the NS dtype) and the first Newton-Schulz step applies r = 1 /
// (||u|| + eps) to its products: A0 = r^2 (X~ X~^T), X1 = r (a X~ + B0 X~).
//
// A workgroup owns a 64x64 tile of the padded X extent (S x L), or a 32x128
// one when u is s x l and no X^T is kept (see tile_of).  It reads the
// matching tile of u's inputs row-wise, 8 consecutive elements per access
// (16-byte loads where the rows allow it, element by element at ragged
// edges), updates the momentum in place, writes X~ into whichever of X / X^T
// has u's layout (16-byte stores) and, through LDS, into the other (16-byte
// stores of 8 elements of one column), and stores its tile's sum of u^2 (a
// fixed-order reduction).  Zero outside the matrix.
// grid = (L/64, S/64, matrices).
// ---------------------------------------------------------------------------
template <typename XT>
struct TileStage {
  static constexpr int LDT = sizeof(XT) == 2 ? 66 : 65;  // LDS row stride (odd word stride)
};

// Tile (i0, j0) of X (origin in X coordinates) of matrix m: the same tile of
// u, its two destinations and their row strides.
template <typename XT>
struct TileDst {
  using E = typename Store<XT>::E;
  int ur0, uc0;
  E* D;        // u's own layout (X when u is s x l, X^T when l x s), or null
  int ldD;
  E* Tb;       // the transpose, through LDS, or null
  int ldT;
  int64_t plane;  // elements from one plane of X to the next
};

// Tile tt (row-major over the (S/64) x (L/64) grid) of matrix m.  A matrix
// with no transpose to write takes 32 x 128 tiles instead (the same count
// and the same 4096 elements each), whose 256-byte row pieces read and
// write more contiguously; `wide` says which.
template <typename XT>
__device__ __forceinline__ TileDst<XT> tile_dst(const MatDesc& md, const ChunkGeom& cg, int m, int i0, int j0,
                                                typename Store<XT>::E* X, typename Store<XT>::E* XTb);

template <typename XT>
__device__ __forceinline__ TileDst<XT> tile_of(const MatDesc& md, const ChunkGeom& cg, int m, int tt,
                                               typename Store<XT>::E* X, typename Store<XT>::E* XTb, bool& wide) {
  wide = md.transposed == 0 && XTb == nullptr;
  if (wide) {
    const int tx = cg.L / 128;
    return tile_dst<XT>(md, cg, m, (tt / tx) * 32, (tt % tx) * 128, X, XTb);
  }
  const int tx = cg.L / 64;
  return tile_dst<XT>(md, cg, m, (tt / tx) * 64, (tt % tx) * 64, X, XTb);
}

template <typename XT>
__device__ __forceinline__ TileDst<XT> tile_dst(const MatDesc& md, const ChunkGeom& cg, int m, int i0, int j0,
                                                typename Store<XT>::E* X, typename Store<XT>::E* XTb) {
  const bool tr = md.transposed != 0;
  const int64_t plane = static_cast<int64_t>(cg.S) * cg.L, matX = plane * Store<XT>::planes;
  auto* Xm = X + m * matX;
  auto* XTm = XTb ? XTb + m * matX : nullptr;
  TileDst<XT> t;
  t.plane = plane;
  t.ur0 = tr ? j0 : i0;
  t.uc0 = tr ? i0 : j0;
  t.D = tr ? XTm : Xm;
  t.ldD = tr ? cg.S : cg.L;
  t.Tb = tr ? Xm : XTm;
  t.ldT = tr ? cg.L : cg.S;
  return t;
}

// Phase 2 of a tile: rows of the transpose out of LDS, 16 bytes a thread.
template <typename XT>
__device__ __forceinline__ void write_transposed(const typename Store<XT>::L* tile, const TileDst<XT>& t) {
  using L = typename Store<XT>::L;
  constexpr int LDT = TileStage<L>::LDT;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int c = threadIdx.x + 256 * k;          // row c / 8 of the transpose, 8 (c % 8) ..
    const int trow = c >> 3, r8 = (c & 7) * 8;
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = to_f32<L>(tile[(r8 + q) * LDT + trow]);
    store8x<XT>(t.Tb, static_cast<int64_t>(t.uc0 + trow) * t.ldT + t.ur0 + r8, t.plane, v);
  }
}

// One tile of the prologue (UPDATE_MOM: advance the momentum and write it
// back; otherwise the momentum has been advanced already).  Returns this
// thread's sum of u^2 (fp64).  out = (u * s1) * s2.
template <typename GT, typename XT, bool MOM, bool UPDATE_MOM, bool WIDE>
__device__ __forceinline__ double prologue_tile(const MatDesc& md, const StepScalars& sc, const TileDst<XT>& t,
                                                float s1, float s2, typename Store<XT>::L* tile) {
  using L = typename Store<XT>::L;
  constexpr int LDT = TileStage<L>::LDT;
  constexpr int CPR = WIDE ? 16 : 8;              // 8-element chunks per tile row
  const GT* __restrict__ g = static_cast<const GT*>(md.g);
  const float beta = sc.beta, omb = sc.one_minus_beta;
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int c = threadIdx.x + 256 * k;          // chunk: row c / CPR, columns 8 (c % CPR) ..
    const int row = c / CPR, col = (c % CPR) * 8;
    const int ur = t.ur0 + row, uc = t.uc0 + col;
    float v[8];
    if (md.row8_ok && ur < md.rows && uc + 8 <= md.cols) {
      float gv[8], bv[8];
      load8(g, view_index(md, ur, uc), gv);
      if (MOM) {
        const int64_t ib = buf_index(md, ur, uc);
        load8(md.buf, ib, bv);
        if (UPDATE_MOM) {
#pragma unroll
          for (int q = 0; q < 8; ++q) bv[q] = fmaf(beta, bv[q], omb * gv[q]);
          store8(md.buf, ib, bv);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = sc.nesterov ? fmaf(beta, bv[q], omb * gv[q]) : bv[q];
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = gv[q];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        acc = fma(static_cast<double>(v[q]), static_cast<double>(v[q]), acc);
        v[q] = (v[q] * s1) * s2;
      }
    } else {  // padding stays exactly zero, whatever the scale
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        v[q] = 0.f;
        if (ur < md.rows && uc + q < md.cols) {
          const float gv = to_f32<GT>(g[view_index(md, ur, uc + q)]);
          if (MOM) {
            const int64_t ib = buf_index(md, ur, uc + q);
            float bn = md.buf[ib];
            if (UPDATE_MOM) {
              bn = fmaf(beta, bn, omb * gv);
              md.buf[ib] = bn;
            }
            v[q] = sc.nesterov ? fmaf(beta, bn, omb * gv) : bn;
          } else {
            v[q] = gv;
          }
          acc = fma(static_cast<double>(v[q]), static_cast<double>(v[q]), acc);
          v[q] = (v[q] * s1) * s2;
        }
      }
    }
    if (t.D) store8x<XT>(t.D, static_cast<int64_t>(ur) * t.ldD + uc, t.plane, v);
    if (!WIDE && t.Tb) {
#pragma unroll
      for (int q = 0; q < 8; ++q) tile[row * LDT + col + q] = from_f32<L>(v[q]);
    }
  }
  return acc;
}

template <typename GT, typename XT, bool MOM>
__global__ __launch_bounds__(256) void k_prologue(const MatDesc* __restrict__ desc, StepScalars sc, ChunkGeom cg,
                                                  typename Store<XT>::E* __restrict__ X,
                                                  typename Store<XT>::E* __restrict__ XTb,
                                                  double* __restrict__ partials) {
  __shared__ typename Store<XT>::L tile[64 * TileStage<typename Store<XT>::L>::LDT];
  __shared__ double red4[4];
  const int m = blockIdx.z;
  const MatDesc md = desc[m];
  bool wide;
  const TileDst<XT> t = tile_of<XT>(md, cg, m, blockIdx.y * gridDim.x + blockIdx.x, X, XTb, wide);
  const double acc = wide ? prologue_tile<GT, XT, MOM, true, true>(md, sc, t, 1.f, 1.f, tile)
                          : prologue_tile<GT, XT, MOM, true, false>(md, sc, t, 1.f, 1.f, tile);
  const double s = block_sum_256(acc, red4);  // (its barrier also publishes the LDS tile)
  if (threadIdx.x == 0)
    partials[static_cast<int64_t>(m) * (gridDim.x * gridDim.y) + blockIdx.y * gridDim.x + blockIdx.x] = s;
  if (!t.Tb) return;  // uniform over the block
  __syncthreads();
  write_transposed<XT>(tile, t);
}

// r = 1 / (sqrt(sum of partials) + eps), one workgroup per matrix, in fp64;
// xscale, the scale the first products apply, and rscale, what k_rescale
// multiplies u by (1: nothing to do).  While r is between 2^-40 and 2^40, X~
// X~^T stays well inside the fp32 range: xscale = r, rscale = 1.  Else X0 =
// r*u is written out: xscale = 1, rscale = r.
// Three planes (split) hold 24 bits of a value down to 2^-110 only, where
// plain fp32 holds them down to 2^-126.  When X0's norm is below 2^-60, X is
// therefore kept times 2^40 through all steps (k_rescale writes 2^40 r u; the
// Gram products and the last step take 2^-40, see gemm_tile_body): at that
// size the products add nothing to a*X, and X X^T stays finite while X grows.
// rscale = -2^40 r marks such a matrix.  1024 threads each sum every 1024th
// partial into four accumulators (independent loads in flight; an 8192 x
// 28672 matrix has 57344 partials), combined in a fixed order.
constexpr float kTinyScale = 0x1p-40f;
__global__ __launch_bounds__(1024) void k_finalize(const double* __restrict__ partials, int nparts, float eps,
                                                   int split, double* __restrict__ rscale,
                                                   float* __restrict__ xscale) {
  __shared__ double red16[16];
  const int m = blockIdx.x;
  const double* p = partials + static_cast<int64_t>(m) * nparts;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  int i = threadIdx.x;
  for (; i + 3 * 1024 < nparts; i += 4 * 1024) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] += p[i + q * 1024];
  }
  if (i < nparts) a[0] += p[i];
  if (i + 1024 < nparts) a[1] += p[i + 1024];
  if (i + 2048 < nparts) a[2] += p[i + 2048];
  double v = (a[0] + a[1]) + (a[2] + a[3]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red16[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) s += red16[w];
  if (threadIdx.x == 0) {
    const double n = sqrt(s), r = 1.0 / (n + static_cast<double>(eps));
    const bool folds = r >= 0x1p-40 && r <= 0x1p40;        // NaN fails both tests
    const bool tiny = split && n > 0.0 && n * r < 0x1p-60;
    rscale[m] = tiny ? -(r * 0x1p40) : folds ? 1.0 : r;
    xscale[m] = tiny ? kTinyScale : folds ? static_cast<float>(r) : 1.0f;
  }
}

// |rscale| u, written over X~, for the matrices that k_finalize says need it (a
// norm outside the range above, zero with eps = 0, NaN, or tiny in three
// planes); every other matrix's workgroups return at once.  The momentum is
// already advanced.
// grid = (workgroups per matrix, matrices); each loops over its tiles.
template <typename GT, typename XT, bool MOM>
__global__ __launch_bounds__(256) void k_rescale(const MatDesc* __restrict__ desc, const double* __restrict__ rscale,
                                                 StepScalars sc, ChunkGeom cg,
                                                 typename Store<XT>::E* __restrict__ X,
                                                 typename Store<XT>::E* __restrict__ XTb) {
  __shared__ typename Store<XT>::L tile[64 * TileStage<typename Store<XT>::L>::LDT];
  const int m = blockIdx.y;
  const double r = fabs(rscale[m]);
  if (r == 1.0) return;  // uniform over the block
  float s1, s2;
  split_scale(r, s1, s2);
  const MatDesc md = desc[m];
  const int ntiles = (cg.L / 64) * (cg.S / 64);
  for (int tt = blockIdx.x; tt < ntiles; tt += gridDim.x) {
    bool wide;
    const TileDst<XT> t = tile_of<XT>(md, cg, m, tt, X, XTb, wide);
    if (wide) (void)prologue_tile<GT, XT, MOM, false, true>(md, sc, t, s1, s2, tile);
    else (void)prologue_tile<GT, XT, MOM, false, false>(md, sc, t, s1, s2, tile);
    if (t.Tb) {  // uniform over the block
      __syncthreads();
      write_transposed<XT>(tile, t);
      __syncthreads();  // the next tile overwrites the LDS tile
    }
  }
}

// ---------------------------------------------------------------------------
// C = P Q^T on MFMA, P: M x K and Q: N x K row-major (K contiguous), all
// extents multiples of 128.  256 threads = 4 wavefronts in a 2 x 2 grid,
// each owning a 64 x 64 sub-tile = 2 x 2 blocks of the 32x32 MFMA.  K is
// staged through LDS 128 bytes per row at a time (64 bf16 or 32 fp32),
// double-buffered, with the next slab prefetched into registers while the
// current one is multiplied.
//
// bf16: v_mfma_f32_32x32x16_bf16, a lane supplies 8 consecutive k of its row.
// fp32: v_mfma_f32_32x32x2_f32, a lane holds 4 consecutive k and issues four
//       MFMAs (lanes 0-31 give k = j, lanes 32-63 give k = 4 + j).
// In both, a lane's operand for a 32-k (bf16) / 8-k (fp32) group is the 16
// bytes at byte offset 16*(lane/32) of the group, so the LDS geometry is the
// same for both element types.
//
// Output layout of a 32x32 block: lane l, register r holds
//   row 8*(r/4) + 4*(l/32) + (r%4), column l%32.
// ---------------------------------------------------------------------------
enum Epi : int { EPI_GRAM = 0, EPI_POLY = 1, EPI_UPDATE = 2, EPI_FINAL = 3,
                 // final-step variants of the 256-tile kernel: update W / write out, bf16 / fp32
                 EPI_FINAL_W_BF16 = 4, EPI_FINAL_W_F32 = 5, EPI_FINAL_O_BF16 = 6, EPI_FINAL_O_F32 = 7,
                 EPI_FINAL_W_BF16_ANY = 8 };  // 4: W rows of 16-byte accesses (w_rows16); 8: any

struct GemmArgs {
  const char* P;   int64_t p_mat;  int32_t ldp;   // bytes
  const char* Q;   int64_t q_mat;  int32_t ldq;
  int32_t k_slabs;                               // K * elem / 128
  int32_t tiles_m, tiles_n, syrk, tiles_per_mat;
  int32_t m_ext, n_ext;                          // rows of P and of Q (tile kernel: multiples of 128)
  const char* E;   int64_t e_mat;  int32_t lde;   // epilogue input (A or X), bytes
  char* C;         int64_t c_mat;  int32_t ldc;   // output, direct orientation
  char* CT;        int64_t ct_mat; int32_t ldct;  // output, transposed orientation
  float alpha, beta;
  const MatDesc* desc;
  int32_t final_kind, param_dtype, w_rows16;
  int32_t s, l;
  int32_t total_tiles;                           // tiles_per_mat * matrices
  // operand storage, tile kernel only: 0 row-major over K; 1 symmetric,
  // upper-triangle 256 x 256 tiles only; 2 (Q) stored K x N
  int32_t p_mode, q_mode;
  // SPLIT kernels: bytes from one plane of the operand or output to the next
  int64_t p_plane, q_plane, c_plane;
  // First Newton-Schulz step: X holds X~ = u unscaled, and the product is
  // scaled per matrix by xscale (the Gram product by its square); null after.
  const float* xscale;
  const double* rscale;                          // SPLIT kernels, every step: negative marks a tiny matrix (k_finalize)
};

constexpr int kRowBytes = 144;                   // 128 data + 16 pad per LDS row
constexpr int kOpBytes = kTile * kRowBytes;      // one operand slab
constexpr int kStageBytes = 2 * kOpBytes;
constexpr int kFStride = 137;                    // fp32 epilogue tile stride (odd)
static_assert(kTile * kFStride * 4 <= 2 * kStageBytes, "epilogue tile fits in LDS");

template <typename T> struct Mma;
template <> struct Mma<uint16_t> {
  __device__ __forceinline__ static void run(const u32x4_t& a, const u32x4_t& b, f32x16_t& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  }
};
template <> struct Mma<float> {
  __device__ __forceinline__ static void run(const u32x4_t& a, const u32x4_t& b, f32x16_t& c) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[j]), __uint_as_float(b[j]), c,
                                               0, 0, 0);
  }
};

template <typename T, int EPI>
__global__ __launch_bounds__(256, 2) void k_gemm_nt(GemmArgs ga) {
  __shared__ __attribute__((aligned(16))) char smem[2 * kStageBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // ---- tile assignment -----------------------------------------------------
  const int mat = blockIdx.x / ga.tiles_per_mat;
  int t = blockIdx.x - mat * ga.tiles_per_mat;
  int bm, bn;
  if (ga.syrk) {  // upper-triangle tiles bm <= bn, row by row
    bm = 0;
    while (t >= ga.tiles_m - bm) { t -= ga.tiles_m - bm; ++bm; }
    bn = bm + t;
  } else {
    bm = t / ga.tiles_n;
    bn = t - bm * ga.tiles_n;
  }
  const char* Pb = ga.P + mat * ga.p_mat + static_cast<int64_t>(bm) * kTile * ga.ldp;
  const char* Qb = ga.Q + mat * ga.q_mat + static_cast<int64_t>(bn) * kTile * ga.ldq;

  // ---- main loop -----------------------------------------------------------
  // Global -> register staging: row (tid/8 + 32v), 16-byte column (tid%8).
  const int lrow = tid >> 3, lcol = (tid & 7) * 16;
  u32x4_t rp[4], rq[4];
  auto gload = [&](int ks) {
    const int64_t koff = static_cast<int64_t>(ks) * 128 + lcol;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      rp[v] = *reinterpret_cast<const u32x4_t*>(Pb + static_cast<int64_t>(lrow + 32 * v) * ga.ldp + koff);
      rq[v] = *reinterpret_cast<const u32x4_t*>(Qb + static_cast<int64_t>(lrow + 32 * v) * ga.ldq + koff);
    }
  };
  auto sstore = [&](int stage) {
    char* sp = smem + stage * kStageBytes;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      *reinterpret_cast<u32x4_t*>(sp + (lrow + 32 * v) * kRowBytes + lcol) = rp[v];
      *reinterpret_cast<u32x4_t*>(sp + kOpBytes + (lrow + 32 * v) * kRowBytes + lcol) = rq[v];
    }
  };

  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int arow = wm * 64 + (lane & 31), brow = wn * 64 + (lane & 31);
  const int khalf = (lane >> 5) * 16;

  gload(0);
  sstore(0);
  __syncthreads();
  for (int ks = 0; ks < ga.k_slabs; ++ks) {
    const int stage = ks & 1;
    if (ks + 1 < ga.k_slabs) gload(ks + 1);
    const char* sp = smem + stage * kStageBytes;
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      u32x4_t a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        a[i] = *reinterpret_cast<const u32x4_t*>(sp + (arow + 32 * i) * kRowBytes + grp * 32 + khalf);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        b[j] = *reinterpret_cast<const u32x4_t*>(sp + kOpBytes + (brow + 32 * j) * kRowBytes + grp * 32 + khalf);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) Mma<T>::run(a[i], b[j], acc[i][j]);
    }
    if (ks + 1 < ga.k_slabs) sstore(stage ^ 1);
    __syncthreads();
  }

  // ---- epilogue: accumulators -> LDS fp32 tile ------------------------------
  // On the first step the products are of X~ = u: the Gram tile is scaled
  // by r^2, the update's product and its a*X term by r.
  float s_acc = 1.f, s_e = 1.f;
  if (ga.xscale && EPI != EPI_POLY) {
    const float r = ga.xscale[mat];
    s_acc = EPI == EPI_GRAM ? r * r : r;
    s_e = r;
  }
  float* ft = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = wm * 64 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int col = wn * 64 + j * 32 + (lane & 31);
        ft[row * kFStride + col] = acc[i][j][r] * s_acc;
      }
  __syncthreads();

  const bool diag = ga.syrk && bm == bn;
  const int gi0 = bm * kTile, gj0 = bn * kTile;  // tile origin (rows of P, rows of Q)
  const MatDesc* md = (EPI == EPI_FINAL) ? ga.desc + mat : nullptr;
  const bool tr = (EPI == EPI_FINAL) ? md->transposed != 0 : false;

  // Phase A: direct orientation, consecutive lanes on consecutive columns.
  for (int idx = tid; idx < kTile * kTile; idx += 256) {
    const int r = idx >> 7, c = idx & 127;
    const int gi = gi0 + r, gj = gj0 + c;
    float v;
    if (EPI == EPI_GRAM || EPI == EPI_POLY) {
      v = diag && r > c ? ft[c * kFStride + r] : ft[r * kFStride + c];
      if (EPI == EPI_POLY) {
        const float e = to_f32<T>(*reinterpret_cast<const T*>(ga.E + mat * ga.e_mat + static_cast<int64_t>(gi) * ga.lde + gj * static_cast<int>(sizeof(T))));
        v = fmaf(ga.alpha, e, ga.beta * v);
      }
      const T o = from_f32<T>(v);
      *reinterpret_cast<T*>(ga.C + mat * ga.c_mat + static_cast<int64_t>(gi) * ga.ldc + gj * static_cast<int>(sizeof(T))) = o;
      if (!diag) ft[r * kFStride + c] = to_f32<T>(o);  // for the mirror store
    } else {
      const float e = to_f32<T>(*reinterpret_cast<const T*>(ga.E + mat * ga.e_mat + static_cast<int64_t>(gi) * ga.lde + gj * static_cast<int>(sizeof(T))));
      v = fmaf(ga.alpha * s_e, e, ft[r * kFStride + c]);
      if (EPI == EPI_UPDATE) {
        const T o = from_f32<T>(v);
        *reinterpret_cast<T*>(ga.C + mat * ga.c_mat + static_cast<int64_t>(gi) * ga.ldc + gj * static_cast<int>(sizeof(T))) = o;
        ft[r * kFStride + c] = to_f32<T>(o);
      } else {  // EPI_FINAL
        if (!tr) {
          if (gi < ga.s && gj < ga.l) {
            const int64_t pidx = view_index(*md, gi, gj);
            if (ga.final_kind == 0) {
              const float w = load_as_f32(md->W, pidx, ga.param_dtype);
              store_from_f32(md->W, pidx, ga.param_dtype, fmaf(md->decay, w, -md->upd_scale * v));
            } else {
              store_from_f32(md->out, pidx, ga.param_dtype, v);
            }
          }
        } else {
          ft[r * kFStride + c] = v;
        }
      }
    }
  }
  const bool phase_b = (EPI == EPI_GRAM || EPI == EPI_POLY) ? !diag : (EPI == EPI_UPDATE ? true : tr);
  if (!phase_b) return;  // uniform across the workgroup
  __syncthreads();
  // Phase B: transposed orientation, consecutive lanes on consecutive rows r.
  for (int idx = tid; idx < kTile * kTile; idx += 256) {
    const int c = idx >> 7, r = idx & 127;
    const float v = ft[r * kFStride + c];
    const int gi = gi0 + r, gj = gj0 + c;
    if (EPI == EPI_FINAL) {
      if (gi < ga.s && gj < ga.l) {  // parameter is l x s: element (gj, gi)
        const int64_t pidx = view_index(*md, gj, gi);
        if (ga.final_kind == 0) {
          const float w = load_as_f32(md->W, pidx, ga.param_dtype);
          store_from_f32(md->W, pidx, ga.param_dtype, fmaf(md->decay, w, -md->upd_scale * v));
        } else {
          store_from_f32(md->out, pidx, ga.param_dtype, v);
        }
      }
    } else {
      *reinterpret_cast<T*>(ga.CT + mat * ga.ct_mat + static_cast<int64_t>(gj) * ga.ldct + gi * static_cast<int>(sizeof(T))) = from_f32<T>(v);
    }
  }
}

// ---------------------------------------------------------------------------
// The tile kernel: C = P Q^T on v_mfma_f32_32x32x16_bf16, extents multiples of
// 128, operands bf16 or (SPLIT) fp32 in three bfloat16 planes.  The tiles of a
// workgroup, one of three configurations (TileCfg; the choice is tiles_of):
//   256 x 256   512 threads = 8 wavefronts in a 2 x 4 grid, each owning a 128 x
//               64 sub-tile = 4 x 2 blocks of 32 x 32, so every operand fragment
//               read from LDS feeds two or four MFMAs; one workgroup per CU;
//   128 x 128   256 threads = 4 wavefronts of 64 x 64, two workgroups per CU, or
//               one with four LDS stages.
// An element sees the same operations in the same order on all of them.
//
// K is staged 64 elements (128 bytes per row) at a time with direct
// global-to-LDS loads (global_load_lds_dwordx4: lane i of a wavefront writes
// bytes [16 i, 16 i + 16) after the wave-uniform LDS base), double-buffered (or
// in four stages).  A wavefront instruction fills 8 consecutive tile rows; lane
// i fetches the 16-byte k-chunk (i % 8) ^ ((row >> 1) % 8) of its row, so LDS
// row r holds chunk c at position c ^ ((r >> 1) % 8).  A fragment read (32 rows,
// one chunk) then spreads over all 64 banks.
//
// The launch is persistent (one workgroup per CU slot).  Workgroup b runs on XCD
// b % 8; every round, the workgroups of one XCD take one compact block of the
// tile order (bands 8 tile-rows high), so they share operand panels in that
// XCD's L2.
//
// The epilogue starts from the accumulator registers: lane l holds rows 8*(r/4)
// + 4*(l/32) + (r%4) of column l%32 in register r of a block, so 4 consecutive
// registers are 4 consecutive rows of one column.  Outputs go to LDS as they are
// and leave as whole rows through transposing LDS reads; the last step's go
// through LDS in the parameter's own layout.
// ---------------------------------------------------------------------------
// Compile-time loop: f(std::integral_constant<int, 0>) ... f(<N-1>), so array
// indices inside f are constants whatever the unroller decides.
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}
template <int V>
using I_ = std::integral_constant<int, V>;

// Lane exchange inside each group of 4 lanes by DPP quad permutation: a VALU
// operand modifier, no LDS traffic.
constexpr int kQuadXor1 = 0xB1;  // quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;  // quad_perm [2,3,0,1]
template <int CTRL>
__device__ __forceinline__ uint32_t quad_swap(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), CTRL, 0xF, 0xF, true));
}

// Lanes 4p..4p+3 each hold x[0..3] = M[t][0..3] (t = lane % 4); afterwards
// lane t holds M[0..3][t].  Two butterfly stages over lane bits 0 and 1.
// Every lane of the quad must be active.
__device__ __forceinline__ void quad_transpose(float x[4]) {
  const int t = threadIdx.x & 3;
  float y[4], n[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) y[k] = __uint_as_float(quad_swap<kQuadXor1>(__float_as_uint(x[k])));
#pragma unroll
  for (int r = 0; r < 4; ++r) n[r] = ((r ^ t) & 1) ? y[r ^ 1] : x[r];
#pragma unroll
  for (int k = 0; k < 4; ++k) y[k] = __uint_as_float(quad_swap<kQuadXor2>(__float_as_uint(n[k])));
#pragma unroll
  for (int r = 0; r < 4; ++r) x[r] = ((r ^ t) & 2) ? y[r ^ 2] : n[r];
}

#ifndef MUON_NT
#define MUON_NT 1
#endif
// Epilogue outputs are written once and read by a later launch: streaming
// (non-temporal) stores keep them from displacing operand data in L2.
__device__ __forceinline__ void store_out(u32x4_t* p, u32x4_t v) {
  if (MUON_NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

__device__ __forceinline__ uint2 pack_bf16x4(const float v[4]) {
  return uint2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}
__device__ __forceinline__ void unpack_bf16x4(uint2 p, float v[4]) {
  v[0] = __uint_as_float(p.x << 16); v[1] = __uint_as_float(p.x & 0xffff0000u);
  v[2] = __uint_as_float(p.y << 16); v[3] = __uint_as_float(p.y & 0xffff0000u);
}

// The matrix that a last step writes, in registers: read through the
// descriptor's pointer, its fields would be loaded again after every store.
struct WView {
  void* dst;                 // W, or out
  int64_t ld, bstride;
  int32_t rb, rows;
  float decay, upd;
  bool vec8, vec4;           // 8 (4) consecutive elements at multiples of 8 (4) columns are aligned for vector accesses
};
template <int FK>
__device__ __forceinline__ WView w_view(const MatDesc* md) {
  WView v;
  v.dst = FK == 0 ? md->W : md->out;
  v.ld = md->ld; v.bstride = md->bstride;
  v.rb = md->rb; v.rows = md->rows;
  v.decay = md->decay; v.upd = md->upd_scale;
  v.vec4 = md->vec4_ok != 0;
  v.vec8 = v.vec4 && md->cols % 8 == 0 && md->ld % 8 == 0 && (md->rb >= md->rows || md->bstride % 8 == 0);
  return v;
}
__device__ __forceinline__ int64_t w_index(const WView& v, int32_t i, int32_t j) {
  if (v.rb >= v.rows) return i * v.ld + j;
  const int32_t q = i / v.rb;
  return q * v.bstride + static_cast<int64_t>(i - q * v.rb) * v.ld + j;
}

// W[idx ..] = decay*W - upd*o (FK = 0) or out[idx ..] = o (FK = 1) for 8
// consecutive elements, of which n are inside the matrix; `w` holds W's when
// vec8 and n = 8 (read ahead by read8).
template <typename PT>
struct Raw8 { u32x4_t q[sizeof(PT) / 2]; };
template <typename PT>
__device__ __forceinline__ Raw8<PT> read8(const WView& v, int64_t idx) {
  const u32x4_t* p = reinterpret_cast<const u32x4_t*>(static_cast<const PT*>(v.dst) + idx);
  Raw8<PT> r;
#pragma unroll
  for (int h = 0; h < static_cast<int>(sizeof(PT)) / 2; ++h) r.q[h] = p[h];
  return r;
}
template <int FK, typename PT>
__device__ __forceinline__ void apply8(const WView& v, int64_t idx, float o[8], int n, const Raw8<PT>& w) {
  PT* dst = static_cast<PT*>(v.dst) + idx;
  if (v.vec8 && n == 8) {
    if constexpr (FK == 0) {
      float wf[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if constexpr (sizeof(PT) == 2) {
          const uint32_t d = w.q[0][q / 2];
          wf[q] = __uint_as_float(q % 2 ? d & 0xffff0000u : d << 16);
        } else {
          wf[q] = __uint_as_float(w.q[q / 4][q % 4]);
        }
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = fmaf(v.decay, wf[q], -v.upd * o[q]);
    }
    store8(dst, 0, o);
    return;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int m = min(4, n - 4 * h);
    if (m <= 0) return;
    if (v.vec4 && m == 4) {
      float t[4];
      if constexpr (sizeof(PT) == 2) {
        uint2* p = reinterpret_cast<uint2*>(dst + 4 * h);
        if (FK == 0) unpack_bf16x4(*p, t);
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = FK == 0 ? fmaf(v.decay, t[q], -v.upd * o[4 * h + q]) : o[4 * h + q];
        *p = pack_bf16x4(t);
      } else {
        float4* p = reinterpret_cast<float4*>(dst + 4 * h);
        if (FK == 0) { const float4 r = *p; t[0] = r.x; t[1] = r.y; t[2] = r.z; t[3] = r.w; }
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = FK == 0 ? fmaf(v.decay, t[q], -v.upd * o[4 * h + q]) : o[4 * h + q];
        *p = make_float4(t[0], t[1], t[2], t[3]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q < m)
          dst[4 * h + q] = from_f32<PT>(FK == 0 ? fmaf(v.decay, to_f32<PT>(dst[4 * h + q]), -v.upd * o[4 * h + q])
                                                : o[4 * h + q]);
    }
  }
}

// Byte offset of an LDS object.
__device__ __forceinline__ uint32_t lds_offset(const char* p) {
  return static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) char*)(p)));
}

// Direct global -> LDS load (global_load_lds_dwordx4): lane i writes the 16
// bytes at base + off (base wave-uniform, off a 32-bit lane offset) to LDS
// bytes [lds + 16 i, lds + 16 i + 16); `lds` is wave-uniform.  Issued as
// inline assembly so that the compiler keeps no record of it: the kernel
// waits for these loads explicitly (vmcnt) before the barrier that publishes
// a slab, and the transposing LDS reads of the other stage must not wait for
// them.  M0 is set inside the statement.
__device__ __forceinline__ void load_lds16(const char* base, uint32_t off, uint32_t lds) {
  // (readfirstlane returns int: widen each half as unsigned, never by sign)
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32)));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b & 0xffffffffu)));
  const uint64_t bs = (static_cast<uint64_t>(hi) << 32) | static_cast<uint64_t>(lo);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(bs), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}

// 8 bytes per lane from LDS through the transposing read (ds_read_b64_tr_b16).
__device__ __forceinline__ uint2 tr_read_b64(const char* p) {
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  const v4i16 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16*)(const_cast<char*>(p)));
  return __builtin_bit_cast(uint2, v);
}

// Tile configuration of the direct-to-LDS MFMA kernel: output tile BM x BN,
// a WM x WN grid of wavefronts (each BM/WM x BN/WN), SLAB bytes of every
// tile row staged per LDS stage, NS stages, WPE wavefronts per SIMD.
template <int BM_, int BN_, int WM_, int WN_, int SLAB_, int NS_, int WPE_>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, SLAB = SLAB_, NS = NS_, WPE = WPE_;
  static constexpr int NW = WM * WN;
  static constexpr int LDS = NS * (BM + BN) * SLAB;
  static_assert(LDS <= 160 * 1024, "LDS budget");
};
// 256 x 256, 8 wavefronts of 128 x 64, one workgroup per CU.
#ifndef MUON_SQ_SLAB
#define MUON_SQ_SLAB 128
#define MUON_SQ_STAGES 2
#endif
using CfgSquare = TileCfg<256, 256, 2, 4, MUON_SQ_SLAB, MUON_SQ_STAGES, 2>;
// 128 x 128, 4 wavefronts of 64 x 64, two workgroups per CU: for launches
// whose 256 x 256 tiles would leave CUs without work (tiles_of).  Every
// element sees the same operations in the same order on both, so the choice
// never changes a result.
using CfgQuarter = TileCfg<128, 128, 2, 2, 128, 2, 2>;
// The same tile with four stages, one workgroup per CU: launches of at most
// one tile per CU, where each slab waits for its loads (deep_tiles).
using CfgDeep = TileCfg<128, 128, 2, 2, 128, 4, 1>;

// Tile `logical` of the launch: matrix-major; inside a matrix, banded
// (GS / GM tile-rows per band, column by column inside a band).
__device__ __forceinline__ void tile_from_logical(const GemmArgs& ga, int logical, int& mat, int& bm,
                                                  int& bn) {
  mat = logical / ga.tiles_per_mat;
  int t = logical - mat * ga.tiles_per_mat;
  if (ga.syrk) {
    // upper-triangle tiles (bm <= bn) in bands of GS tile-rows, column by
    // column inside a band, so concurrent tiles share row and column panels
#ifndef MUON_GS
#define MUON_GS 8
#endif
    constexpr int GS = MUON_GS;
    const int T = ga.tiles_m;
    int b0 = 0;
    for (;;) {
      const int rows = min(GS, T - b0);
      const int size = rows * (rows + 1) / 2 + (T - b0 - rows) * rows;
      if (t < size) break;
      t -= size;
      b0 += GS;
    }
    const int rows = min(GS, T - b0);
    int c = 0;
    while (t >= min(rows, c + 1)) { t -= min(rows, c + 1); ++c; }
    bn = b0 + c;
    bm = b0 + t;
  } else {
#ifndef MUON_GM
#define MUON_GM 8
#endif
    constexpr int GM = MUON_GM;
    const int band = t / (GM * ga.tiles_n);
    const int within = t - band * GM * ga.tiles_n;
    const int rows = min(GM, ga.tiles_m - band * GM);
    bm = band * GM + within % rows;
    bn = within / rows;
  }
}

// SPLIT: the operands and outputs are fp32 values in three bfloat16 planes
// (Split3), and each product of values is the six bfloat16 products whose
// weight is above 2^-24 (the method of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations",
// ARITH 2019).  A first pass over k adds the five small ones, per
// slab of 64 k in the order
//   (P, Q) = (h, l) (h, m) (m, m) (m, h) (l, h),
// in which one operand changes at a time (six operand slabs loaded for five
// slabs of MFMA work); a second pass adds (h, h).  The sums are thus rounded
// at their full size once per 16 k, where one pass over all six pairs would
// round them six times (and the fp32 instruction eight times).  The MFMA rate
// for bf16 is 16 times that for fp32, so the six cost 0.375 of the fp32
// instruction; what the pairs (m, l), (l, m), (l, l) would add is below the
// rounding of the fp32 accumulation.  Error of an orthogonalised matrix
// against 64 bits: see tests/test_split_error_gpu.py.
template <int EPI, class Cfg, bool SPLIT>
__device__ __forceinline__ void gemm_tile_body(const GemmArgs& ga, char* smem, int mat, int bm, int bn) {
  constexpr int BM = Cfg::BM, BN = Cfg::BN, WM = Cfg::WM, WN = Cfg::WN, NW = Cfg::NW;
  constexpr int SLAB = Cfg::SLAB, NS = Cfg::NS;
  constexpr int BI = BM / WM / 32;            // 32x32 blocks per wave, rows
  constexpr int BJ = BN / WN / 32;            // and columns
  constexpr int CPR = SLAB / 16;              // 16-byte chunks per staged row
  constexpr int SH = CPR == 8 ? 1 : 2;        // swizzle key: (row >> SH) & (CPR - 1)
  constexpr int RPI = 1024 / SLAB;            // rows one wave load instruction fills
  constexpr int PR = BM / NW, QR = BN / NW;   // operand rows each wave loads
  constexpr int NLP = PR / RPI, NLQ = QR / RPI;
  static_assert(NLP * RPI == PR && NLQ * RPI == QR, "load split");
  constexpr int GPS = SLAB / 32;              // 16-k MFMA groups per slab
  constexpr int OPQ = BM * SLAB;              // Q slab offset in a stage
  constexpr int STAGE = (BM + BN) * SLAB;
  constexpr bool FINAL = EPI >= EPI_FINAL_W_BF16;
  constexpr int FK = (EPI == EPI_FINAL_O_BF16 || EPI == EPI_FINAL_O_F32) ? 1 : 0;
  constexpr int PDT = (EPI == EPI_FINAL_W_F32 || EPI == EPI_FINAL_O_F32) ? DT_F32 : DT_BF16;
  static_assert(!FINAL || FK == 1 || EPI == EPI_FINAL_W_BF16 || EPI == EPI_FINAL_W_F32 || EPI == EPI_FINAL_W_BF16_ANY,
                "last-step variants");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  static_assert(SLAB == 128 && (NS == 2 || (NS == 4 && !SPLIT)) && GPS == 4 && (BM == 256 || BM == 128) && BN == BM && RPI == 8,
                "slab geometry: 64 k of BM rows, or 64 k-rows of BM columns");
  constexpr int TRB = BM * 2;                 // bytes of a transposed slab row, of a staged tile row
  constexpr int TRC = TRB / 16;               // its 16-byte chunks
  constexpr int TRI = 1024 / TRB;             // transposed rows one wave load instruction fills
  // The tile's rows of P and of Q inside the padded extents, which are
  // multiples of 128: 256, or 128 in the last tile of an odd extent.  Loads
  // of the rows (or columns) past them are sent 128 back, so they stay in
  // bounds; what they produce is never written.
  const int mv = min(BM, ga.m_ext - bm * BM), nv = min(BN, ga.n_ext - bn * BN);

  // ---- operand slabs ---------------------------------------------------------
  // A slab holds 64 consecutive k of the tile's 256 rows of P (and of Q), in
  // one of two geometries:
  //  - direct: 256 rows of 128 bytes (k contiguous), for an operand stored
  //    row-major over k;
  //  - transposed: 64 rows k of 512 bytes (the tile's rows contiguous), for
  //    an operand stored K x rows, read back with ds_read_b64_tr_b16.
  // Mode 0 reads every slab direct; mode 2 (Q only) every slab transposed:
  // the update products read X itself as their second operand.  Mode 1 is
  // the symmetric matrices A and B stored as their upper-triangle 256 x 256
  // tiles only: rows of tile-row b below the diagonal block (k < 256 b) are
  // columns of the stored tile (k-block, b), read transposed.
  const int nk = ga.k_slabs;
  const int p_tr_end = ga.p_mode == 1 ? bm * (BM / 64) : 0;   // slabs [0, p_tr_end) transposed
  const int q_tr_end = ga.q_mode == 2 ? nk : (ga.q_mode == 1 ? bn * (BN / 64) : 0);
  constexpr bool QTR = EPI == EPI_UPDATE || FINAL;           // update products: Q always transposed
  constexpr bool CAN_PT = EPI != EPI_GRAM, CAN_QT = EPI != EPI_GRAM, CAN_QD = !QTR;
  const char* const Pm = ga.P + mat * ga.p_mat;
  const char* const Qm = ga.Q + mat * ga.q_mat;
  const char* const Pd = Pm + static_cast<int64_t>(bm) * BM * ga.ldp;   // + ks * SLAB
  const char* const Qd = Qm + static_cast<int64_t>(bn) * BN * ga.ldq;
  const char* const Pt = Pm + bm * BM * 2;                               // + ks * 64 * ld
  const char* const Qt = Qm + bn * BN * 2;

  // Loads: a wave instruction fills 1 KB of the stage (8 direct rows or 2
  // transposed rows); lane l writes 16 bytes at 16 l and fetches the chunk
  // that belongs there.  Direct: LDS row r holds k-chunk c at position
  // c ^ ((r >> 1) % 8), which spreads the 32 rows of a fragment read over all
  // 64 banks.  Transposed: row k holds 16-byte chunk c at position
  // c ^ 4*(k % 4).  Per-lane offsets are 32-bit, added to a wave-uniform base.
  uint32_t pdo[NLP], pto[NLP], qdo[NLQ], qto[NLQ];
#pragma unroll
  for (int i = 0; i < NLP; ++i) {
    const int r = wave * PR + RPI * i + lane / CPR;
    pdo[i] = static_cast<uint32_t>((r < mv ? r : r - 128) * ga.ldp + ((lane % CPR) ^ ((r >> SH) & (CPR - 1))) * 16);
    const int t = wave * (TRI * NLP) + TRI * i + lane / TRC;
    const int c = (lane % TRC) ^ ((t & 3) << 2);
    pto[i] = static_cast<uint32_t>(t * ga.ldp + (8 * c < mv ? c : c - 16) * 16);
  }
#pragma unroll
  for (int i = 0; i < NLQ; ++i) {
    const int r = wave * QR + RPI * i + lane / CPR;
    qdo[i] = static_cast<uint32_t>((r < nv ? r : r - 128) * ga.ldq + ((lane % CPR) ^ ((r >> SH) & (CPR - 1))) * 16);
    const int t = wave * (TRI * NLQ) + TRI * i + lane / TRC;
    const int c = (lane % TRC) ^ ((t & 3) << 2);
    qto[i] = static_cast<uint32_t>(t * ga.ldq + (8 * c < nv ? c : c - 16) * 16);
  }
  const uint32_t lds0 = lds_offset(smem);
  // The loads of slab ks, one operand at a time: P's NLP instructions or Q's
  // NLQ, into the slab's stage.
  auto issue_op = [&](auto qc, int ks, int at, int64_t plane = 0) __attribute__((always_inline)) {
    const uint32_t base = lds0 + at;   // the stage's byte offset
    if constexpr (!decltype(qc)::value) {
      if (CAN_PT && ks < p_tr_end) {
        const char* b = Pt + plane + static_cast<int64_t>(ks) * 64 * ga.ldp;
#pragma unroll
        for (int i = 0; i < NLP; ++i) load_lds16(b, pto[i], base + (wave * PR + RPI * i) * SLAB);
      } else {
        const char* b = Pd + plane + ks * SLAB;
#pragma unroll
        for (int i = 0; i < NLP; ++i) load_lds16(b, pdo[i], base + (wave * PR + RPI * i) * SLAB);
      }
    } else {
      if (CAN_QT && (!CAN_QD || ks < q_tr_end)) {
        const char* b = Qt + plane + static_cast<int64_t>(ks) * 64 * ga.ldq;
#pragma unroll
        for (int i = 0; i < NLQ; ++i) load_lds16(b, qto[i], base + OPQ + (wave * QR + RPI * i) * SLAB);
      } else {
        const char* b = Qd + plane + ks * SLAB;
#pragma unroll
        for (int i = 0; i < NLQ; ++i) load_lds16(b, qdo[i], base + OPQ + (wave * QR + RPI * i) * SLAB);
      }
    }
  };
  auto issue = [&](int ks) __attribute__((always_inline)) {
    issue_op(std::false_type{}, ks, (ks & (NS - 1)) * STAGE);
    issue_op(std::true_type{}, ks, (ks & (NS - 1)) * STAGE);
  };

  f32x16_t acc[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Fragments.  Direct: row (.. + lane % 32), k-chunk 2*grp + lane / 32 at its
  // swizzled position, one ds_read_b128.  Transposed: ds_read_b64_tr_b16
  // hands lane t of each 16-lane group G, as its r-th element, element t % 4
  // of the 8 bytes addressed by lane 4r + t / 4 of the group.  Lane L of
  // group G therefore addresses row 16*grp + 8*(G/2) + 4*h + L/4, columns
  // c0 + 16*(G%2) + 4*(L%4) .. +3, and two reads (h = 0, 1) give the 8
  // consecutive k of column c0 + lane % 32 that the MFMA takes.  The 4 rows k
  // of one read differ in k % 4, so the swizzle spreads them over all banks.
  const int frow = lane & 31, fsel = lane >> 5, fsw = (frow >> SH) & (CPR - 1);
  const int a_off = (wm * (BM / WM) + frow) * SLAB;
  const int b_off = OPQ + (wn * (BN / WN) + frow) * SLAB;
  auto tr_off = [&](int c0) {
    const int G = lane >> 4, L = lane & 15;
    const int row = 8 * (G >> 1) + (L >> 2);
    const int cb = 2 * c0 + 32 * (G & 1) + 8 * (L & 3);
    return row * TRB + (cb ^ ((L >> 2) << 6));
  };
  int tpo[BI], tqo[BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i) tpo[i] = tr_off(wm * (BM / WM) + i * 32);
#pragma unroll
  for (int j = 0; j < BJ; ++j) tqo[j] = OPQ + tr_off(wn * (BN / WN) + j * 32);

  // ---- the a*X (or A) term, taken from the operand slabs ----------------------
  // The tile that the epilogue combines with the product passes through LDS
  // as part of an operand, so it is added to the accumulators there instead
  // of being read from memory again:
  //  - update products: rows bm*256 + [0, 256) of X are the Q slabs
  //    4 bm .. 4 bm + 3 (transposed geometry); the wave's 128 rows are slabs
  //    4 bm + 2 wm + h, h = 0, 1, holding its row blocks 2h and 2h + 1;
  //  - polynomial: A[bm, bn] is the P slabs 4 bn .. 4 bn + 3 (direct, as
  //    bn >= bm); the wave's 64 columns are slab 4 bn + wn.
  // One transposing read gives a lane the 4 consecutive rows of one column
  // that 4 accumulator registers hold: lane 4e + q of 16-lane group G
  // addresses row 4(G/2) + e, columns 16(G%2) + 4q .. +3 of the block's
  // register group, and lane t receives column 16(G%2) + t, rows 0..3.
  // The polynomial adds alpha = b/c times A and scales by beta = c at the
  // end (with c = 0 there is no product: k_scale_upper).
  // SPLIT adds the term after the last slab instead, plane by plane from
  // slabs loaded again: an fp32 sum that starts from its largest term rounds
  // every later product to that term's last bit (measured: up to 8 times the
  // error where a*X dominates), and b/c would be a rounded coefficient.
  constexpr bool EUPD = QTR;
  static_assert(BN / WN == 64, "A term: a wave's columns of A are one P slab");
  constexpr int ERS = (BM / WM) / 64;           // Q slabs holding a wave's rows of X
  static_assert(ERS * 2 == BI, "X term: whole slabs per wave");
  constexpr bool epoly = EPI == EPI_POLY;
  int e_ks0 = -1, e_ks1 = -1;
  if (EUPD) {
    e_ks0 = bm * (BM / 64) + ERS * wm;
    if (ERS > 1) e_ks1 = e_ks0 + 1;
  } else if (epoly) {
    e_ks0 = bn * (BN / 64) + wn;
  }
  int eo[BJ][2];
  {
    const int G = lane >> 4, L = lane & 15;
#pragma unroll
    for (int j = 0; j < BJ; ++j)
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) {
        if (EUPD)  // Q slab: row k holds chunk c at c ^ 4(k % 4)
          eo[j][gp] = OPQ + (4 * (G >> 1) + (L >> 2)) * TRB +
                      ((2 * (wn * (BN / WN) + 32 * j) + 32 * (G & 1) + 8 * (L & 3)) ^ ((L >> 2) << 6));
        else       // P slab: row r holds chunk c at c ^ ((r >> 1) % 8)
          eo[j][gp] = (wm * (BM / WM) + 4 * (G >> 1) + (L >> 2)) * SLAB +
                      (((4 * j + 2 * (G & 1) + ((L >> 1) & 1)) ^ (4 * gp + 2 * (G >> 1) + (L >> 3))) << 4) +
                      8 * (L & 1);
      }
  }
  // The factor the accumulators leave with: c for a polynomial; on the first step, whose X holds u unscaled,
  // r^2 for the Gram product and r for the update products.  A tiny matrix's X is 2^40 times the iterate in
  // every step but the last's output.
  float osc = 1.f;
  if (EPI == EPI_POLY) {
    osc = ga.beta;
  } else {
    float r = ga.xscale ? ga.xscale[mat] : 1.f;
    if constexpr (SPLIT)
      if (ga.rscale[mat] < 0.0) r = EPI == EPI_UPDATE ? 1.f : kTinyScale;
    osc = EPI == EPI_GRAM ? r * r : r;
  }
  const float alpha = SPLIT && EUPD ? ga.alpha * osc : ga.alpha;
  // Row blocks [i0, i0 + ni) of the wave's accumulators take the term from the
  // slab at sp.
  auto add_e = [&](const char* sp, auto i0c, auto nic) __attribute__((always_inline)) {
    constexpr int i0 = decltype(i0c)::value, ni = decltype(nic)::value;
    static_for<ni>([&](auto II) {
      constexpr int i = i0 + decltype(II)::value;
      uint2 ev[BJ][4];
      static_for<BJ>([&](auto J) {
        static_for<4>([&](auto Gc) {
          constexpr int j = decltype(J)::value, g = decltype(Gc)::value;
          ev[j][g] = EUPD ? tr_read_b64(sp + eo[j][0] + (32 * (i & 1) + 8 * g) * TRB)
                           : tr_read_b64(sp + eo[j][g & 1] + (32 * i + 8 * g) * SLAB);
        });
      });
      static_for<BJ>([&](auto J) {
        static_for<4>([&](auto Gc) {
          constexpr int j = decltype(J)::value, g = decltype(Gc)::value;
          float e[4];
          unpack_bf16x4(ev[j][g], e);
          f32x16_t& c = acc[i][j];
          c[4 * g + 0] = fmaf(alpha, e[0], c[4 * g + 0]);
          c[4 * g + 1] = fmaf(alpha, e[1], c[4 * g + 1]);
          c[4 * g + 2] = fmaf(alpha, e[2], c[4 * g + 2]);
          c[4 * g + 3] = fmaf(alpha, e[3], c[4 * g + 3]);
        });
      });
    });
  };

  // Software pipeline: the fragments of group g+1 are read into the other
  // register set while group g's MFMAs issue, one LDS read between
  // consecutive MFMAs; the slab barrier sits before the last group's MFMAs.
  u32x4_t fa[2][BI], fb[2][BJ];
  auto rd = [&](auto ptc, auto qtc, const char* sP, const char* sQ, auto grpc, auto setc) __attribute__((always_inline)) {
    constexpr bool PT = decltype(ptc)::value, QT = decltype(qtc)::value;
    constexpr int grp = decltype(grpc)::value, set = decltype(setc)::value;
    const int pos = ((2 * grp + fsel) ^ fsw) * 16;
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      if (PT) {
        const char* q = sP + tpo[i] + grp * 16 * TRB;
        const uint2 lo = tr_read_b64(q), hi = tr_read_b64(q + 4 * TRB);
        fa[set][i] = u32x4_t{lo.x, lo.y, hi.x, hi.y};
      } else {
        fa[set][i] = *reinterpret_cast<const u32x4_t*>(sP + a_off + i * 32 * SLAB + pos);
      }
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      if (QT) {
        const char* q = sQ + tqo[j] + grp * 16 * TRB;
        const uint2 lo = tr_read_b64(q), hi = tr_read_b64(q + 4 * TRB);
        fb[set][j] = u32x4_t{lo.x, lo.y, hi.x, hi.y};
      } else {
        fb[set][j] = *reinterpret_cast<const u32x4_t*>(sQ + b_off + j * 32 * SLAB + pos);
      }
    }
  };
  auto mm = [&](auto setc) __attribute__((always_inline)) {
    constexpr int set = decltype(setc)::value;
    static_for<BI>([&](auto I) {
      static_for<BJ>([&](auto J) { Mma<uint16_t>::run(fa[set][I.value], fb[set][J.value], acc[I.value][J.value]); });
    });
  };
  auto interleave = [&](auto ptc, auto qtc) __attribute__((always_inline)) {
    constexpr int NRD = (decltype(ptc)::value ? 2 : 1) * BI + (decltype(qtc)::value ? 2 : 1) * BJ;
    constexpr int NPAIR = NRD < BI * BJ ? NRD : BI * BJ;
#pragma unroll
    for (int i = 0; i < NPAIR; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
    }
    if constexpr (BI * BJ > NPAIR) __builtin_amdgcn_sched_group_barrier(0x008, BI * BJ - NPAIR, 0);
    if constexpr (NRD > NPAIR) __builtin_amdgcn_sched_group_barrier(0x100, NRD - NPAIR, 0);
  };
  // One slab in mode (PT, QT); group 0's fragments are already in set 0.
  // With NEXT, the fragments of the next slab's group 0 (same mode) are read
  // while the last group's MFMAs issue; without, the last group runs alone
  // (the slab before a change of mode, and the last one).
  // When a slab's loads are issued, one operand at a time, so that the
  // workgroups of an XCD do not ask for a whole slab at once:
  //  - Gram product (EARLY): Q's right after the barrier that frees the
  //    stage, P's at the top of the next slab (the slab of lead that was
  //    measured faster for its long K);
  //  - the other products: Q's at the top of the slab before, P's after
  //    that slab's first MFMA group (3/4 and 1/2 of a slab ahead).
  // Splitting the burst by operand measured 2-3% faster on the step than
  // issuing a slab at once; splitting each operand in halves, or P later,
  // measured slower.
  //  - with four stages (DEEP), whole slabs three ahead: a launch of one
  //    128 x 128 tile per CU waits on latency, not on contention.
  constexpr bool DEEP = NS > 2;
  constexpr bool EARLY = EPI == EPI_GRAM && !SPLIT && !DEEP;
  // The a*X (or A) term of slab ks, if it holds some of this wave's.
  auto take_e = [&](const char* sp, int ks) __attribute__((always_inline)) {
    if (ks == e_ks0 || ks == e_ks1) {  // wave-uniform; at most twice a tile
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!EUPD || ERS == 1) {
        add_e(sp, I_<0>{}, I_<BI>{});
      } else {
        // (the comments keep the compiler from merging the two calls into one
        // with a run-time row block, which would put the accumulators in memory)
        if (ks == e_ks0) {
          add_e(sp, I_<0>{}, I_<2>{});
          asm volatile("; row blocks 0, 1");
        } else {
          add_e(sp, I_<2>{}, I_<2>{});
          asm volatile("; row blocks 2, 3");
        }
      }
    }
  };
  auto slab = [&](auto ptc, auto qtc, auto nextc, auto ec, int ks) __attribute__((always_inline)) {
    const char* sp = smem + (ks & (NS - 1)) * STAGE;
    if constexpr (DEEP) {
      if (ks + 3 < nk) issue(ks + 3);                       // over slab ks - 1, which every wave has left
    } else if (ks + 1 < nk) {
      if (!EARLY) issue_op(std::true_type{}, ks + 1, ((ks + 1) & 1) * STAGE);
      else if (ks >= 1) issue_op(std::false_type{}, ks + 1, ((ks + 1) & 1) * STAGE);  // slab 1 went out whole with slab 0
    }
    if constexpr (decltype(ec)::value) take_e(sp, ks);
    __builtin_amdgcn_sched_barrier(0);
    rd(ptc, qtc, sp, sp, I_<1>{}, I_<1>{}); mm(I_<0>{}); interleave(ptc, qtc);
    __builtin_amdgcn_sched_barrier(0);
    if (!EARLY && !DEEP && ks + 1 < nk) issue_op(std::false_type{}, ks + 1, ((ks + 1) & 1) * STAGE);
    __builtin_amdgcn_sched_barrier(0);
    rd(ptc, qtc, sp, sp, I_<2>{}, I_<0>{}); mm(I_<1>{}); interleave(ptc, qtc);
    __builtin_amdgcn_sched_barrier(0);
    rd(ptc, qtc, sp, sp, I_<3>{}, I_<1>{}); mm(I_<0>{}); interleave(ptc, qtc);
    __builtin_amdgcn_sched_barrier(0);
    // slab ks + 1 has landed (DEEP: the two after it may not have)
    if (DEEP && ks + 3 < nk) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * (NLP + NLQ)) : "memory");
    else if (DEEP && ks + 2 < nk) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NLP + NLQ) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // every wave is done with slab ks: its stage can take slab ks + 2
    if (EARLY && ks + 2 < nk) issue_op(std::true_type{}, ks + 2, (ks & 1) * STAGE);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(nextc)::value) {
      const char* sn = smem + ((ks + 1) & (NS - 1)) * STAGE;
      rd(ptc, qtc, sn, sn, I_<0>{}, I_<0>{});
      mm(I_<1>{}); interleave(ptc, qtc);
    } else {
      mm(I_<1>{});
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // SPLIT: one slab of one plane pair, (pass, slab, phase) = (pass, sks, ph),
  // P in buffer pb and Q in qb.  An operand that changes for the next step is
  // loaded during this one into its other buffer, whose last reader ended at
  // least a step ago.  The step is a run-time value: unrolled, the phases'
  // addresses are hoisted out of the loop and spill.
  int pass = 0, sks = 0, ph = 0, pb = 0, qb = 0;
  auto step = [&](auto ptc, auto qtc, auto nextc) __attribute__((always_inline)) {
    int npass = pass, nks = sks, nph = ph + 1;
    if (pass == 1 || ph == 4) {
      nph = 0;
      nks = sks + 1;
      if (pass == 0 && nks == nk) { npass = 1; nks = 0; }
    }
    const bool more = nks < nk, both = nph == 0, newq = both || (nph & 1) != 0, newp = both || (nph & 1) == 0;
    const int npb = pb ^ (newp ? 1 : 0), nqb = qb ^ (newq ? 1 : 0);
    const int pplane = nph >> 1, qplane = npass == 1 ? 0 : (nph == 0 ? 2 : (nph == 1 ? 1 : 0));
    const char* sP = smem + pb * STAGE;
    const char* sQ = smem + qb * STAGE;
    if (more) {
      if (newq) issue_op(std::true_type{}, nks, nqb * STAGE, qplane * ga.q_plane);
      else issue_op(std::false_type{}, nks, npb * STAGE, pplane * ga.p_plane);
    }
    __builtin_amdgcn_sched_barrier(0);
    rd(ptc, qtc, sP, sQ, I_<1>{}, I_<1>{}); mm(I_<0>{}); interleave(ptc, qtc);
    __builtin_amdgcn_sched_barrier(0);
    if (more && both) issue_op(std::false_type{}, nks, npb * STAGE, 0);
    __builtin_amdgcn_sched_barrier(0);
    rd(ptc, qtc, sP, sQ, I_<2>{}, I_<0>{}); mm(I_<1>{}); interleave(ptc, qtc);
    __builtin_amdgcn_sched_barrier(0);
    rd(ptc, qtc, sP, sQ, I_<3>{}, I_<1>{}); mm(I_<0>{}); interleave(ptc, qtc);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the next step's operands have landed
    __syncthreads();
    pass = npass; sks = nks; ph = nph; pb = npb; qb = nqb;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(nextc)::value) {
      rd(ptc, qtc, smem + pb * STAGE, smem + qb * STAGE, I_<0>{}, I_<0>{});
      mm(I_<1>{}); interleave(ptc, qtc);
    } else {
      mm(I_<1>{});
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Slabs [a, b) in one mode.  Each run starts from a published slab and
  // ends with the next one published, so runs chain without carrying
  // fragments across a change of mode (which happens at most twice a tile).
  // With ec, the run may hold the slabs that carry the a*X (or A) term.
  auto run = [&](auto ptc, auto qtc, auto ec, int a, int b) __attribute__((always_inline)) {
    if (a >= b) return;
    if constexpr (SPLIT) {
      rd(ptc, qtc, smem + pb * STAGE, smem + qb * STAGE, I_<0>{}, I_<0>{});
#pragma unroll 1
      for (int t = (pass == 0 ? 5 : 1) * (b - a) - 1; t > 0; --t) step(ptc, qtc, std::true_type{});
      step(ptc, qtc, std::false_type{});
    } else {
      const char* sa = smem + (a & (NS - 1)) * STAGE;
      rd(ptc, qtc, sa, sa, I_<0>{}, I_<0>{});
      for (int ks = a; ks < b - 1; ++ks) slab(ptc, qtc, std::true_type{}, ec, ks);
      slab(ptc, qtc, std::false_type{}, ec, b - 1);
    }
  };
  using T_ = std::true_type;
  using F_ = std::false_type;
  if constexpr (SPLIT) {
    issue_op(F_{}, 0, 0, 0);
    issue_op(T_{}, 0, 0, 2 * ga.q_plane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else if (issue(0); DEEP) {
    if (nk > 1) issue(1);
    if (nk > 2) issue(2);
    if (nk > 2) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * (NLP + NLQ)) : "memory");
    else if (nk > 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NLP + NLQ) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else if (EARLY && nk > 1) {
    issue(1);
    // slab 0 has landed, slab 1 (NLP + NLQ loads) may not
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NLP + NLQ) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  // Mode runs: P transposed for [0, p_tr_end), Q for [0, q_tr_end).  The
  // launches keep p_tr_end <= q_tr_end (GRAM none, POLY bm <= bn, update
  // products Q transposed throughout).
  // The term's slabs lie in the last run (k >= 256 bm for the update
  // products, k >= 256 bn for the polynomial).
#pragma unroll 1
  for (int sweep = 0; sweep < (SPLIT ? 2 : 1); ++sweep) {
  if constexpr (EPI == EPI_GRAM) {
    run(F_{}, F_{}, F_{}, 0, nk);
  } else if constexpr (QTR) {
    run(T_{}, T_{}, F_{}, 0, p_tr_end);
    run(F_{}, T_{}, T_{}, p_tr_end, nk);
  } else {
    run(T_{}, T_{}, F_{}, 0, p_tr_end);
    run(F_{}, T_{}, F_{}, p_tr_end, q_tr_end);
    run(F_{}, F_{}, T_{}, max(p_tr_end, q_tr_end), nk);
  }
  }

  if constexpr (SPLIT && EPI != EPI_GRAM) {
    static_for<BI>([&](auto I) {
      static_for<BJ>([&](auto J) {
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[I.value][J.value][q] *= osc;
      });
    });
    constexpr int NE = BM / 64, OPSZ = BM * SLAB;   // slabs that hold the term, and their size
    const int k0 = (EUPD ? bm : bn) * NE;
    const int64_t plane = EUPD ? ga.q_plane : ga.p_plane;
#pragma unroll 1
    for (int pl = 2; pl >= 0; --pl) {               // smallest first
#pragma unroll
      for (int j = 0; j < NE; ++j)
        if (k0 + j < nk) issue_op(std::bool_constant<EUPD>{}, k0 + j, EUPD ? j * OPSZ - OPQ : j * OPSZ, pl * plane);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if constexpr (EUPD) {
        take_e(smem + ERS * wm * OPSZ - OPQ, e_ks0);
        if (ERS > 1) take_e(smem + (ERS * wm + 1) * OPSZ - OPQ, e_ks1);
      } else {
        take_e(smem + wn * OPSZ, e_ks0);
      }
      __syncthreads();
    }
  }

  // ---- epilogue from registers ----------------------------------------------
  // Lane l holds, per 32x32 block and register group g, rows row0..row0+3 of
  // one column `col` (the natural layout: also 4 consecutive elements of row
  // `col` of the transposed tile).  A 4-lane transpose gives the direct
  // layout: lane t = l % 4 holds row row0+t, columns c0..c0+3, and 8 lanes
  // cover 64 contiguous bytes of a row.
  //  - The a*X (or A) term is already in the accumulators (added in the main
  //    loop).
  //  - Outputs are rounded to bfloat16 once and leave through LDS as whole
  //    512-byte rows.  The symmetric products write upper-triangle tiles only,
  //    and X' needs no transposed copy: the next products read tiles below the
  //    diagonal, and X, through transposing LDS reads.
  //  - The last step's parameter update runs in the parameter's layout:
  //    direct when it is s x l, natural when it is l x s.
  const bool diag = ga.syrk && bm == bn;
  // 256 x 256 tiles read the diagonal 256 x 256 blocks of A and B
  // whole: of such a block, a launch on 128 x 128 tiles also writes the quarter below
  // the diagonal, the mirror of its (even, odd) tile.
  const bool pair_mirror = BM == 128 && ga.syrk && (bm & 1) == 0 && bn == bm + 1;
  const MatDesc* md = FINAL ? ga.desc + mat : nullptr;
  const bool tr = FINAL ? md->transposed != 0 : false;
  using PT = typename std::conditional<PDT == DT_BF16, uint16_t, float>::type;
  WView wv{};
  if constexpr (FINAL) wv = w_view<FK>(md);
  const int q4 = lane & 3;
  const int row_base = bm * BM + wm * (BM / WM) + 4 * fsel;
  const int col_base = bn * BN + wn * (BN / WN) + frow;
  char* C = ga.C + mat * ga.c_mat;
  constexpr int TST = BM * 2 + 8;             // staged column, bytes
  // Natural staging of the output tile: each lane's 4 consecutive rows of one
  // column go to LDS as they are, 8 bytes at column-major position (col, row)
  // with a column pitch of TST bytes, and the copy-out reads whole rows back
  // through transposing LDS reads.  No register transposes; diagonal tiles of the symmetric products take
  // their lower triangle from the mirrored column at copy-out.
  constexpr bool stage_n = !FINAL;
  // Diagonal tiles of the symmetric products are written exactly symmetric:
  // the value computed for (row, col) with row <= col also goes to (col, row),
  // at copy-out.  The output tile goes through LDS because whole 512-byte
  // rows measured faster than 64-byte row pieces from the registers.
  // The last step with a bfloat16 parameter whose rows take 16-byte accesses:
  // W goes through LDS the same way, loaded and written back as whole
  // 512-byte rows of its own layout.  Its staged row r holds chunk c at
  // c ^ key(r), key(r) = 4*(r % 4) + (r / 4) % 4, which spreads both the
  // direct accesses (8 rows x 64 bytes) and the natural ones (32 rows x 16
  // bytes) over all banks.  At the matrix's edge the block has wrv rows and
  // wcv columns (a multiple of 8): loads past them repeat the last row or
  // chunk, and only the block is written back.
  constexpr bool stage_w = EPI == EPI_FINAL_W_BF16;
  const int wr0 = tr ? bn * BN : bm * BM, wc0 = tr ? bm * BM : bn * BN;  // W block origin
  int wrv = 0, wcv = 0;
  if constexpr (stage_w) {
    wrv = min(BM, md->rows - wr0);
    wcv = min(BM, md->cols - wc0);
  }
  auto wpos = [](int r, int b) {
    const int key = ((r & 3) << 2) | ((r >> 2) & 3);
    return r * TRB + (((b >> 4) ^ key) << 4) + (b & 15);
  };
  // (every wave finished its operand-slab reads before the last slab's
  // barrier, so the staging area, which overlaps the slabs, is free)
  if constexpr (stage_w) {
    constexpr int KW = BM * BN * 2 / 1024 / NW;   // load instructions per wave
    static_assert(KW * NW * 1024 == BM * BN * 2, "W tile: whole instructions per wave");
    const char* wb = static_cast<const char*>(wv.dst) + (static_cast<int64_t>(wr0) * wv.ld + wc0) * 2;
    const uint32_t ldw = static_cast<uint32_t>(wv.ld) * 2;
    const uint32_t lds0 = lds_offset(smem);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int row = TRI * (wave * KW + k) + lane / TRC;
      const int c = (lane % TRC) ^ (((row & 3) << 2) | ((row >> 2) & 3));
      load_lds16(wb, static_cast<uint32_t>(min(row, wrv - 1)) * ldw + static_cast<uint32_t>(min(c * 16, wcv * 2 - 16)),
                 lds0 + (wave * KW + k) * 1024);
    }
  }
  // (The loads and the per-block work sit in one lambda: inlined that way the
  // compiler keeps every value in registers; written at function scope it
  // spilled.)
  auto blocks = [&](float scale) {
    if constexpr (stage_w) {  // the W block has landed in LDS
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    auto w_update = [&](char* p, const float o[4]) {  // 4 staged W values, in place
      float w[4], r[4];
      unpack_bf16x4(*reinterpret_cast<const uint2*>(p), w);
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = fmaf(wv.decay, w[q], -wv.upd * o[q]);
      *reinterpret_cast<uint2*>(p) = pack_bf16x4(r);
    };
    static_for<BI>([&](auto I) {
      static_for<BJ>([&](auto J) {
        static_for<4>([&](auto G) {
          constexpr int i = decltype(I)::value, j = decltype(J)::value, g = decltype(G)::value;
          const int row0 = row_base + i * 32 + 8 * g;  // rows row0 .. row0 + 3
          const int col = col_base + j * 32;
          const int c0 = col - q4;                     // direct layout: columns c0 .. c0 + 3
          float v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = acc[i][j][4 * g + q] * scale;
          if (!FINAL || tr) {  // natural layout
            if (stage_n) {
              const uint2 h = pack_bf16x4(v);
              *reinterpret_cast<uint2*>(smem + (col - bn * BN) * TST + (row0 - bm * BM) * 2) = h;
              if constexpr (SPLIT) {  // what the next plane holds
                float e[4];
                unpack_bf16x4(h, e);
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[i][j][4 * g + q] = v[q] - e[q];
              }
            } else {                   // parameter is l x s: elements (col, row0 .. row0 + 3)
              w_update(smem + wpos(col - wr0, (row0 - wc0) * 2), v);
            }
          } else {             // parameter is s x l: elements (row0 + q4, c0 .. c0 + 3)
            quad_transpose(v);
            w_update(smem + wpos(row0 + q4 - wr0, (c0 - wc0) * 2), v);
          }
        });
      });
    });
  };
  if constexpr (stage_w) {
    blocks(SPLIT ? 1.f : osc);
    __syncthreads();
    // updated W rows -> W, 16 bytes a thread
    for (int idx = threadIdx.x; idx < BM * TRC; idx += 64 * NW) {
      const int r = idx / TRC, ch = idx % TRC;
      if (r >= wrv || ch * 8 >= wcv) continue;
      *reinterpret_cast<u32x4_t*>(static_cast<char*>(wv.dst) + (static_cast<int64_t>(wr0 + r) * wv.ld + wc0) * 2 +
                                  ch * 16) = *reinterpret_cast<const u32x4_t*>(smem + wpos(r, ch * 16));
    }
    __syncthreads();  // the next tile's loads overwrite the staging area
  }
  if constexpr (FINAL && !stage_w) {
    // Outputs, fp32 parameters and parameters without 16-byte rows: O goes
    // through LDS in fp32, half a tile at a time (the rows of the wavefronts
    // wm = half), in the parameter's layout, and leaves as whole rows, 8
    // elements a thread and unit, W read up to 4 units ahead.  Straight from
    // the registers (16-byte pieces of 32 rows, or 64 to 128 bytes of 8) the
    // last step of 72 fp32 parameters of hidden 768 took 325 us a launch, this
    // way 177; of 512 mixed bf16 outputs 2.60 and 1.5 ms in all.
    constexpr int HR = BM / WM;                            // rows of X in a half
    constexpr int NUN = HR * BN / 8 / (64 * NW);           // units per thread
    float* const os = reinterpret_cast<float*>(smem);
    static_assert(HR * BN * 4 <= BN * (BM * 2 + 8) || HR * BN * 4 <= Cfg::LDS, "half a tile in fp32");
    // element (row, col) of the half: row-major, or (parameter l x s) by
    // columns with 16-byte chunk k of column c at k ^ (c % 16)
    auto oat = [](int r, int c) { return r * BN + c; };
    auto oat_t = [](int c, int r) { return c * HR + ((((r >> 2) ^ (c & 15)) << 2) | (r & 3)); };
    const int ush = 31 - __builtin_clz((tr ? HR : BN) / 8);  // units per row: a power of two
#pragma unroll 1
    for (int half = 0; half < WM; ++half) {
      if (wm == half) {
        const float sc = SPLIT ? 1.f : osc;
        static_for<BI>([&](auto I) {
          static_for<BJ>([&](auto J) {
            static_for<4>([&](auto G) {
              constexpr int i = decltype(I)::value, j = decltype(J)::value, g = decltype(G)::value;
              const int r = i * 32 + 8 * g + 4 * fsel, c = wn * (BN / WN) + j * 32 + frow;
              const f32x16_t& o = acc[i][j];
              if (tr) {
                *reinterpret_cast<float4*>(os + oat_t(c, r)) =
                    make_float4(sc * o[4 * g], sc * o[4 * g + 1], sc * o[4 * g + 2], sc * o[4 * g + 3]);
              } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) os[oat(r + q, c)] = sc * o[4 * g + q];
              }
            });
          });
        });
      }
      __syncthreads();
      const int r0 = bm * BM + half * HR, x0 = bn * BN;    // the half's origin in X
      const int wr = tr ? x0 : r0, wc = tr ? r0 : x0;      // and in the parameter
      const int rows = tr ? min(BN, ga.l - x0) : min(HR, ga.s - r0), cols = tr ? min(HR, ga.s - r0) : min(BN, ga.l - x0);
      constexpr int AH = 4;
#pragma unroll 1
      for (int t0 = 0; t0 < NUN; t0 += AH) {
        Raw8<PT> w[AH];
        int r[AH], c[AH];
#pragma unroll
        for (int t = 0; t < AH; ++t) {
          const int u = threadIdx.x + 64 * NW * (t0 + t);
          r[t] = u >> ush;
          c[t] = (u & ((1 << ush) - 1)) * 8;
          if (FK == 0 && wv.vec8 && r[t] < rows && c[t] + 8 <= cols) w[t] = read8<PT>(wv, w_index(wv, wr + r[t], wc + c[t]));
        }
#pragma unroll
        for (int t = 0; t < AH; ++t) {
          const int n = min(8, cols - c[t]);
          if (r[t] >= rows || n <= 0) continue;
          float o[8];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float4 v = *reinterpret_cast<const float4*>(os + (tr ? oat_t(r[t], c[t] + 4 * h) : oat(r[t], c[t] + 4 * h)));
            o[4 * h] = v.x; o[4 * h + 1] = v.y; o[4 * h + 2] = v.z; o[4 * h + 3] = v.w;
          }
          apply8<FK, PT>(wv, w_index(wv, wr + r[t], wc + c[t]), o, n, w[t]);
        }
      }
      __syncthreads();  // the next half, or the next tile's loads, overwrite the staging area
    }
  }
  if constexpr (stage_n) {
#pragma unroll 1
  for (int plane = 0; plane < (SPLIT ? 3 : 1); ++plane) {
    blocks(plane == 0 && !(SPLIT && EPI != EPI_GRAM) ? osc : 1.f);
    __syncthreads();
    int ow = wave;
    if constexpr (SPLIT) asm volatile("" : "+s"(ow));  // (keeps the row addresses inside the loop: hoisted, they spill)
    // Copy-out: a wave instruction writes 4 rows x 256 bytes.  In each
    // 16-lane group G, lane t (r = t / 4, q = t % 4) addresses the 8 bytes
    // (rows R .. R + 3) of column C0 + 8 q + r, then of column C0 + 8 q + 4 + r;
    // ds_read_b64_tr_b16 hands lane t row R + t % 4, columns C0 + 8 (t / 4)
    // .. + 3 and + 4 .. + 7: 16 consecutive bytes of one row.
    const int G = lane >> 4, t = lane & 15;
    const int ra = ((t & 3) * 8 + (t >> 2)) * TST;     // column offset of this lane's first address
    const int rrow = t & 3, rcol = 8 * (t >> 2);       // what it receives
    constexpr int KC = BM * BN * 2 / 1024 / NW;   // store instructions per wave
    static_assert(KC * NW * 1024 == BM * BN * 2, "copy-out: whole instructions per wave");
    auto out_row = [&](int it, auto diagc) __attribute__((always_inline)) {
      const int task = it * NW + ow;                   // 4 rows x 128 columns
      constexpr int CB = BN / 128;
      const int R = 4 * (task / CB), C0 = 128 * (task % CB) + 32 * G;
      if (R >= mv || 128 * (task % CB) >= nv) return;  // (wave-uniform)
      const char* a = smem + C0 * TST + ra + 2 * R;
      const uint2 lo = tr_read_b64(a), hi = tr_read_b64(a + 4 * TST);
      u32x4_t v{lo.x, lo.y, hi.x, hi.y};
      const int row = R + rrow, c = C0 + rcol;
      if (decltype(diagc)::value && c < row) {
        // columns c .. c + 7 below the diagonal hold (col, row): row `row`
        // of the staged column-major tile, i.e. column `row`, rows c ..
        const char* m = smem + row * TST + 2 * c;
        const uint2 l0 = *reinterpret_cast<const uint2*>(m), l1 = *reinterpret_cast<const uint2*>(m + 8);
        const u32x4_t low{l0.x, l0.y, l1.x, l1.y};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int c2 = c + 2 * d;                    // elements c2 (low half) and c2 + 1
          v[d] = c2 + 1 < row ? low[d] : (c2 < row ? ((low[d] & 0xffffu) | (v[d] & 0xffff0000u)) : v[d]);
        }
      }
      store_out(reinterpret_cast<u32x4_t*>(C + static_cast<int64_t>(bm * BM + row) * ga.ldc + (bn * BN + c) * 2), v);
    };
    if (diag) {
      for (int it = 0; it < KC; ++it) out_row(it, std::true_type{});
    } else {
#pragma unroll
      for (int it = 0; it < KC; ++it) out_row(it, std::false_type{});
      if (pair_mirror) {  // its rows are the staged columns
        for (int idx = threadIdx.x; idx < BN * TRC; idx += 64 * NW) {
          const int c = idx / TRC, ch = idx % TRC;
          const char* m = smem + c * TST + ch * 16;
          const uint2 l0 = *reinterpret_cast<const uint2*>(m), l1 = *reinterpret_cast<const uint2*>(m + 8);
          store_out(reinterpret_cast<u32x4_t*>(C + static_cast<int64_t>(bn * BN + c) * ga.ldc + bm * BM * 2 + ch * 16),
                    u32x4_t{l0.x, l0.y, l1.x, l1.y});
        }
      }
    }
    __syncthreads();  // the next plane, or the next tile's loads, overwrite the staging area
    C += ga.c_plane;
  }
  }
}

// Persistent launch: one workgroup per CU slot loops over tiles in rounds.
// Workgroup b runs on XCD b % 8; in round r the XCD's workgroups take the
// contiguous logical range r*G + (b % 8)*(G/8) + [0, G/8), i.e. a compact
// block of the banded order, and start it together, so the tiles of a block
// stay in step and share each operand slab through the XCD's L2.
template <int EPI, class Cfg, bool SPLIT>
__global__ __launch_bounds__(64 * Cfg::NW) __attribute__((amdgpu_waves_per_eu(Cfg::WPE, Cfg::WPE)))
void k_gemm_tile(GemmArgs ga) {
  // epilogue staging: the output tile (direct rows) or the mirrored tile
  constexpr int STAGED_C = Cfg::BM * Cfg::BN * 2, STAGED_T = Cfg::BN * (Cfg::BM * 2 + 8);
  constexpr int STAGED = STAGED_C > STAGED_T ? STAGED_C : STAGED_T;
  static_assert(STAGED <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(1024))) char smem[Cfg::LDS > STAGED ? Cfg::LDS : STAGED];
  const int G = static_cast<int>(gridDim.x), b = static_cast<int>(blockIdx.x);
  for (int r = 0;; ++r) {
    const int logical = (G % 8 == 0) ? r * G + (b & 7) * (G / 8) + (b >> 3) : r * G + b;
    if (logical >= ga.total_tiles) break;
    int mat, bm, bn;
    tile_from_logical(ga, logical, mat, bm, bn);
    gemm_tile_body<EPI, Cfg, SPLIT>(ga, smem, mat, bm, bn);
  }
}

// One launch over the tiles of several chunks (a group): the product of
// the same Newton-Schulz step for every chunk, each with its own arguments.
// Tiles are numbered chunk by chunk (start[c] is chunk c's first), and the
// rounds run as in k_gemm_tile, so a tile of one chunk and a tile of the
// next can share a round.  Each tile's arithmetic is that of k_gemm_tile.
constexpr int kMaxGroup = 8;
struct GroupArgs {
  GemmArgs ga[kMaxGroup];
  int32_t start[kMaxGroup + 1];
  int32_t n;
};
static_assert(sizeof(GroupArgs) <= 4096, "kernel argument size");

template <int EPI, class Cfg>
__global__ __launch_bounds__(64 * Cfg::NW) __attribute__((amdgpu_waves_per_eu(Cfg::WPE, Cfg::WPE)))
void k_gemm_group(GroupArgs gr) {
  constexpr int STAGED_C = Cfg::BM * Cfg::BN * 2, STAGED_T = Cfg::BN * (Cfg::BM * 2 + 8);
  constexpr int STAGED = STAGED_C > STAGED_T ? STAGED_C : STAGED_T;
  __shared__ __attribute__((aligned(1024))) char smem[Cfg::LDS > STAGED ? Cfg::LDS : STAGED];
  const int G = static_cast<int>(gridDim.x), b = static_cast<int>(blockIdx.x);
  const int total = gr.start[gr.n];
  for (int r = 0;; ++r) {
    const int logical = (G % 8 == 0) ? r * G + (b & 7) * (G / 8) + (b >> 3) : r * G + b;
    if (logical >= total) break;
    int c = 0;
    while (c + 1 < gr.n && logical >= gr.start[c + 1]) ++c;
    const GemmArgs& ga = gr.ga[c];
    int mat, bm, bn;
    tile_from_logical(ga, logical - gr.start[c], mat, bm, bn);
    gemm_tile_body<EPI, Cfg, false>(ga, smem, mat, bm, bn);
  }
}

// B = b A for a step with c = 0 (cubic tables): no product, one pass over the
// stored (upper-triangle 256 x 256) tiles of A, a 128 x 128 block a workgroup.
template <typename XT>
__global__ __launch_bounds__(256) void k_scale_upper(GemmArgs ga, int t) {
  const int mat = blockIdx.x / (t * t), b = blockIdx.x % (t * t), bm = b / t, bn = b % t;
  if (bn / 2 < bm / 2) return;
  const char* E = ga.E + mat * ga.e_mat + static_cast<int64_t>(bm) * 128 * ga.lde + bn * 256;
  char* C = ga.C + mat * ga.c_mat + static_cast<int64_t>(bm) * 128 * ga.ldc + bn * 256;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = i * 16 + (threadIdx.x >> 4), col = (threadIdx.x & 15) * 8;
    float v[8], w[8];
    const char* e = E + static_cast<int64_t>(row) * ga.lde;
    load8(reinterpret_cast<const uint16_t*>(e), col, v);
    for (int p = 1; p < Store<XT>::planes; ++p) {
      load8(reinterpret_cast<const uint16_t*>(e + p * ga.p_plane), col, w);
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] += w[q];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] *= ga.alpha;
    store8x<XT>(reinterpret_cast<uint16_t*>(C + static_cast<int64_t>(row) * ga.ldc), col, ga.c_plane / 2, v);
  }
}

// Update from X0 when K = 0: O is X0 in the caller's layout (the direct
// buffer), one thread per element of the u-domain; grid = (ceil(rows*cols /
// 256), matrices).
template <typename XT>
__global__ __launch_bounds__(256) void k_apply_x0(const MatDesc* __restrict__ desc, ChunkGeom cg,
                                                  const XT* __restrict__ X, const XT* __restrict__ XTb,
                                                  const float* __restrict__ xscale, int final_kind) {
  const int m = blockIdx.y;
  const MatDesc md = desc[m];
  const int64_t numel = static_cast<int64_t>(md.rows) * md.cols;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= numel) return;
  const int64_t ur = i / md.cols, uc = i - ur * md.cols;
  const int64_t matX = static_cast<int64_t>(cg.S) * cg.L;
  const XT* D = (md.transposed ? XTb : X) + m * matX;
  const int ldD = md.transposed ? cg.S : cg.L;
  const float o = to_f32<XT>(D[ur * ldD + uc]) * xscale[m];  // X0 = r X~ (or X0 itself, scale 1)
  const int64_t w = view_index(md, ur, uc);
  if (final_kind == 0) {
    const float wv = load_as_f32(md.W, w, cg.param_dtype);
    store_from_f32(md.W, w, cg.param_dtype, fmaf(md.decay, wv, -md.upd_scale * o));
  } else {
    store_from_f32(md.out, w, cg.param_dtype, o);
  }
}

// ---------------------------------------------------------------------------
// Host-side launch sequence for one chunk.
// ---------------------------------------------------------------------------
#ifndef MUON_PERSISTENT
#define MUON_PERSISTENT 1
#endif

// Compute units of the current device (queried once per device).
int device_cu_count() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cache[dev] = n;
  }
  return cache[dev];
}

template <typename XT>
hipError_t launch_scale_upper(const GemmArgs& ga, int nmat, hipStream_t st) {
  const int t = ga.m_ext / 128;
  hipLaunchKernelGGL(k_scale_upper<XT>, dim3(static_cast<unsigned>(t * t) * static_cast<unsigned>(nmat)), dim3(256), 0,
                     st, ga, t);
  return hipGetLastError();
}

// The launchers set `exec` to the flops the launch's MFMAs execute: whole
// tiles of the kernel that runs the product, of the symmetric ones the upper
// tiles, six products of planes for one of SPLIT values; none for a scaling.
template <class Cfg>
double executed(const GemmArgs& ga, int pairs) {  // ga in tiles of Cfg
  return 2.0 * pairs * double(ga.total_tiles) * Cfg::BM * Cfg::BN * double(ga.k_slabs) * (Cfg::SLAB / 2);
}

template <class Cfg, bool SPLIT>
hipError_t launch_tile(int epi, GemmArgs ga, int nmat, hipStream_t st, double& exec) {
  // ga arrives in 128 x 128 tiles and 128-byte slabs
  ga.m_ext = ga.tiles_m * kTile;
  ga.n_ext = ga.tiles_n * kTile;
  ga.tiles_m = (ga.m_ext + Cfg::BM - 1) / Cfg::BM;
  ga.tiles_n = (ga.n_ext + Cfg::BN - 1) / Cfg::BN;
  ga.tiles_per_mat = ga.syrk ? ga.tiles_m * (ga.tiles_m + 1) / 2 : ga.tiles_m * ga.tiles_n;
  ga.k_slabs = ga.k_slabs * 128 / Cfg::SLAB;
  ga.total_tiles = ga.tiles_per_mat * nmat;
  exec = epi == EPI_POLY && ga.beta == 0.f ? 0.0 : executed<Cfg>(ga, SPLIT ? 6 : 1);
  // B = b A + c A^2 = c (A^2 + (b/c) A): the A term joins the accumulators
  // in the main loop
  if (epi == EPI_POLY) {
    if (ga.beta == 0.f) return launch_scale_upper<std::conditional_t<SPLIT, Split3, uint16_t>>(ga, nmat, st);
    if (!SPLIT) ga.alpha = ga.alpha / ga.beta;
  }
  // one workgroup per CU slot (persistent), never more workgroups than tiles
  const int slots = device_cu_count() * (160 * 1024 / Cfg::LDS);
  const int g = MUON_PERSISTENT ? min(ga.total_tiles, slots) : ga.total_tiles;
  const dim3 grid(static_cast<unsigned>(g)), block(64 * Cfg::NW);
  switch (epi) {
    case EPI_GRAM: hipLaunchKernelGGL((k_gemm_tile<EPI_GRAM, Cfg, SPLIT>), grid, block, 0, st, ga); break;
    case EPI_POLY: hipLaunchKernelGGL((k_gemm_tile<EPI_POLY, Cfg, SPLIT>), grid, block, 0, st, ga); break;
    case EPI_UPDATE: hipLaunchKernelGGL((k_gemm_tile<EPI_UPDATE, Cfg, SPLIT>), grid, block, 0, st, ga); break;
    default: {
      const bool o = ga.final_kind != 0, f32 = ga.param_dtype == DT_F32;
      if (!o && !f32 && ga.w_rows16) hipLaunchKernelGGL((k_gemm_tile<EPI_FINAL_W_BF16, Cfg, SPLIT>), grid, block, 0, st, ga);
      else if (!o && !f32) hipLaunchKernelGGL((k_gemm_tile<EPI_FINAL_W_BF16_ANY, Cfg, SPLIT>), grid, block, 0, st, ga);
      else if (!o) hipLaunchKernelGGL((k_gemm_tile<EPI_FINAL_W_F32, Cfg, SPLIT>), grid, block, 0, st, ga);
      else if (!f32) hipLaunchKernelGGL((k_gemm_tile<EPI_FINAL_O_BF16, Cfg, SPLIT>), grid, block, 0, st, ga);
      else hipLaunchKernelGGL((k_gemm_tile<EPI_FINAL_O_F32, Cfg, SPLIT>), grid, block, 0, st, ga);
      break;
    }
  }
  return hipGetLastError();
}

// The products of one step for a group of chunks on 256 x 256 tiles:
// each chunk's arguments prepared as launch_tile prepares them, one
// persistent launch over all their tiles.  The chunks share the product, the
// final kind and the parameter dtype.
template <class Cfg>
hipError_t launch_group(int epi, const GemmArgs* gas, const int* nmats, int n, hipStream_t st, double& exec) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  exec = 0.0;
  GroupArgs gr{};
  gr.start[0] = 0;
  bool rows16 = true;
  for (int i = 0; i < n; ++i) {
    GemmArgs ga = gas[i];
    const int c = gr.n;
    ga.m_ext = ga.tiles_m * kTile;
    ga.n_ext = ga.tiles_n * kTile;
    ga.tiles_m = (ga.m_ext + Cfg::BM - 1) / Cfg::BM;
    ga.tiles_n = (ga.n_ext + Cfg::BN - 1) / Cfg::BN;
    ga.tiles_per_mat = ga.syrk ? ga.tiles_m * (ga.tiles_m + 1) / 2 : ga.tiles_m * ga.tiles_n;
    ga.k_slabs = ga.k_slabs * 128 / Cfg::SLAB;
    ga.total_tiles = ga.tiles_per_mat * nmats[i];
    if (epi == EPI_POLY) {
      if (ga.beta == 0.f) {
        const hipError_t e = launch_scale_upper<uint16_t>(ga, nmats[i], st);
        if (e != hipSuccess) return e;
        continue;
      }
      ga.alpha = ga.alpha / ga.beta;
    }
    if (c > 0 && (ga.final_kind != gr.ga[0].final_kind || ga.param_dtype != gr.ga[0].param_dtype))
      return hipErrorInvalidValue;
    exec += executed<Cfg>(ga, 1);
    rows16 = rows16 && ga.w_rows16;
    gr.ga[c] = ga;
    gr.start[c + 1] = gr.start[c] + ga.total_tiles;
    gr.n = c + 1;
  }
  const int total = gr.start[gr.n];
  if (total == 0) return hipSuccess;
  const int slots = device_cu_count() * (160 * 1024 / Cfg::LDS);
  const dim3 grid(static_cast<unsigned>(min(total, slots))), block(64 * Cfg::NW);
  switch (epi) {
    case EPI_GRAM: hipLaunchKernelGGL((k_gemm_group<EPI_GRAM, Cfg>), grid, block, 0, st, gr); break;
    case EPI_POLY: hipLaunchKernelGGL((k_gemm_group<EPI_POLY, Cfg>), grid, block, 0, st, gr); break;
    case EPI_UPDATE: hipLaunchKernelGGL((k_gemm_group<EPI_UPDATE, Cfg>), grid, block, 0, st, gr); break;
    default: {
      const bool o = gr.ga[0].final_kind != 0, f32 = gr.ga[0].param_dtype == DT_F32;
      if (!o && !f32 && rows16) hipLaunchKernelGGL((k_gemm_group<EPI_FINAL_W_BF16, Cfg>), grid, block, 0, st, gr);
      else if (!o && !f32) hipLaunchKernelGGL((k_gemm_group<EPI_FINAL_W_BF16_ANY, Cfg>), grid, block, 0, st, gr);
      else if (!o) hipLaunchKernelGGL((k_gemm_group<EPI_FINAL_W_F32, Cfg>), grid, block, 0, st, gr);
      else if (!f32) hipLaunchKernelGGL((k_gemm_group<EPI_FINAL_O_BF16, Cfg>), grid, block, 0, st, gr);
      else hipLaunchKernelGGL((k_gemm_group<EPI_FINAL_O_F32, Cfg>), grid, block, 0, st, gr);
      break;
    }
  }
  return hipGetLastError();
}

int64_t quarter_tiles(const GemmArgs& ga) {  // 128 x 128 tiles of a matrix
  const int64_t m = ga.tiles_m, n = ga.tiles_n;
  return ga.syrk ? m * (m + 1) / 2 : m * n;
}
// At most one 128 x 128 tile per CU and at least 16 slabs: four stages.  Two
// and four stages, us per launch: Gram of 1024 x 4096 54 / 38, of 2048 x 5632
// 72 / 52, update of 2048 x 2048 36 / 31 (one matrix each); with 8 slabs or
// fewer the three slabs issued first cost what they gain: 512 x 512 12.5 / 12.8,
// eight 256 x 1024 9.1 / 10.3.
bool deep_tiles(const GemmArgs& ga, int nmat) {
  return ga.k_slabs >= 16 && quarter_tiles(ga) * nmat <= device_cu_count();
}
// Whether a launch runs on 128 x 128 tiles (CfgQuarter): where 256 x 256
// tiles would leave many CUs idle, in a last round or in the only one.
// The model is fitted to single launches on an MI355X (us, nk slabs of 64 k):
//   256 x 256: each round of one tile per CU takes (1.15 + 0.4 f) nk + 4 + 8 f,
//     f the share of the rounds' slots that have a tile (a full chip runs at
//     a lower clock and misses more often in L2);
//   128 x 128: a round of two tiles per CU takes nk + 5, a last round costs
//     about half of one more, and a single round is a little cheaper.
// Measured per launch, 256 / 128: Gram of 2048 x 5632, three matrices 119 / 89,
// one 114 / 73; update of 512 x 512, one matrix 21 / 12, 256 matrices 104 /
// 122; update of 4096 x 11008 319 / 387; Gram of 768 x 768, 48 matrices 54 / 39.
// The smaller tiles are taken where the model says they save a tenth: nearer
// ties are within its error, and in a call on two streams the other stream's
// work would have used the CUs that 256 x 256 tiles leave idle, while 128 x 128
// tiles load twice as much (two streams, 2 x 4096^2 and 4096 x 11008, whose
// Gram and polynomial are at 0.96: 5.40 ms on the small tiles, 5.23 on the
// large; 3 and 2 of them 9.36 and 8.95; no other of 34 calls moved by more
// than the runs differ, and at 0.65 several lost 5 to 60%).
struct TileCosts { double small, large; };         // us on 128 x 128 and on 256 x 256 tiles
double large_tile_us(double f, double nk) { return (1.15 + 0.4 * f) * nk + 4.0 + 8.0 * f; }
int64_t large_tiles(const GemmArgs& ga) {
  const int64_t m = (ga.tiles_m + 1) / 2, n = (ga.tiles_n + 1) / 2;
  return ga.syrk ? m * (m + 1) / 2 : m * n;
}
TileCosts tile_costs(const GemmArgs& ga, int nmat, bool split) {
  const double t1 = double(nmat) * double(quarter_tiles(ga)), t2 = double(nmat) * double(large_tiles(ga));
  const double cus = device_cu_count(), nk = ga.k_slabs * (split ? 6 : 1);
  const double rounds2 = std::ceil(t2 / cus), f = t2 / (rounds2 * cus);
  const double r1 = t1 / (2.0 * cus), rounds1 = std::ceil(r1);
  TileCosts c;
  c.large = rounds2 * large_tile_us(f, nk);
  c.small = r1 <= 1.0 ? 0.95 * nk + 2.0 : (1.03 * r1 + 0.5) * nk + 5.0 * rounds1;
  if (!split && deep_tiles(ga, nmat)) c.small = 0.6 * nk + 4.0;
  return c;
}
enum class Tiles { square, quarter, deep };
Tiles tiles_of(const GemmArgs& ga, int nmat, bool split) {
  const TileCosts c = tile_costs(ga, nmat, split);
  if (c.small >= 0.9 * c.large) return Tiles::square;
  return !split && deep_tiles(ga, nmat) ? Tiles::deep : Tiles::quarter;
}

// The products on k_gemm_nt: rows past the tile kernel's 32-bit offsets
// (chunk_on_tiles).
template <typename T>
hipError_t launch_gemm(int epi, GemmArgs ga, int nmat, hipStream_t st, double& exec) {
  exec = 2.0 * double(nmat) * ga.tiles_per_mat * kTile * kTile * double(ga.k_slabs) * (128 / sizeof(T));
  const dim3 grid(static_cast<unsigned>(ga.tiles_per_mat) * nmat), block(256);
  switch (epi) {
    case EPI_GRAM: hipLaunchKernelGGL((k_gemm_nt<T, EPI_GRAM>), grid, block, 0, st, ga); break;
    case EPI_POLY: hipLaunchKernelGGL((k_gemm_nt<T, EPI_POLY>), grid, block, 0, st, ga); break;
    case EPI_UPDATE: hipLaunchKernelGGL((k_gemm_nt<T, EPI_UPDATE>), grid, block, 0, st, ga); break;
    default: hipLaunchKernelGGL((k_gemm_nt<T, EPI_FINAL>), grid, block, 0, st, ga); break;
  }
  return hipGetLastError();
}

// Brackets one launch with the optional timer.
struct Timed {
  LaunchTimer* t;
  int kind;
  hipStream_t st;
  Timed(LaunchTimer* timer, int k, hipStream_t s) : t(timer), kind(k), st(s) {
    if (t) t->begin(kind, st);
  }
  void done(double flops, double exec_flops, double bytes) {
    if (t) t->end(kind, st, flops, exec_flops, bytes);
  }
};

// ---------------------------------------------------------------------------
// Fused Newton-Schulz for the smaller matrices of short side up to 128
// (k_ns_small; which, chunk_is_small): the whole step
// of a chunk -- momentum, norm, X0, every Newton-Schulz step and the update --
// in one launch.  Such matrices are far too small for the tile kernels: a
// 128 x 256 fp32 product fills one or two workgroups, so separate launches
// leave the device idle and each product runs on a single compute unit.
//
// Each matrix is taken by a group of G = RB x CB workgroups: RB row blocks
// of 32 rows of X (the padded short side Sx = 32 RB) times CB column groups
// (a function of the shape alone, so results do not depend on the batch).
// Per step, every product on MFMA in 16 x 16 units shared out over the four
// wavefronts:
//   A[Ri, Cc] = X[Ri, :] X[Cc, :]^T             column blocks c = j, j + CB, ..
//   -- group barrier --
//   B[Ri, Cc] = b A[Ri, Cc] + c A[Ri, :] A[Cc, :]^T   (A symmetric)
//   -- group barrier (CB > 1: rows Ri of B come from several workgroups) --
//   X'[Ri, Dd] = a X[Ri, Dd] + B[Ri, :] X^T[Dd, :]^T  column blocks d = j, j + CB, ..
//   -- group barrier --
// X is kept in both orientations, so every operand is a row-major matrix
// with K contiguous, stored tiled (see ti).  The prologue writes u itself
// into X and applies r = 1 / (||u|| + eps) in the first step's products
// (exact fp32 u; X0 = r u is formed first when r is far from 1).  The last
// step writes W (or the output) straight from the fp32 values, in the
// parameter's own layout.  Extents are padded to multiples of 32; the
// padding of X, A and B is written as zeros and stays zero.
//
// The members of a group run on one XCD (workgroup b runs on XCD b % 8, and
// each workgroup checks its XCC_ID against its group's): their data meets in
// that XCD's L2, so a barrier drains the memory operations of every wave and
// bumps a counter, and every read of data that other members wrote is a
// non-temporal load, which bypasses the compute unit's own (incoherent) L1.
// Should a group find its members spread over XCDs, every barrier of that
// group also writes back and invalidates at device scope.  Spins are
// bounded, so every wave ends whatever happens.
// ---------------------------------------------------------------------------
struct SmallArgs {
  const MatDesc* desc;
  StepScalars sc;
  int32_t s, l, S, L, Sx, Lx;
  int32_t nmat, G, RB, CB, groups, K;
  int32_t param_dtype;
  char* X[2];
  char* XT[2];
  char* A;
  char* B;
  int64_t matX, matA;        // bytes per matrix
  double* partials;          // nmat x kSmallMaxGroup
  unsigned* sync;            // per group: [0] counter, [1] spin timeouts, [2 .. 2 + G) member XCC ids
  float coeffs[3 * 64];      // (a, b, c) per step
};

__device__ __forceinline__ unsigned xcc_id() {
  return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 15u;  // HW_REG_XCC_ID, bits [3:0]
}

__device__ __forceinline__ void group_barrier(unsigned* sync, unsigned target, bool local) {
  __builtin_amdgcn_s_waitcnt(0);  // this wave's loads and stores are done (stores reached L2)
  __syncthreads();
  if (threadIdx.x == 0) {
    if (!local) __threadfence();
    __hip_atomic_fetch_add(sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned spins = 0;
    while (__hip_atomic_load(sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      __builtin_amdgcn_s_sleep(2);
      if (++spins > (1u << 22)) {  // never expected: count it and go on
        __hip_atomic_fetch_add(sync + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
    if (!local) __atomic_thread_fence(__ATOMIC_ACQUIRE);
  }
  __syncthreads();
}

// Loads of data other members wrote: non-temporal, so they never allocate, and
// never hit, a line in this compute unit's L1, which is not coherent with
// the other compute units (measured: plain loads after the barrier return
// stale L1 lines; non-temporal ones do not).  The L2 they read is the one
// the writers' stores reached.
__device__ __forceinline__ u32x4_t ld16(const char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
}

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// 16 x 16 blocks of P Q^T (fp32), K in k-groups of 16 elements (64 bytes of a
// row).  Lane l loads the 16 bytes of row l % 16 at byte 16 (l / 16) of a
// group and issues four v_mfma_f32_16x16x4_f32, the j-th taking element j
// (k = j, 4 + j, 8 + j, 12 + j across the lanes' four row quarters); even
// and odd groups accumulate apart and are added at the end of the block.
// Result layout: lane l, register r holds row 4 (l / 16) + r, column l % 16.
//
// small_units runs the 16 x 16 units of one phase, shared out round-robin
// over the four wavefronts.  unit(u, P, Q, row0, col0) gives unit u's
// operands (the first chunks of its 16-row blocks, tiled layout) and origin; pre(row, col) is loaded
// with the unit's first operands; epi(row, col, value, term) receives the 4
// values of each lane.  A wavefront's units and their K batches form one
// stream: the loads of the next batch (of the same or the next unit) are in
// flight while the MFMAs of the current one issue.
constexpr int kSmallBatch = 8;  // k-groups per batch
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// The fused launch keeps X, X^T, A and B in a tiled layout: each 16-row x
// 16-k chunk of a row-major matrix is 1 KB, stored in the order of the lanes
// that take it as an MFMA operand (lane l: row l % 16, k 4 (l / 16) .. + 3),
// chunks row-block major.  A wavefront's operand load is then 1 KB of
// consecutive bytes (whole cache lines), where the row-major layout touched
// 16 lines for 64 bytes each (measured 4x slower).  Element (r, k) of a
// matrix with kg k-groups per row, in floats:
__device__ __forceinline__ int64_t ti(int r, int k, int kg) {
  return (static_cast<int64_t>(r >> 4) * kg + (k >> 4)) * 256 + (((k & 15) >> 2) * 16 + (r & 15)) * 4 + (k & 3);
}
// The bf16 form: 16-row x 32-k chunks of 1 KB (lane l: row l % 16,
// k 8 (l / 16) .. + 7, the operand of v_mfma_f32_16x16x32_bf16), kg k-groups
// of 32 per row, in elements.
__device__ __forceinline__ int64_t ti_b(int r, int k, int kg) {
  return (static_cast<int64_t>(r >> 4) * kg + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (r & 15)) * 8 + (k & 7);
}
template <typename XT>
__device__ __forceinline__ int64_t tix(int r, int k, int kg) {
  if constexpr (sizeof(XT) == 2) return ti_b(r, k, kg);
  else return ti(r, k, kg);
}

template <typename XT, typename Unit, typename Pre, typename Epi>
__device__ __forceinline__ void small_units(int nunits, int kg, Unit&& unit, Pre&& pre, Epi&& epi) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int mine = nunits > wave ? (nunits - wave + 3) / 4 : 0;  // this wavefront's units
  const int nbat = (kg + kSmallBatch - 1) / kSmallBatch;
  const int total = mine * nbat;
  if (total == 0) return;
  struct Batch {
    u32x4_t a[kSmallBatch], b[kSmallBatch];
    float term[4];
  };
  // the operands of stream item `it` (unit it / nbat, batch it % nbat)
  auto issue = [&](int it, Batch& bt) __attribute__((always_inline)) {
    const int u = wave + 4 * (it / nbat), bb = it % nbat;
    const char* P;
    const char* Q;
    int row0, col0;
    unit(u, P, Q, row0, col0);
    const char* pr = P + lane * 16;
    const char* qr = Q + lane * 16;
    const int g0 = bb * kSmallBatch;
#pragma unroll
    for (int t = 0; t < kSmallBatch; ++t)
      if (g0 + t < kg) {
        bt.a[t] = ld16(pr + static_cast<int64_t>(g0 + t) * 1024);
        bt.b[t] = ld16(qr + static_cast<int64_t>(g0 + t) * 1024);
      }
    if (bb == 0) {
      const int row = row0 + 4 * (lane >> 4), col = col0 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) bt.term[r] = pre(row + r, col);
    }
  };
  f32x4_t acc[2];
  float term[4];
  auto consume = [&](int it, Batch& bt) __attribute__((always_inline)) {
    const int bb = it % nbat, g0 = bb * kSmallBatch;
    if (bb == 0) {
      acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r) term[r] = bt.term[r];
    }
#pragma unroll
    for (int t = 0; t < kSmallBatch; ++t)
      if (g0 + t < kg) {
        if constexpr (sizeof(XT) == 2) {
          acc[t & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, bt.a[t]),
                                                               __builtin_bit_cast(bf16x8_t, bt.b[t]), acc[t & 1], 0, 0, 0);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[t & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(bt.a[t][j]), __uint_as_float(bt.b[t][j]),
                                                              acc[t & 1], 0, 0, 0);
        }
      }
    if (bb == nbat - 1) {
      const int u = wave + 4 * (it / nbat);
      const char* P;
      const char* Q;
      int row0, col0;
      unit(u, P, Q, row0, col0);
      const f32x4_t v = acc[0] + acc[1];
      const int row = row0 + 4 * (lane >> 4), col = col0 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) epi(row + r, col, v[r], term[r]);
    }
  };
  Batch b0, b1;
  issue(0, b0);
  for (int it = 0; it < total; it += 2) {
    if (it + 1 < total) issue(it + 1, b1);
    consume(it, b0);
    if (it + 1 >= total) break;
    if (it + 2 < total) issue(it + 2, b0);
    consume(it + 1, b1);
  }
}

template <typename T>
__device__ __forceinline__ void put(char* base, int64_t idx, float v) {
  reinterpret_cast<T*>(base)[idx] = from_f32<T>(v);
}
template <typename T>
__device__ __forceinline__ float get(const char* base, int64_t idx) {
  return to_f32<T>(__builtin_nontemporal_load(reinterpret_cast<const T*>(base) + idx));
}

// XT: float (fp32 Newton-Schulz, X exact u) or uint16_t (bf16: X, A and B
// stored as bfloat16 between the products, fp32 accumulation).
template <typename GT, typename XT, bool MOM>
__global__ __launch_bounds__(256) void k_ns_small(SmallArgs sa) {
  constexpr int KG = sizeof(XT) == 2 ? 32 : 16;  // k per operand chunk
  __shared__ double red4[4];
  const int b = blockIdx.x, xcd = b & 7, slot = b >> 3;
  const int group = (slot / sa.G) * 8 + xcd, member = slot % sa.G;
  const int bi = member / sa.CB, bj = member % sa.CB;  // row block, column group
  unsigned* const sync = sa.sync + group * 64;
  if (threadIdx.x == 0) __hip_atomic_store(sync + 2 + member, xcc_id(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  unsigned nbar = 0;
  bool local = false;
  const int kgx = sa.L / KG, kgs = sa.S / KG;      // k-groups per row of X, of X^T, A and B
  const int ncb = sa.Lx / 32;                                    // column blocks of X
  const int c0 = bj * ncb / sa.CB, c1 = (bj + 1) * ncb / sa.CB;  // this member's, in the prologue
  const int w = (c1 - c0) * 32;                                  // prologue columns of this member
  const float beta = sa.sc.beta, omb = sa.sc.one_minus_beta;
  for (int m = group; m < sa.nmat; m += sa.groups) {
    const MatDesc md = sa.desc[m];
    const bool tr = md.transposed != 0;
    const GT* g = static_cast<const GT*>(md.g);
    char* X0 = sa.X[0] + m * sa.matX;
    char* XT0 = sa.XT[0] + m * sa.matX;
    // element e of the member's 32 x w block of X: consecutive threads on
    // consecutive elements of u's rows (coalesced for either orientation)
    auto coord = [&](int e, int& xr, int& xc) {
      if (tr) { xr = bi * 32 + (e & 31); xc = c0 * 32 + (e >> 5); }
      else { xr = bi * 32 + e / w; xc = c0 * 32 + e % w; }
    };
    // ---- prologue pass 1: momentum, u into X (fp32, exact), sum of u^2 ----
    double acc2 = 0.0;
    const int ne = 32 * w;
    for (int e0 = threadIdx.x; e0 < ne; e0 += 256 * 8) {
      float gv[8], bv[8];
      int64_t gi[8], bix[8];
      bool in[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        int xr, xc;
        coord(e0 + 256 * t, xr, xc);
        in[t] = e0 + 256 * t < ne && xr < sa.s && xc < sa.l;
        const int ur = tr ? xc : xr, uc = tr ? xr : xc;
        gi[t] = in[t] ? view_index(md, ur, uc) : 0;
        bix[t] = (MOM && in[t]) ? buf_index(md, ur, uc) : 0;
        gv[t] = in[t] ? to_f32<GT>(g[gi[t]]) : 0.f;
        bv[t] = (MOM && in[t]) ? md.buf[bix[t]] : 0.f;
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (e0 + 256 * t >= ne) continue;
        float u = gv[t];
        if (MOM && in[t]) {
          const float bn = fmaf(beta, bv[t], omb * gv[t]);
          md.buf[bix[t]] = bn;
          u = sa.sc.nesterov ? fmaf(beta, bn, omb * gv[t]) : bn;
        }
        acc2 = fma(static_cast<double>(u), static_cast<double>(u), acc2);
        int xr, xc;
        coord(e0 + 256 * t, xr, xc);
        put<XT>(X0, tix<XT>(xr, xc, kgx), u);
        put<XT>(XT0, tix<XT>(xc, xr, kgs), u);
      }
    }
    const double part = block_sum_256(acc2, red4);
    if (threadIdx.x == 0) sa.partials[static_cast<int64_t>(m) * kSmallMaxGroup + member] = part;
    ++nbar;
    group_barrier(sync, nbar * sa.G, local);
    if (nbar == 1) {  // the members' XCDs are known from here on
      bool same = true;
      for (int q = 0; q < sa.G; ++q)
        same = same && __hip_atomic_load(sync + 2 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                           __hip_atomic_load(sync + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      local = same;
    }
    double nsq = 0.0;
    for (int q = 0; q < sa.G; ++q)
      nsq += __builtin_nontemporal_load(sa.partials + static_cast<int64_t>(m) * kSmallMaxGroup + q);
    const double r = 1.0 / (sqrt(nsq) + static_cast<double>(sa.sc.eps));
    // X holds u itself (exact in fp32).  While r keeps (r u)(r u)^T far
    // inside the fp32 range, the first step applies it (A0 = r^2 u u^T,
    // X1 = r (a u + B0 u)); otherwise, and for K = 0, X0 = r u is formed here.
    const bool fold = sa.K > 0 && r >= 0x1p-40 && r <= 0x1p40;
    const float xs = fold ? static_cast<float>(r) : 1.f;
    float s1, s2;
    split_scale(r, s1, s2);
    // ---- prologue pass 2 (unless folded): X0 = r u over the member's block ----
    if (!fold)
    for (int e0 = threadIdx.x; e0 < ne; e0 += 256 * 8) {
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        int xr, xc;
        coord(e0 + 256 * t, xr, xc);
        float u = 0.f;
        if (e0 + 256 * t < ne) {
          if constexpr (sizeof(XT) == 4) {
            u = get<XT>(X0, tix<XT>(xr, xc, kgx));  // u itself, exact
          } else if (xr < sa.s && xc < sa.l) {
            // X holds u rounded to bf16: form u again from g and the advanced
            // momentum (this thread's own writes), so r u is rounded once
            const int ur = tr ? xc : xr, uc = tr ? xr : xc;
            const float gv = to_f32<GT>(g[view_index(md, ur, uc)]);
            u = gv;
            if (MOM) {
              const float bn = md.buf[buf_index(md, ur, uc)];
              u = sa.sc.nesterov ? fmaf(beta, bn, omb * gv) : bn;
            }
          }
        }
        v[t] = (u * s1) * s2;
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (e0 + 256 * t >= ne) continue;
        int xr, xc;
        coord(e0 + 256 * t, xr, xc);
        if (sa.K == 0) {
          if (xr < sa.s && xc < sa.l) {
            const int64_t pidx = view_index(md, tr ? xc : xr, tr ? xr : xc);
            if (sa.sc.final_kind == 0)
              store_from_f32(md.W, pidx, sa.param_dtype,
                             fmaf(md.decay, load_as_f32(md.W, pidx, sa.param_dtype), -md.upd_scale * v[t]));
            else
              store_from_f32(md.out, pidx, sa.param_dtype, v[t]);
          }
        } else {
          put<XT>(X0, tix<XT>(xr, xc, kgx), v[t]);
          put<XT>(XT0, tix<XT>(xc, xr, kgs), v[t]);
        }
      }
    }
    if (sa.K == 0) continue;
    if (!fold) {
      ++nbar;
      group_barrier(sync, nbar * sa.G, local);
    }
    int cur = 0;
    const int na = (sa.RB - bj + sa.CB - 1) / sa.CB;      // 32-column blocks of A and B of this member
    for (int k = 0; k < sa.K; ++k) {
      const float ca = sa.coeffs[3 * k], cb = sa.coeffs[3 * k + 1], cc = sa.coeffs[3 * k + 2];
      const float sa_ = k == 0 ? xs * xs : 1.f, sx_ = k == 0 ? xs : 1.f;  // the folded r on the first step
      const char* Xc = sa.X[cur] + m * sa.matX;
      const char* XTc = sa.XT[cur] + m * sa.matX;
      char* Am = sa.A + m * sa.matA;
      char* Bm = sa.B + m * sa.matA;
      // unit u of a phase over 32 x 32 blocks: block u / 4, quarter u % 4
      // A = X X^T: rows bi, column blocks bj, bj + CB, ..
      small_units<XT>(
          4 * na, sa.Lx / KG,
          [&](int u, const char*& P, const char*& Q, int& row0, int& col0) {
            row0 = bi * 32 + 16 * ((u & 3) >> 1);
            col0 = (bj + (u >> 2) * sa.CB) * 32 + 16 * (u & 1);
            P = Xc + tix<XT>(row0, 0, kgx) * static_cast<int64_t>(sizeof(XT));
            Q = Xc + tix<XT>(col0, 0, kgx) * static_cast<int64_t>(sizeof(XT));
          },
          [](int, int) { return 0.f; },
          [&](int row, int col, float v, float) { put<XT>(Am, tix<XT>(row, col, kgs), sa_ * v); });
      ++nbar;
      group_barrier(sync, nbar * sa.G, local);
      // B = b A + c A A (A symmetric: column block c of A is row block c)
      small_units<XT>(
          4 * na, sa.Sx / KG,
          [&](int u, const char*& P, const char*& Q, int& row0, int& col0) {
            row0 = bi * 32 + 16 * ((u & 3) >> 1);
            col0 = (bj + (u >> 2) * sa.CB) * 32 + 16 * (u & 1);
            P = Am + tix<XT>(row0, 0, kgs) * static_cast<int64_t>(sizeof(XT));
            Q = Am + tix<XT>(col0, 0, kgs) * static_cast<int64_t>(sizeof(XT));
          },
          [&](int row, int col) { return get<XT>(Am, tix<XT>(row, col, kgs)); },
          [&](int row, int col, float v, float a_) { put<XT>(Bm, tix<XT>(row, col, kgs), fmaf(cb, a_, cc * v)); });
      if (sa.CB > 1) {
        ++nbar;
        group_barrier(sync, nbar * sa.G, local);
      }
      // X' = a X + B X: rows bi, column blocks bj, bj + CB, .. of X
      const bool last = k + 1 == sa.K;
      char* Xn = sa.X[cur ^ 1] + m * sa.matX;
      char* XTn = sa.XT[cur ^ 1] + m * sa.matX;
      const int nx = (ncb - bj + sa.CB - 1) / sa.CB;
      small_units<XT>(
          4 * nx, sa.Sx / KG,
          [&](int u, const char*& P, const char*& Q, int& row0, int& col0) {
            row0 = bi * 32 + 16 * ((u & 3) >> 1);
            col0 = (bj + (u >> 2) * sa.CB) * 32 + 16 * (u & 1);
            P = Bm + tix<XT>(row0, 0, kgs) * static_cast<int64_t>(sizeof(XT));
            Q = XTc + tix<XT>(col0, 0, kgs) * static_cast<int64_t>(sizeof(XT));
          },
          [&](int row, int col) { return get<XT>(Xc, tix<XT>(row, col, kgx)); },
          [&](int xr, int xc, float v, float x_) {
            const float o = sx_ * fmaf(ca, x_, v);
            if (!last) {
              put<XT>(Xn, tix<XT>(xr, xc, kgx), o);
              put<XT>(XTn, tix<XT>(xc, xr, kgs), o);
            } else if (xr < sa.s && xc < sa.l) {
              const int64_t pidx = view_index(md, tr ? xc : xr, tr ? xr : xc);
              if (sa.sc.final_kind == 0)
                store_from_f32(md.W, pidx, sa.param_dtype,
                               fmaf(md.decay, load_as_f32(md.W, pidx, sa.param_dtype), -md.upd_scale * o));
              else
                store_from_f32(md.out, pidx, sa.param_dtype, o);
            }
          });
      if (!last) {
        ++nbar;
        group_barrier(sync, nbar * sa.G, local);
      }
      cur ^= 1;
    }
  }
}

// ---------------------------------------------------------------------------
// Newton-Schulz for short sides up to 128 (k_slice_*).  The tile kernel
// has one Gram tile per such matrix (64 slabs of k on one compute unit for
// 128 x 4096) and half-empty update tiles; here X is cut into column slices
// of 64 KB, one per workgroup, and a step is two launches over all matrices:
//   k_slice_reduce  A = sum of the slices' Gram partials (fp32, in slice
//                   order; r^2 on the first step), stored whole in the
//                   iterate's type;
//   k_slice_step    per slice: B = b A + c A A (up to 32 KB of A in bf16, 64 in
//                   fp32: cheaper to form
//                   in each workgroup than to launch for), X' = a X + B X in
//                   LDS, X' to memory, and the Gram partial of X'; the last
//                   step writes the parameter (or output) instead.
// k_slice_first does the prologue (momentum, u, its square sum) and the first
// Gram partial while the slice is in LDS.  The slice width is a function of
// the short side, the precision and the step alone, so results do not depend on
// the batch.
// What bounds it: the launches (about 4 us each, 2 K + 2 of them) for a few
// matrices, HBM and L2 traffic of the slices for many.
//
// RB: 32-row blocks of the padded short side (1, 2 or 4).  A wavefront owns 128 /
// RB columns of its slice in the update.  bf16 slices have 8 wavefronts (1024 /
// RB columns, 64 KB), in the last step 4 (32 KB); fp32 ones always 4 (512 / RB
// columns, 64 KB): SliceCfg.  LDS row r of a slice holds 16-byte chunk c at position
// c ^ key(r), key(r) = 4 (r % 4) + (r / 4) % 4: the transposing reads of
// 32 columns x 4 rows, the fragment reads of 32 rows x 16 bytes and the 8-byte
// accesses of 32 rows all spread over the banks.
// ---------------------------------------------------------------------------
struct SliceArgs {
  const MatDesc* desc;
  StepScalars sc;
  int32_t s, l, L;
  int32_t nsl, np;           // slices and Gram partials per matrix
  int32_t nmat;
  int32_t nnorm;             // slices of the prologue (square sums) per matrix
  int32_t first;
  void* X;                   // per matrix: S x L (matX elements), rows of stride L
  int64_t matX;
  float* part;               // per matrix: np x NB x 1024, MFMA output order
  void* A;                   // per matrix: Sx x Sx
  double* norm;              // per matrix: nsl
  float a, b, c;
};

// XT: the iterate's type, bfloat16 or fp32 (whose products are fp32 MFMA).
// NW: wavefronts of the workgroup: 8 for bf16, or 4 in its last step, whose
// slices are half as wide (no Gram partial depends on them), so that two
// workgroups fit a compute unit and one computes while the other waits for W;
// 4 for fp32, whose A takes the other 64 KB of the LDS.
template <typename XT, int RB, int NW>
struct SliceCfg {
  static constexpr int ES = sizeof(XT), EPC = 16 / ES;               // bytes an element, elements a 16-byte chunk
  static constexpr int Sx = 32 * RB, SW = 128 / RB;                  // SW: columns of a wavefront
  static constexpr int W = NW * SW, PITCH = ES * W;                  // PITCH: bytes of a slice row
  static constexpr int NB = RB * (RB + 1) / 2;                       // upper 32 x 32 blocks of A
  static constexpr int AP = ES * Sx, ABYTES = Sx * AP;               // A row, A
  static constexpr bool KSPLIT = RB < 4;  // Gram: each wavefront its own columns (a partial each), else output blocks
  static constexpr int PPS = KSPLIT ? NW : 1;                        // partials of a full slice
};
template <typename XT> constexpr int kSliceWaves = sizeof(XT) == 2 ? 8 : 4;
__device__ __forceinline__ int slice_key(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
// LDS byte of column col (in elements) of slice row r
template <class C>
__device__ __forceinline__ int slice_at(int r, int col) {
  return r * C::PITCH + (((col / C::EPC) ^ slice_key(r)) << 4) + (col % C::EPC) * C::ES;
}
// LDS byte of element (r, c) of A or B
template <class C>
__device__ __forceinline__ int slice_a_at(int r, int c) {
  return r * C::AP + (((c / C::EPC) ^ (slice_key(r) & (C::AP / 16 - 1))) << 4) + (c % C::EPC) * C::ES;
}
template <typename XT> struct Four { using T = uint2; };
template <> struct Four<float> { using T = float4; };
__device__ __forceinline__ void get4(const uint2& t, float v[4]) { unpack_bf16x4(t, v); }
__device__ __forceinline__ void get4(const float4& t, float v[4]) { v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w; }
__device__ __forceinline__ void set4(uint2& t, const float v[4]) { t = pack_bf16x4(v); }
__device__ __forceinline__ void set4(float4& t, const float v[4]) { t = make_float4(v[0], v[1], v[2], v[3]); }

// Workgroup b's matrix and slice.  Workgroup b runs on XCD b % 8: from 8
// matrices on, a matrix's slices share an XCD, whose L2 then holds its A once,
// and that XCD sees every column range (dealt out one by one, XCD x would see
// columns of the slices x, x + 8, .. only, which at power-of-two row strides
// are few of its L2 channels).  With fewer, a matrix's slices spread over all.
__device__ __forceinline__ bool slice_of(const SliceArgs& sa, int& m, int& j) {
  const int b = blockIdx.x;
  if (sa.nmat < 8) {
    m = b / sa.nsl;
    j = b - m * sa.nsl;
    return true;
  }
  const int q = b >> 3, mq = q / sa.nsl;
  m = mq * 8 + (b & 7);
  j = q - mq * sa.nsl;
  return m < sa.nmat;
}

// r = 1 / (||u|| + eps) from a matrix's slice sums, by all 256 or 512 threads
// of the workgroup in a fixed order (red: one double per wavefront).
__device__ __forceinline__ double slice_r(const double* norm, int n, float eps, double* red) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 256)
    if (threadIdx.x < 256) v += norm[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0 && threadIdx.x < 256) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double s = ((red[0] + red[1]) + red[2]) + red[3];
  return 1.0 / (sqrt(s) + static_cast<double>(eps));
}
// The first step's scale: r itself where r^2 u u^T stays well inside the fp32
// range, else 1 (X then holds r u, see k_slice_first<RESCALE>).
__device__ __forceinline__ bool slice_folds(double r) { return r >= 0x1p-40 && r <= 0x1p40; }

// fp32 products of k in kSums interleaved sums, added at the end: one chain of
// 64 additions (k = 128) left up to 1.7 times the error of the fused launch,
// which keeps two of 16 each.
constexpr int kSums = 4;
__device__ __forceinline__ f32x16_t add_sums(const f32x16_t p[kSums]) { return (p[0] + p[1]) + (p[2] + p[3]); }
// Mma<XT>::run into one sum (bf16) or its four interleaved ones (fp32).
template <typename XT>
__device__ __forceinline__ void mma_sums(const u32x4_t& a, const u32x4_t& b, f32x16_t* p) {
  if constexpr (sizeof(XT) == 2) {
    Mma<XT>::run(a, b, p[0]);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      p[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[j]), __uint_as_float(b[j]), p[j], 0, 0, 0);
  }
}
template <typename XT>
__device__ __forceinline__ f32x16_t all_sums(const f32x16_t* p) {
  if constexpr (sizeof(XT) == 2) return p[0];
  else return add_sums(p);
}

// The Gram partial(s) of the slice in LDS (nv columns, a multiple of 128).
// One fragment pair is 16 (bf16) or 8 (fp32) columns.
template <typename XT, class C, int NW>
__device__ __forceinline__ void slice_gram(const char* xs, int nv, float* part) {
  constexpr int RB = C::Sx / 32, KC = 32 / C::ES, NS = sizeof(XT) == 2 ? 1 : kSums;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto frag = [&](int rb, int col) {
    return *reinterpret_cast<const u32x4_t*>(xs + slice_at<C>(32 * rb + (lane & 31), col + C::EPC * (lane >> 5)));
  };
  auto put = [&](float* p, const f32x16_t& v) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(p + g * 256 + lane * 4) = make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
  };
  if constexpr (C::KSPLIT) {
    const int c0 = wave * C::SW;
    if (c0 >= nv) return;
    f32x16_t acc[C::NB][NS] = {};
#pragma unroll
    for (int g = 0; g < C::SW / KC; ++g) {
      u32x4_t f[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) f[i] = frag(i, c0 + KC * g);
#pragma unroll
      for (int j = 0; j < RB; ++j)
#pragma unroll
        for (int i = 0; i <= j; ++i) mma_sums<XT>(f[i], f[j], acc[j * (j + 1) / 2 + i]);
    }
    float* p = part + static_cast<int64_t>(wave) * C::NB * 1024;
#pragma unroll
    for (int n = 0; n < C::NB; ++n) put(p + n * 1024, all_sums<XT>(acc[n]));
  } else if constexpr (NW == 8) {
    // wavefront (wm, wn): row blocks 2 wm and 2 wm + 1 of column block wn, those on or above the diagonal
    const int wm = wave >> 2, wn = wave & 3;
    if (2 * wm > wn) return;
    const bool two = 2 * wm + 1 <= wn;
    f32x16_t acc[2][NS] = {};
    for (int g = 0; g < nv / KC; ++g) {
      const u32x4_t q = frag(wn, KC * g);
      mma_sums<XT>(frag(2 * wm, KC * g), q, acc[0]);
      if (two) mma_sums<XT>(frag(2 * wm + 1, KC * g), q, acc[1]);
    }
    float* p = part + (wn * (wn + 1) / 2 + 2 * wm) * 1024;
    put(p, all_sums<XT>(acc[0]));
    if (two) put(p + 1024, all_sums<XT>(acc[1]));
  } else {
    // the 10 upper blocks dealt to 4 wavefronts: blocks wave, wave + 4, wave + 8
    static_assert(RB == 4 && NW == 4, "block split");
    f32x16_t acc[3][NS] = {};
    int bi[3], bj[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int n = min(wave + 4 * t, C::NB - 1);
      bj[t] = n >= 6 ? 3 : n >= 3 ? 2 : n >= 1 ? 1 : 0;
      bi[t] = n - bj[t] * (bj[t] + 1) / 2;
    }
    const bool third = wave + 8 < C::NB;
    for (int g = 0; g < nv / KC; ++g) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < 2 || third) mma_sums<XT>(frag(bi[t], KC * g), frag(bj[t], KC * g), acc[t]);
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (t < 2 || third) put(part + (wave + 4 * t) * 1024, all_sums<XT>(acc[t]));
  }
}

// The slice in LDS -> memory, 16 bytes a thread.
template <typename XT, class C, int NW>
__device__ __forceinline__ void slice_store(const char* xs, int nv, XT* X, int L) {
  constexpr int CPR = C::W / C::EPC;
  for (int i = threadIdx.x; i < C::Sx * CPR; i += 64 * NW) {
    const int r = i / CPR, col = i % CPR * C::EPC;
    if (col >= nv) continue;
    *reinterpret_cast<u32x4_t*>(X + static_cast<int64_t>(r) * L + col) =
        *reinterpret_cast<const u32x4_t*>(xs + slice_at<C>(r, col));
  }
}

// Prologue: momentum in place, u (zero outside the matrix) into LDS
// and X, its square sum, the first Gram partial.  RESCALE: the matrices whose
// r cannot be applied to the products get X0 = r u and its Gram partial
// instead (the momentum is already advanced); all others return at once.
template <typename GT, typename XT, int RB, bool MOM, bool RESCALE>
__global__ __launch_bounds__(64 * kSliceWaves<XT>) void k_slice_first(SliceArgs sa) {
  constexpr int NW = kSliceWaves<XT>;
  using C = SliceCfg<XT, RB, NW>;
  __shared__ __attribute__((aligned(16))) char xs[C::Sx * C::PITCH];
  __shared__ double red[8];
  int m, j;
  if (!slice_of(sa, m, j)) return;
  const int c0 = j * C::W, nv = min(C::W, sa.L - c0);
  float s1 = 1.f, s2 = 1.f;
  if (RESCALE) {
    const double r = slice_r(sa.norm + static_cast<int64_t>(m) * sa.nnorm, sa.nnorm, sa.sc.eps, red);
    if (slice_folds(r)) return;
    split_scale(r, s1, s2);
  }
  const MatDesc md = sa.desc[m];
  const bool tr = md.transposed != 0;
  const GT* g = static_cast<const GT*>(md.g);
  const float beta = sa.sc.beta, omb = sa.sc.one_minus_beta;
  double acc = 0.0;
  // units of 8 consecutive elements of a row of u: 8 columns of X (u s x l), or
  // 8 rows of X (u l x s)
  const int upr = tr ? C::Sx / 8 : nv / 8;                 // units per row of u
  const int nu = tr ? nv * upr : C::Sx * upr;
  for (int i = threadIdx.x; i < nu; i += 64 * NW) {
    const int a = i / upr, e = (i - a * upr) * 8;
    const int ur = tr ? c0 + a : a, uc = tr ? e : c0 + e;
    float v[8];
    if (md.row8_ok && ur < md.rows && uc + 8 <= md.cols) {
      float gv[8], bv[8];
      load8(g, view_index(md, ur, uc), gv);
      if (MOM) {
        const int64_t ib = buf_index(md, ur, uc);
        load8(md.buf, ib, bv);
        if (!RESCALE) {
#pragma unroll
          for (int q = 0; q < 8; ++q) bv[q] = fmaf(beta, bv[q], omb * gv[q]);
          store8(md.buf, ib, bv);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = sa.sc.nesterov ? fmaf(beta, bv[q], omb * gv[q]) : bv[q];
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = gv[q];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        acc = fma(static_cast<double>(v[q]), static_cast<double>(v[q]), acc);
        v[q] = (v[q] * s1) * s2;
      }
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        v[q] = 0.f;  // padding stays exactly zero, whatever the scale
        if (ur < md.rows && uc + q < md.cols) {
          const float gv = to_f32<GT>(g[view_index(md, ur, uc + q)]);
          v[q] = gv;
          if (MOM) {
            const int64_t ib = buf_index(md, ur, uc + q);
            float bn = md.buf[ib];
            if (!RESCALE) {
              bn = fmaf(beta, bn, omb * gv);
              md.buf[ib] = bn;
            }
            v[q] = sa.sc.nesterov ? fmaf(beta, bn, omb * gv) : bn;
          }
          acc = fma(static_cast<double>(v[q]), static_cast<double>(v[q]), acc);
          v[q] = (v[q] * s1) * s2;
        }
      }
    }
    if (tr) {
#pragma unroll
      for (int q = 0; q < 8; ++q) *reinterpret_cast<XT*>(xs + slice_at<C>(e + q, a)) = from_f32<XT>(v[q]);
    } else {
#pragma unroll
      for (int h = 0; h < 8; h += C::EPC) {
        XT* p = reinterpret_cast<XT*>(xs + slice_at<C>(a, e + h));
        if constexpr (C::EPC == 8) store8(p, 0, v);
        else *reinterpret_cast<float4*>(p) = make_float4(v[h], v[h + 1], v[h + 2], v[h + 3]);
      }
    }
  }
  if (!RESCALE) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  }
  __syncthreads();
  if (!RESCALE && threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += red[w];
    sa.norm[static_cast<int64_t>(m) * sa.nnorm + j] = t;
  }
  slice_store<XT, C, NW>(xs, nv, static_cast<XT*>(sa.X) + m * sa.matX + c0, sa.L);
  slice_gram<XT, C, NW>(xs, nv, sa.part + (static_cast<int64_t>(m) * sa.np + j * C::PPS) * (C::NB * 1024));
}

// A = sum of the partials (times r^2 on the first step), one 32 x 32 block
// per workgroup, written on both sides of the diagonal.
template <typename XT, int RB>
__global__ __launch_bounds__(256) void k_slice_reduce(SliceArgs sa) {
  using C = SliceCfg<XT, RB, kSliceWaves<XT>>;
  __shared__ double red[4];
  const int m = blockIdx.x / C::NB, nb = blockIdx.x % C::NB;
  float scale = 1.f;
  if (sa.first) {
    const double r = slice_r(sa.norm + static_cast<int64_t>(m) * sa.nnorm, sa.nnorm, sa.sc.eps, red);
    const float rf = slice_folds(r) ? static_cast<float>(r) : 1.f;
    scale = rf * rf;
  }
  constexpr int64_t PS = C::NB * 1024;
  const float* p = sa.part + static_cast<int64_t>(m) * sa.np * PS + nb * 1024 + threadIdx.x * 4;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < sa.np; i += 8) {
    float4 t[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (i + q < sa.np) t[q] = *reinterpret_cast<const float4*>(p + (i + q) * PS);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (i + q < sa.np) {
        v[0] += t[q].x; v[1] += t[q].y; v[2] += t[q].z; v[3] += t[q].w;
      }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] *= scale;
  int bj = 0;
  while ((bj + 1) * (bj + 2) / 2 <= nb) ++bj;
  const int bi = nb - bj * (bj + 1) / 2, lane = threadIdx.x & 63;
  const int row = 32 * bi + 8 * (threadIdx.x >> 6) + 4 * (lane >> 5), col = 32 * bj + (lane & 31);
  XT* A = static_cast<XT*>(sa.A) + static_cast<int64_t>(m) * C::Sx * C::Sx;
  using F4 = typename Four<XT>::T;
  F4 h;
  set4(h, v);
  *reinterpret_cast<F4*>(A + col * C::Sx + row) = h;
  if (bi != bj) {
#pragma unroll
    for (int q = 0; q < 4; ++q) A[(row + q) * C::Sx + col] = from_f32<XT>(v[q]);
  }
}

// FK: -1 a middle step; 0 the last, updating W; 1 the last, writing out (both
// of dtype PDT).
template <typename XT, int RB, int FK, int PDT>
__global__ __launch_bounds__(FK >= 0 ? 256 : 64 * kSliceWaves<XT>, sizeof(XT) == 2 ? 2 : 1)
void k_slice_step(SliceArgs sa) {
  constexpr bool FINAL = FK >= 0, BF = sizeof(XT) == 2;
  constexpr int NW = FINAL ? 4 : kSliceWaves<XT>;
  using C = SliceCfg<XT, RB, NW>;
  using F4 = typename Four<XT>::T;
  constexpr int XB = C::Sx * C::PITCH;                     // 8 KB a wavefront (fp32: 16)
  constexpr int OB = FINAL ? C::Sx * C::W * 4 : 0;         // O of the slice in fp32, over both
  __shared__ __attribute__((aligned(1024))) char smem[OB > XB + C::ABYTES ? OB : XB + C::ABYTES];
  __shared__ double red[4];
  char* const xs = smem;
  char* const as = smem + XB;
  int m, j;
  if (!slice_of(sa, m, j)) return;
  const int c0 = j * C::W, nv = min(C::W, sa.L - c0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds0 = lds_offset(smem);
  XT* const X = static_cast<XT*>(sa.X) + m * sa.matX + c0;
  const char* const Ag = static_cast<const char*>(sa.A) + static_cast<int64_t>(m) * C::ABYTES;
  float osc = 1.f;
  if (sa.first) {
    const double r = slice_r(sa.norm + static_cast<int64_t>(m) * sa.nnorm, sa.nnorm, sa.sc.eps, red);
    if (slice_folds(r)) osc = static_cast<float>(r);
  }
  // the last step: the slice's part of the matrix in the parameter's layout, 8
  // elements a thread and unit, and its W values, read ahead.  (96 matrices of
  // 128 x 4096: 80 us; 147 with the descriptor's fields read where they are
  // used, 216 with 4 elements a unit, 251 with W read where it is used.)
  using PT = typename std::conditional<PDT == DT_BF16, uint16_t, float>::type;
  constexpr int NU = FINAL ? C::Sx * C::W / 8 / (64 * NW) : 1;   // units per thread
  const MatDesc* md = FINAL ? sa.desc + m : nullptr;
  const bool tr = FINAL && md->transposed != 0;
  WView w{};
  if constexpr (FINAL) w = w_view<FK == 0 ? 0 : 1>(md);
  const int nx = min(C::W, sa.l - c0), wrows = tr ? nx : sa.s, wcols = tr ? sa.s : nx;
  const int ush = 31 - __builtin_clz((tr ? C::Sx : C::W) / 8);   // units per row: a power of two
  auto w_unit = [&](int t, int& r, int& c) {
    const int i = threadIdx.x + 64 * NW * t;
    r = i >> ush;
    c = (i & ((1 << ush) - 1)) * 8;
  };
  auto w_at = [&](int r, int c) { return tr ? w_index(w, c0 + r, c) : w_index(w, r, c0 + c); };
  Raw8<PT> wv[NU];
  auto read_w = [&]() __attribute__((always_inline)) {
    if constexpr (FK == 0) {
      if (!w.vec8) return;
#pragma unroll
      for (int t = 0; t < NU; ++t) {
        int r, c;
        w_unit(t, r, c);
        if (r < wrows && c + 8 <= wcols) wv[t] = read8<PT>(w, w_at(r, c));
      }
    }
  };
  // ---- A and the slice into LDS: 1 KB per wavefront instruction, lane i the
  // 16 bytes at 16 i; each lane fetches the chunk that belongs there ----------
  constexpr int ACH = C::AP / 16, AI = C::ABYTES / 1024;   // chunks of an A row; instructions
#pragma unroll
  for (int k = 0; k < (AI + NW - 1) / NW; ++k) {
    const int t = wave + NW * k;
    if (t < AI) {
      const int p = t * 64 + lane, r = p / ACH;
      load_lds16(Ag, static_cast<uint32_t>(r * C::AP + ((p % ACH) ^ (slice_key(r) & (ACH - 1))) * 16),
                 lds0 + XB + t * 1024);
    }
  }
  constexpr int XCH = C::PITCH / 16;                       // chunks of a slice row
  constexpr int XI = XB / 1024 / NW;                       // instructions of a wavefront
#pragma unroll
  for (int k = 0; k < XI; ++k) {
    const int t = wave + NW * k, p = t * 64 + lane, r = p / XCH;
    int ch = (p % XCH) ^ slice_key(r);
    if (C::EPC * ch >= nv) ch &= 8 * C::ES - 1;            // past the matrix: any chunk of the row (not used)
    load_lds16(reinterpret_cast<const char*>(X), static_cast<uint32_t>(r) * static_cast<uint32_t>(sa.L * C::ES) + ch * 16,
               lds0 + t * 1024);
  }
  if constexpr (FINAL) {
    read_w();                                              // in flight together with A and the slice
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(XI) : "memory");  // A has landed, the slice may not
  }
  __syncthreads();
  // ---- B = b A + c A A, in place --------------------------------------------
  constexpr int PB = RB == 4 ? 16 / NW : 1;                // 32 x 32 blocks of B per wavefront
  const int pi = RB == 4 ? PB * (wave >> 2) : wave / RB, pj = RB == 4 ? (wave & 3) : wave % RB;
  const bool pact = RB == 4 || wave < RB * RB;
  F4 bh[PB][4];
  if (pact) {
    f32x16_t acc[PB] = {};
    if constexpr (BF) {
      auto afrag = [&](int rb, int g) {
        return *reinterpret_cast<const u32x4_t*>(as + slice_a_at<C>(32 * rb + (lane & 31), 16 * g + 8 * (lane >> 5)));
      };
#pragma unroll
      for (int g = 0; g < C::Sx / 16; ++g) {
        const u32x4_t q = afrag(pj, g);
#pragma unroll
        for (int i = 0; i < PB; ++i) Mma<uint16_t>::run(afrag(pi + i, g), q, acc[i]);
      }
    } else {
      // A is symmetric: the operands' rows at k are row k of A
      f32x16_t part[PB][kSums] = {};
      for (int k0 = 0; k0 < C::Sx; k0 += 2 * kSums)
#pragma unroll
        for (int t = 0; t < kSums; ++t) {
          const int k = k0 + 2 * t + (lane >> 5);
          const float q = *reinterpret_cast<const float*>(as + slice_a_at<C>(k, 32 * pj + (lane & 31)));
#pragma unroll
          for (int i = 0; i < PB; ++i)
            part[i][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                *reinterpret_cast<const float*>(as + slice_a_at<C>(k, 32 * (pi + i) + (lane & 31))), q, part[i][t], 0, 0, 0);
        }
#pragma unroll
      for (int i = 0; i < PB; ++i) acc[i] = add_sums(part[i]);
    }
#pragma unroll
    for (int i = 0; i < PB; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        // rows row .. row + 3 of column col; A is symmetric, so they lie in row col
        const int row = 32 * (pi + i) + 8 * g + 4 * (lane >> 5), col = 32 * pj + (lane & 31);
        float e[4], v[4];
        get4(*reinterpret_cast<const F4*>(as + slice_a_at<C>(col, row)), e);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = fmaf(sa.b, e[q], sa.c * acc[i][4 * g + q]);
        set4(bh[i][g], v);
      }
  }
  __syncthreads();                                         // every read of A is done
  if (pact) {
#pragma unroll
    for (int i = 0; i < PB; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int row = 32 * (pi + i) + 8 * g + 4 * (lane >> 5), col = 32 * pj + (lane & 31);
        *reinterpret_cast<F4*>(as + slice_a_at<C>(col, row)) = bh[i][g];  // B is symmetric too
      }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the slice has landed
  __syncthreads();
  // ---- X'^T = a X^T + X^T B over the wavefront's columns: a lane gets 4
  // consecutive columns of one row ----------------------------------------------
  constexpr int CBW = C::SW / 32;                          // 32-column blocks of a wavefront
  const int w0 = wave * C::SW;
  f32x16_t acc[CBW][RB] = {};
  if (w0 < nv) {
    if constexpr (BF) {
      const int G = lane >> 4, Lq = lane & 15;
#pragma unroll
      for (int g = 0; g < C::Sx / 16; ++g) {
        u32x4_t bf[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i)
          bf[i] = *reinterpret_cast<const u32x4_t*>(as + slice_a_at<C>(32 * i + (lane & 31), 16 * g + 8 * (lane >> 5)));
#pragma unroll
        for (int k = 0; k < CBW; ++k) {
          const int row = 16 * g + 8 * (G >> 1) + (Lq >> 2), col = w0 + 32 * k + 16 * (G & 1) + 4 * (Lq & 3);
          const uint2 lo = tr_read_b64(xs + slice_at<C>(row, col)), hi = tr_read_b64(xs + slice_at<C>(row + 4, col));
          const u32x4_t xf{lo.x, lo.y, hi.x, hi.y};
#pragma unroll
          for (int i = 0; i < RB; ++i) Mma<uint16_t>::run(xf, bf[i], acc[k][i]);
        }
      }
    } else {
      // both operands take row k as it lies (B is symmetric): 32 consecutive floats
      f32x16_t part[CBW][RB][kSums] = {};
      for (int k0 = 0; k0 < C::Sx; k0 += 2 * kSums)
#pragma unroll
        for (int t = 0; t < kSums; ++t) {
          const int row = k0 + 2 * t + (lane >> 5);
          float bf[RB];
#pragma unroll
          for (int i = 0; i < RB; ++i)
            bf[i] = *reinterpret_cast<const float*>(as + slice_a_at<C>(row, 32 * i + (lane & 31)));
#pragma unroll
          for (int k = 0; k < CBW; ++k) {
            const float xf = *reinterpret_cast<const float*>(xs + slice_at<C>(row, w0 + 32 * k + (lane & 31)));
#pragma unroll
            for (int i = 0; i < RB; ++i)
              part[k][i][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(xf, bf[i], part[k][i][t], 0, 0, 0);
          }
        }
#pragma unroll
      for (int k = 0; k < CBW; ++k)
#pragma unroll
        for (int i = 0; i < RB; ++i) acc[k][i] = add_sums(part[k][i]);
    }
#pragma unroll
    for (int k = 0; k < CBW; ++k)
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int row = 32 * i + (lane & 31), col = w0 + 32 * k + 8 * g + 4 * (lane >> 5);
          F4* p = reinterpret_cast<F4*>(xs + slice_at<C>(row, col));
          float e[4], v[4];
          get4(*p, e);
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = osc * fmaf(sa.a, e[q], acc[k][i][4 * g + q]);
          if constexpr (FINAL) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[k][i][4 * g + q] = v[q];
          } else {
            set4(*p, v);
          }
        }
  }
  __syncthreads();
  if constexpr (!FINAL) {
    slice_store<XT, C, NW>(xs, nv, X, sa.L);
    slice_gram<XT, C, NW>(xs, nv, sa.part + (static_cast<int64_t>(m) * sa.np + j * C::PPS) * (C::NB * 1024));
  } else {
    // ---- the parameter (or output): O in fp32 through LDS in the parameter's
    // layout, whole rows back --------------------------------------------------------
    float* const os = reinterpret_cast<float*>(smem);
    // row-major [Sx][W], 16-byte chunk ch of row r at ch ^ (r % 16); or [W][Sx] (parameter l x s)
    auto oat = [](int r, int c) { return r * C::W + ((((c >> 2) ^ (r & 15)) << 2) | (c & 3)); };
    if (w0 < nv) {
#pragma unroll
      for (int k = 0; k < CBW; ++k)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int row = 32 * i + (lane & 31), col = w0 + 32 * k + 8 * g + 4 * (lane >> 5);
            const f32x16_t& o = acc[k][i];
            if (tr) {
#pragma unroll
              for (int q = 0; q < 4; ++q) os[(col + q) * C::Sx + row] = o[4 * g + q];
            } else {
              *reinterpret_cast<float4*>(os + oat(row, col)) =
                  make_float4(o[4 * g], o[4 * g + 1], o[4 * g + 2], o[4 * g + 3]);
            }
          }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NU; ++t) {
      int r, c;
      w_unit(t, r, c);
      const int n = min(8, wcols - c);
      if (r >= wrows || n <= 0) continue;
      float o[8];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4 ov = *reinterpret_cast<const float4*>(os + (tr ? r * C::Sx + c + 4 * h : oat(r, c + 4 * h)));
        o[4 * h] = ov.x; o[4 * h + 1] = ov.y; o[4 * h + 2] = ov.z; o[4 * h + 3] = ov.w;
      }
      apply8<FK == 0 ? 0 : 1, PT>(w, w_at(r, c), o, n, wv[t]);
    }
  }
}

template <typename GT, typename XT, int RB>
hipError_t run_slices(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb, const StepScalars& sc,
                      const float* coeffs, int K, hipStream_t st, double& exec) {
  constexpr int NW = kSliceWaves<XT>;
  using C = SliceCfg<XT, RB, NW>;
  using CF = SliceCfg<XT, RB, 4>;                          // the last step's slices
  SliceArgs sa{};
  sa.desc = d_desc;
  sa.sc = sc;
  sa.s = cg.s; sa.l = cg.l; sa.L = cg.L;
  sa.nsl = (cg.L + C::W - 1) / C::W;
  sa.nnorm = sa.nsl;
  sa.np = C::KSPLIT ? cg.L / C::SW : sa.nsl;
  sa.X = wb.X[0];
  sa.matX = static_cast<int64_t>(cg.S) * cg.L;
  sa.part = static_cast<float*>(wb.X[1]);                  // over X[1], XT[0] and XT[1]
  sa.A = wb.A;
  sa.norm = wb.partials;
  sa.nmat = cg.nmat;
  const unsigned mats = cg.nmat < 8 ? cg.nmat : (cg.nmat + 7) / 8 * 8;
  const dim3 slices(static_cast<unsigned>(sa.nsl) * mats);
  const dim3 blocks(static_cast<unsigned>(C::NB) * static_cast<unsigned>(cg.nmat));
  if (sc.momentum) {
    hipLaunchKernelGGL((k_slice_first<GT, XT, RB, true, false>), slices, dim3(64 * NW), 0, st, sa);
    hipLaunchKernelGGL((k_slice_first<GT, XT, RB, true, true>), slices, dim3(64 * NW), 0, st, sa);
  } else {
    hipLaunchKernelGGL((k_slice_first<GT, XT, RB, false, false>), slices, dim3(64 * NW), 0, st, sa);
    hipLaunchKernelGGL((k_slice_first<GT, XT, RB, false, true>), slices, dim3(64 * NW), 0, st, sa);
  }
  for (int k = 0; k < K; ++k) {
    sa.first = k == 0 ? 1 : 0;
    sa.a = coeffs[3 * k]; sa.b = coeffs[3 * k + 1]; sa.c = coeffs[3 * k + 2];
    hipLaunchKernelGGL((k_slice_reduce<XT, RB>), blocks, dim3(256), 0, st, sa);
    if (k + 1 < K) hipLaunchKernelGGL((k_slice_step<XT, RB, -1, DT_BF16>), slices, dim3(64 * NW), 0, st, sa);
  }
  // what the MFMAs execute: per step the upper blocks of A and X' over all
  // columns, and B in every slice
  const int nlast = (cg.L + CF::W - 1) / CF::W;
  const double Sx = C::Sx, Lp = cg.L;
  exec = double(cg.nmat) * (K * 2.0 * Lp * (C::NB * 1024.0 + Sx * Sx) + 2.0 * Sx * Sx * Sx * ((K - 1.0) * sa.nsl + nlast));
  const bool o = sc.final_kind != 0, f32 = cg.param_dtype == DT_F32;
  sa.nsl = nlast;
  const dim3 halves(static_cast<unsigned>(sa.nsl) * mats);
  if (!o && !f32) hipLaunchKernelGGL((k_slice_step<XT, RB, 0, DT_BF16>), halves, dim3(256), 0, st, sa);
  else if (!o) hipLaunchKernelGGL((k_slice_step<XT, RB, 0, DT_F32>), halves, dim3(256), 0, st, sa);
  else if (!f32) hipLaunchKernelGGL((k_slice_step<XT, RB, 1, DT_BF16>), halves, dim3(256), 0, st, sa);
  else hipLaunchKernelGGL((k_slice_step<XT, RB, 1, DT_F32>), halves, dim3(256), 0, st, sa);
  return hipGetLastError();
}

template <typename GT, typename XT>
hipError_t run_sliced_chunk(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb, const StepScalars& sc,
                            const float* coeffs, int K, hipStream_t st, LaunchTimer* timer) {
  Timed tm(timer, KK_SMALL, st);
  const int Sx = cg.s <= 32 ? 32 : cg.s <= 64 ? 64 : 128;
  double exec = 0.0;
  const hipError_t e = Sx == 32   ? run_slices<GT, XT, 1>(cg, d_desc, wb, sc, coeffs, K, st, exec)
                       : Sx == 64 ? run_slices<GT, XT, 2>(cg, d_desc, wb, sc, coeffs, K, st, exec)
                                  : run_slices<GT, XT, 4>(cg, d_desc, wb, sc, coeffs, K, st, exec);
  if (e != hipSuccess) return e;
  const double nm = cg.nmat, s = cg.s, l = cg.l;
  const double gsz = sizeof(GT), psz = cg.param_dtype == DT_BF16 ? 2.0 : 4.0;
  tm.done(nm * K * (4.0 * s * s * l + 2.0 * s * s * s), exec,
          nm * s * l * (gsz + (sc.momentum ? 8.0 : 0.0) + (sc.final_kind == 0 ? 2.0 * psz : psz)));
  return hipSuccess;
}

// Zeroes n words (the group counters before a fused launch).
__global__ __launch_bounds__(256) void k_zero_words(unsigned* p, int n) {
  for (int i = threadIdx.x; i < n; i += 256) p[i] = 0u;
}

template <typename GT, typename XT>
hipError_t run_small(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb, const StepScalars& sc,
                     const float* coeffs, int K, hipStream_t st, LaunchTimer* timer) {
  SmallArgs sa{};
  sa.desc = d_desc;
  sa.sc = sc;
  sa.s = cg.s; sa.l = cg.l; sa.S = cg.S; sa.L = cg.L;
  sa.Sx = (cg.s + 31) / 32 * 32;
  sa.Lx = (cg.l + 31) / 32 * 32;
  sa.nmat = cg.nmat;
  sa.RB = sa.Sx / 32;
  const int cus = device_cu_count();
  // column groups: 4, or as many as there are 32-column blocks of X.  A
  // function of the shape alone, so that the order of every sum, and with
  // it each matrix's result, does not depend on the other matrices of the call.
  sa.CB = min(4, sa.Lx / 32);
  sa.G = sa.RB * sa.CB;
  // groups: 8 per round (one per XCD), as many rounds as fit one workgroup per CU
  const int rounds = max(1, min((cg.nmat + 7) / 8, cus / (8 * sa.G)));
  sa.groups = 8 * rounds;
  sa.K = K;
  sa.param_dtype = cg.param_dtype;
  sa.X[0] = static_cast<char*>(wb.X[0]); sa.X[1] = static_cast<char*>(wb.X[1]);
  sa.XT[0] = static_cast<char*>(wb.XT[0]); sa.XT[1] = static_cast<char*>(wb.XT[1]);
  sa.A = static_cast<char*>(wb.A); sa.B = static_cast<char*>(wb.B);
  sa.matX = static_cast<int64_t>(cg.S) * cg.L * sizeof(XT);
  sa.matA = static_cast<int64_t>(cg.S) * cg.S * sizeof(XT);
  sa.partials = wb.partials;
  sa.sync = wb.sync;
  for (int i = 0; i < 3 * K; ++i) sa.coeffs[i] = coeffs[i];
  Timed tm(timer, KK_SMALL, st);
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(256), 0, st, wb.sync, sa.groups * 64);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid(static_cast<unsigned>(sa.groups * sa.G));
  if (sc.momentum)
    hipLaunchKernelGGL((k_ns_small<GT, XT, true>), grid, dim3(256), 0, st, sa);
  else
    hipLaunchKernelGGL((k_ns_small<GT, XT, false>), grid, dim3(256), 0, st, sa);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const double nm = cg.nmat, s = cg.s, l = cg.l, Sx = sa.Sx, Lx = sa.Lx;
  const double gsz = sizeof(GT), psz = cg.param_dtype == DT_BF16 ? 2.0 : 4.0;
  tm.done(nm * K * (4.0 * s * s * l + 2.0 * s * s * s), nm * K * (4.0 * Sx * Sx * Lx + 2.0 * Sx * Sx * Sx),
          nm * s * l * (gsz + (sc.momentum ? 8.0 : 0.0) + (sc.final_kind == 0 ? 2.0 * psz : psz)));
  return hipSuccess;
}

// Whether a chunk stored as XT runs its products on the tile kernel.
template <typename XT>
bool runs_on_tiles(const ChunkGeom& cg, int K) {
  if (std::is_same<XT, Split3>::value) return true;
  return !std::is_same<XT, float>::value && chunk_on_tiles(cg.S, cg.L, K);
}

template <typename GT, typename XT>
hipError_t run_prologue_t(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb,
                       const StepScalars& sc, const float* coeffs, int K, hipStream_t st,
                       LaunchTimer* timer) {
  const int nmat = cg.nmat;
  const double nm = nmat;
  const int64_t numel = static_cast<int64_t>(cg.s) * cg.l;
  const double ne = double(numel);
  const int nparts = static_cast<int>(norm_tiles(cg.S, cg.L));
  using E = typename Store<XT>::E;
  const double gsz = sizeof(GT), xsz = sizeof(E) * Store<XT>::planes;
  const double psz = cg.param_dtype == DT_BF16 ? 2.0 : 4.0;
  // On the tile kernel the update products read X through transposing
  // LDS reads, so no X^T is kept (K = 0 applies X0 from whichever layout
  // matches the parameter).
  const bool qtr = runs_on_tiles<XT>(cg, K);
  E* const xt0 = qtr ? nullptr : static_cast<E*>(wb.XT[0]);
  hipError_t e;
  E* const x0 = static_cast<E*>(wb.X[0]);
  {
    Timed tm(timer, KK_PARTIALS, st);
    const dim3 grid(cg.L / 64, cg.S / 64, nmat);
    if (sc.momentum)
      hipLaunchKernelGGL((k_prologue<GT, XT, true>), grid, dim3(256), 0, st, d_desc, sc, cg, x0, xt0, wb.partials);
    else
      hipLaunchKernelGGL((k_prologue<GT, XT, false>), grid, dim3(256), 0, st, d_desc, sc, cg, x0, xt0, wb.partials);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // reads g (and the momentum), writes the momentum and X~ (and X~^T)
    tm.done(0, 0, nm * ne * (gsz + (sc.momentum ? 8.0 : 0.0) + (qtr ? 1.0 : 2.0) * xsz) + nm * nparts * 8.0);
  }
  {
    Timed tm(timer, KK_FINALIZE, st);
    hipLaunchKernelGGL(k_finalize, dim3(nmat), dim3(1024), 0, st, wb.partials, nparts, sc.eps,
                       std::is_same<XT, Split3>::value ? 1 : 0, wb.rscale, wb.xscale);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    tm.done(0, 0, nm * nparts * 8.0 + nm * 12.0);
  }
  {
    Timed tm(timer, KK_NORMALIZE, st);
    const dim3 grid(64, nmat);
    if (sc.momentum)
      hipLaunchKernelGGL((k_rescale<GT, XT, true>), grid, dim3(256), 0, st, d_desc, wb.rscale, sc, cg, x0, xt0);
    else
      hipLaunchKernelGGL((k_rescale<GT, XT, false>), grid, dim3(256), 0, st, d_desc, wb.rscale, sc, cg, x0,
                         xt0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    tm.done(0, 0, nm * 12.0);  // nothing else unless a norm is out of range
  }

  if constexpr (!std::is_same<XT, Split3>::value) if (K == 0) {
    Timed tm(timer, KK_APPLY_X0, st);
    const int64_t blocks = (numel + 255) / 256;
    hipLaunchKernelGGL((k_apply_x0<XT>), dim3(static_cast<unsigned>(blocks), nmat), dim3(256), 0, st,
                       d_desc, cg, static_cast<const XT*>(wb.X[0]), static_cast<const XT*>(wb.XT[0]),
                       wb.xscale, sc.final_kind);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    tm.done(0, 0, nm * ne * (xsz + (sc.final_kind == 0 ? 2.0 * psz : psz)));
    return hipSuccess;
  }
  return hipSuccess;
}

// The three products of Newton-Schulz step k of a chunk (after the
// prologue): their launch arguments and work accounting.  `cur` selects the
// iterate the step reads.
struct StepProducts {
  GemmArgs gram, poly, upd;
  bool last;              // upd is the last step's product (parameter update or O)
  double f[3], b[3];      // dense flops (Eq. 1, on the real extents) and bytes of gram, poly, upd
};

template <typename XT>
StepProducts step_products(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb,
                           const StepScalars& sc, const float* coeffs, int K, int k, int cur) {
  const bool qtr = runs_on_tiles<XT>(cg, K);
  const double nm = cg.nmat;
  const double s = cg.s, l = cg.l;
  constexpr int planes = Store<XT>::planes;
  const int es = static_cast<int>(sizeof(typename Store<XT>::E));
  const double xsz = es * planes;
  const double psz = cg.param_dtype == DT_BF16 ? 2.0 : 4.0;
  const int64_t planeX = static_cast<int64_t>(cg.S) * cg.L * es, matX = planeX * planes;
  const int64_t planeA = static_cast<int64_t>(cg.S) * cg.S * es, matA = planeA * planes;
  const int ts = cg.S / kTile, tl = cg.L / kTile;
  StepProducts r{};
  const float a = coeffs[3 * k], b = coeffs[3 * k + 1], c = coeffs[3 * k + 2];
  const char* X = static_cast<const char*>(wb.X[cur]);
  const char* XTc = static_cast<const char*>(wb.XT[cur]);
  // A = X X^T: M = N = S, K = L.
  GemmArgs& g = r.gram;
  GemmArgs& u = r.upd;
  g.P = X; g.p_mat = matX; g.ldp = cg.L * es;
  g.Q = X; g.q_mat = matX; g.ldq = cg.L * es;
  g.k_slabs = cg.L * es / 128;
  g.tiles_m = ts; g.tiles_n = ts; g.syrk = 1; g.tiles_per_mat = ts * (ts + 1) / 2;
  g.C = static_cast<char*>(wb.A); g.c_mat = matA; g.ldc = cg.S * es;
  g.p_plane = g.q_plane = planeX; g.c_plane = planeA;
  g.xscale = k == 0 ? wb.xscale : nullptr;  // A0 = r^2 X~ X~^T
  g.rscale = u.rscale = planes == 3 ? wb.rscale : nullptr;
  // Under qtr every consumer of A and B runs on the tile kernel and
  // reads them as upper-triangle tiles (mode 1): no mirrored tile is
  // written.  Otherwise the lower triangle is written as the mirror.
  if (!qtr) { g.CT = g.C; g.ct_mat = matA; g.ldct = g.ldc; }
  r.f[0] = nm * 2 * s * s * l; r.b[0] = nm * (s * l + s * s) * xsz;
  // B = b A + c A A^T: M = N = K = S.
  GemmArgs& pp = r.poly;
  pp = g;
  pp.xscale = nullptr;
  pp.P = static_cast<const char*>(wb.A); pp.p_mat = matA; pp.ldp = cg.S * es;
  pp.Q = pp.P; pp.q_mat = matA; pp.ldq = pp.ldp;
  pp.k_slabs = cg.S * es / 128;
  pp.E = pp.P; pp.e_mat = matA; pp.lde = pp.ldp;
  pp.C = static_cast<char*>(wb.B); pp.CT = qtr ? nullptr : pp.C;
  pp.p_mode = pp.q_mode = qtr ? 1 : 0;
  pp.p_plane = pp.q_plane = planeA;
  pp.alpha = b; pp.beta = c;
  r.f[1] = nm * 2 * s * s * s; r.b[1] = nm * 2 * s * s * xsz;
  // X' = a X + B X: M = S, N = L, K = S.  The second operand is X^T (N x K,
  // K contiguous) on the 128 x 128 kernel, X itself (K x N) under qtr.
  u.P = static_cast<const char*>(wb.B); u.p_mat = matA; u.ldp = cg.S * es;
  if (qtr) {
    u.Q = X; u.q_mat = matX; u.ldq = cg.L * es;
    u.p_mode = 1;  // B: upper-triangle tiles
    u.q_mode = 2;  // X: K x N
  } else {
    u.Q = XTc; u.q_mat = matX; u.ldq = cg.S * es;
  }
  u.p_plane = planeA; u.q_plane = u.c_plane = planeX;
  u.k_slabs = cg.S * es / 128;
  u.tiles_m = ts; u.tiles_n = tl; u.syrk = 0; u.tiles_per_mat = ts * tl;
  u.E = X; u.e_mat = matX; u.lde = cg.L * es;
  u.alpha = a;
  u.s = cg.s; u.l = cg.l;
  u.xscale = k == 0 ? wb.xscale : nullptr;  // X1 = r (a X~ + B0 X~)
  r.f[2] = nm * 2 * s * s * l;
  r.last = k + 1 == K;
  if (!r.last) {
    u.C = static_cast<char*>(wb.X[cur ^ 1]); u.c_mat = matX; u.ldc = cg.L * es;
    if (!qtr) { u.CT = static_cast<char*>(wb.XT[cur ^ 1]); u.ct_mat = matX; u.ldct = cg.S * es; }
    // reads B, X (twice under qtr, else X^T and X); writes X' (and X'^T)
    r.b[2] = nm * (s * s + (qtr ? 3 : 4) * s * l) * xsz;
  } else {
    u.desc = d_desc; u.final_kind = sc.final_kind; u.param_dtype = cg.param_dtype; u.w_rows16 = cg.w_rows16;
    // reads B, X^T, X (and W); writes W or out
    r.b[2] = nm * ((s * s + 2 * s * l) * xsz + s * l * (sc.final_kind == 0 ? 2 * psz : psz));
  }
  return r;
}

template <typename GT, typename XT>
hipError_t run_chunk_t(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb,
                       const StepScalars& sc, const float* coeffs, int K, hipStream_t st,
                       LaunchTimer* timer) {
  constexpr bool split = std::is_same<XT, Split3>::value;
  if constexpr (!split)
    if (wb.sync) return run_small<GT, XT>(cg, d_desc, wb, sc, coeffs, K, st, timer);
  hipError_t e = run_prologue_t<GT, XT>(cg, d_desc, wb, sc, coeffs, K, st, timer);
  if (e != hipSuccess || K == 0) return e;
  const bool qtr = runs_on_tiles<XT>(cg, K);
  const int nmat = cg.nmat;
  double exec = 0.0;
  auto launch = [&](int epi, const GemmArgs& ga) {
    if constexpr (!split)
      if (!qtr) return launch_gemm<XT>(epi, ga, nmat, st, exec);
    if constexpr (std::is_same<XT, float>::value)
      return hipErrorInvalidValue;
    else {
      const Tiles kind = tiles_of(ga, nmat, split);
      if (kind == Tiles::square) return launch_tile<CfgSquare, split>(epi, ga, nmat, st, exec);
      if constexpr (!split)
        if (kind == Tiles::deep) return launch_tile<CfgDeep, false>(epi, ga, nmat, st, exec);
      return launch_tile<CfgQuarter, split>(epi, ga, nmat, st, exec);
    }
  };
  int cur = 0;
  for (int k = 0; k < K; ++k) {
    const StepProducts sp = step_products<XT>(cg, d_desc, wb, sc, coeffs, K, k, cur);
    {
      Timed tm(timer, KK_GRAM, st);
      if ((e = launch(EPI_GRAM, sp.gram)) != hipSuccess) return e;
      tm.done(sp.f[0], exec, sp.b[0]);
    }
    {
      Timed tm(timer, KK_POLY, st);
      if ((e = launch(EPI_POLY, sp.poly)) != hipSuccess) return e;
      tm.done(sp.f[1], exec, sp.b[1]);
    }
    {
      const int epi = sp.last ? EPI_FINAL : EPI_UPDATE;
      Timed tm(timer, sp.last ? KK_FINAL : KK_UPDATE, st);
      if ((e = launch(epi, sp.upd)) != hipSuccess) return e;
      tm.done(sp.f[2], exec, sp.b[2]);
    }
    cur ^= 1;
  }
  return hipSuccess;
}

}  // namespace

hipError_t run_chunk(const ChunkGeom& cg, const MatDesc* d_desc, const ChunkBuffers& wb,
                     const StepScalars& sc, const float* coeffs, int K, hipStream_t st,
                     LaunchTimer* timer) {
  const bool gbf = cg.grad_dtype == DT_BF16;
  if (chunk_is_sliced(cg.s, cg.l, cg.ns_f32 != 0, K)) {
    if (cg.ns_f32)
      return gbf ? run_sliced_chunk<uint16_t, float>(cg, d_desc, wb, sc, coeffs, K, st, timer)
                 : run_sliced_chunk<float, float>(cg, d_desc, wb, sc, coeffs, K, st, timer);
    return gbf ? run_sliced_chunk<uint16_t, uint16_t>(cg, d_desc, wb, sc, coeffs, K, st, timer)
               : run_sliced_chunk<float, uint16_t>(cg, d_desc, wb, sc, coeffs, K, st, timer);
  }
  if (cg.ns_f32 && !wb.sync && chunk_on_tiles(cg.S, cg.L, K)) {
    return gbf ? run_chunk_t<uint16_t, Split3>(cg, d_desc, wb, sc, coeffs, K, st, timer)
               : run_chunk_t<float, Split3>(cg, d_desc, wb, sc, coeffs, K, st, timer);
  }
  if (cg.ns_f32) {
    return gbf ? run_chunk_t<uint16_t, float>(cg, d_desc, wb, sc, coeffs, K, st, timer)
               : run_chunk_t<float, float>(cg, d_desc, wb, sc, coeffs, K, st, timer);
  }
  return gbf ? run_chunk_t<uint16_t, uint16_t>(cg, d_desc, wb, sc, coeffs, K, st, timer)
             : run_chunk_t<float, uint16_t>(cg, d_desc, wb, sc, coeffs, K, st, timer);
}

// The kernels a chunk runs on alone, for the plan printed to stderr.
std::string route_of(const ChunkGeom& cg, int K) {
  const bool f32 = cg.ns_f32 != 0;
  if (chunk_is_small(cg.s, cg.l, f32, K)) return "fused";
  if (chunk_is_sliced(cg.s, cg.l, f32, K)) return "slices";
  if (!chunk_on_tiles(cg.S, cg.L, K)) return K == 0 ? "no products" : "long rows";
  const float coeffs[3] = {1.f, 1.f, 1.f};
  const StepProducts sp =
      f32 ? step_products<Split3>(cg, nullptr, ChunkBuffers{}, StepScalars{}, coeffs, 1, 0, 0)
          : step_products<uint16_t>(cg, nullptr, ChunkBuffers{}, StepScalars{}, coeffs, 1, 0, 0);
  std::string r = "tiles";
  for (const GemmArgs* ga : {&sp.gram, &sp.poly, &sp.upd}) {
    const Tiles kind = tiles_of(*ga, cg.nmat, f32);
    r += kind == Tiles::square ? " 256" : kind == Tiles::quarter ? " 128" : " 128x4";
  }
  return r;
}

bool group_eligible(const ChunkGeom& cg, int K) {
  return !cg.ns_f32 && K > 0 && cg.S % 256 == 0 && cg.L % 256 == 0 && tile_rows_fit(cg.S, cg.L, 2) &&
         !chunk_is_small(cg.s, cg.l, false, K) && !chunk_is_sliced(cg.s, cg.l, false, K);
}

// A group's launches run all members' tiles on 256 x 256 tiles: as one round
// while they fit (then as long as the longest takes), else as rounds of their
// mean.  Alone, a member's launches take the faster tile size.  On one stream,
// us per step call, grouped / alone / the model's ratio: 3 x 512^2 + 3 x 512 x
// 1536 + 2 x 768 x 1024 489 / 630 / 0.70; 4 x 2048^2 + 3 x 2048 x 5632 2284 /
// 2391 / 0.97; 4096^2 + 2 x 1024 x 4096 1690 / 1874 / 0.95; 4 x 1024^2 + 3 x 1024
// x 2816 691 / 668 / 1.06; 4 x 768^2 + 2 x 768 x 3072 643 / 575 / 1.06; 1024^2 +
// 1024 x 4096 725 / 609 / 1.18.
bool group_pays(const ChunkGeom* geoms, int n) {
  double grouped = 0.0, alone = 0.0;
  for (int q = 0; q < 3; ++q) {
    double tiles = 0.0, slabs_us = 0.0, longest = 0.0;
    GemmArgs ga[kMaxGroup];
    for (int c = 0; c < n; ++c) {
      const float coeffs[3] = {1.f, 1.f, 1.f};
      const StepProducts sp = step_products<uint16_t>(geoms[c], nullptr, ChunkBuffers{}, StepScalars{}, coeffs, 1, 0, 0);
      ga[c] = q == 0 ? sp.gram : q == 1 ? sp.poly : sp.upd;
      const TileCosts own = tile_costs(ga[c], geoms[c].nmat, false);
      alone += own.small < 0.9 * own.large ? own.small : own.large;
      tiles += double(geoms[c].nmat) * double(large_tiles(ga[c]));
    }
    const double cus = device_cu_count(), rounds = std::ceil(tiles / cus), f = tiles / (rounds * cus);
    for (int c = 0; c < n; ++c) {
      const double us = large_tile_us(f, ga[c].k_slabs);
      longest = std::max(longest, us);
      slabs_us += us * double(geoms[c].nmat) * double(large_tiles(ga[c]));
    }
    grouped += std::max(longest, rounds * slabs_us / tiles);
  }
  return grouped < alone;
}

hipError_t run_group(const GroupMember* m, int n, const StepScalars& sc, int K, hipStream_t st,
                     LaunchTimer* timer) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  for (int c = 0; c < n; ++c)
    if (!group_eligible(m[c].geom, K) || m[c].geom.param_dtype != m[0].geom.param_dtype) return hipErrorInvalidValue;
  hipError_t e;
  for (int c = 0; c < n; ++c) {
    const bool gbf = m[c].geom.grad_dtype == DT_BF16;
    e = gbf ? run_prologue_t<uint16_t, uint16_t>(m[c].geom, m[c].desc, m[c].wb, sc, m[c].coeffs, K, st, timer)
            : run_prologue_t<float, uint16_t>(m[c].geom, m[c].desc, m[c].wb, sc, m[c].coeffs, K, st, timer);
    if (e != hipSuccess) return e;
  }
  int cur = 0;
  for (int k = 0; k < K; ++k) {
    GemmArgs ga[3][kMaxGroup];
    int nm[kMaxGroup];
    double f[3] = {0, 0, 0}, b[3] = {0, 0, 0};
    bool last = false;
    for (int c = 0; c < n; ++c) {
      const StepProducts sp = step_products<uint16_t>(m[c].geom, m[c].desc, m[c].wb, sc, m[c].coeffs, K, k, cur);
      ga[0][c] = sp.gram; ga[1][c] = sp.poly; ga[2][c] = sp.upd;
      nm[c] = m[c].geom.nmat;
      for (int q = 0; q < 3; ++q) { f[q] += sp.f[q]; b[q] += sp.b[q]; }
      last = sp.last;
    }
    const int kinds[3] = {KK_GRAM, KK_POLY, last ? KK_FINAL : KK_UPDATE};
    const int epis[3] = {EPI_GRAM, EPI_POLY, last ? EPI_FINAL : EPI_UPDATE};
    for (int q = 0; q < 3; ++q) {
      Timed tm(timer, kinds[q], st);
      double exec = 0.0;
      if ((e = launch_group<CfgSquare>(epis[q], ga[q], nm, n, st, exec)) != hipSuccess) return e;
      tm.done(f[q], exec, b[q]);
    }
    cur ^= 1;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// AdamW over many tensors in one launch: workgroup b updates elements
// [8192 j, 8192 (j + 1)) of the tensor whose range of workgroups holds b
// (found by binary search over first_block).  HBM-bound: each element reads
// p, g, m, v and writes p, m, v once; 8 consecutive elements per thread
// (16-byte accesses) when the tensor allows it.
// ---------------------------------------------------------------------------
template <typename PT, typename GT>
__device__ __forceinline__ void adam_one(float& p, float g, float& m, float& v, const AdamScalars& sc) {
  m = fmaf(sc.beta1, m, sc.one_minus_beta1 * g);
  v = fmaf(sc.beta2, v, sc.one_minus_beta2 * (g * g));
  const float denom = fmaf(sqrtf(v), sc.inv_sqrt_bc2, sc.eps);
  p = fmaf(p, sc.decay, -sc.step_size * (m / denom));
}

template <typename PT, typename GT>
__global__ __launch_bounds__(256) void k_adamw(const AdamDesc* __restrict__ desc, int n, AdamScalars sc) {
  const int64_t b = blockIdx.x;
  int lo = 0, hi = n - 1;  // last tensor with first_block <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (desc[mid].first_block <= b) lo = mid;
    else hi = mid - 1;
  }
  const AdamDesc a = desc[lo];
  const int64_t start = (b - a.first_block) * kAdamElemsPerBlock;
  const int64_t end = min(a.numel, start + static_cast<int64_t>(kAdamElemsPerBlock));
  PT* __restrict__ p = static_cast<PT*>(a.p);
  const GT* __restrict__ g = static_cast<const GT*>(a.g);
  float* __restrict__ m = a.m;
  float* __restrict__ v = a.v;
  if (a.vec_ok) {
    for (int64_t i = start + threadIdx.x * 8; i < end; i += 256 * 8) {
      float pv[8], gv[8], mv[8], vv[8];
      load8(p, i, pv);
      load8(g, i, gv);
      load8(m, i, mv);
      load8(v, i, vv);
#pragma unroll
      for (int q = 0; q < 8; ++q) adam_one<PT, GT>(pv[q], gv[q], mv[q], vv[q], sc);
      store8(p, i, pv);
      store8(m, i, mv);
      store8(v, i, vv);
    }
  } else {
    for (int64_t i = start + threadIdx.x; i < end; i += 256) {
      float pv = to_f32<PT>(p[i]), mv = m[i], vv = v[i];
      adam_one<PT, GT>(pv, to_f32<GT>(g[i]), mv, vv, sc);
      p[i] = from_f32<PT>(pv);
      m[i] = mv;
      v[i] = vv;
    }
  }
}

// Descriptor records copied into device memory by a kernel that takes them
// as its arguments: the allocation-free entry point fills its table this
// way, with no host staging buffer.  Indices are compile-time constants, so
// the records are read straight from the argument segment.
namespace {
__global__ __launch_bounds__(64) void k_put_desc(DescBatch b, MatDesc* __restrict__ dst) {
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int i = 0; i < kDescPerLaunch; ++i)
    if (i < b.n) dst[i] = b.d[i];
}
}  // namespace

hipError_t put_descriptors(const MatDesc* host, int n, MatDesc* dev, hipStream_t st) {
  for (int first = 0; first < n; first += kDescPerLaunch) {
    DescBatch b{};
    b.n = min(kDescPerLaunch, n - first);
    for (int i = 0; i < b.n; ++i) b.d[i] = host[first + i];
    hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(64), 0, st, b, dev + first);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Streaming copy, the reference for what HBM delivers to the elementwise
// kernels: each workgroup copies its own contiguous 256 KiB with 16-byte
// non-temporal accesses, four in flight per thread (measured the fastest of
// grid-stride and block-contiguous variants, 1-8 accesses per thread).
namespace {
constexpr int64_t kCopyVecsPerBlock = 16384;
__global__ __launch_bounds__(256) void k_stream_copy(const u32x4_t* __restrict__ src, u32x4_t* __restrict__ dst,
                                                     int64_t n) {
  const int64_t lo = static_cast<int64_t>(blockIdx.x) * kCopyVecsPerBlock;
  const int64_t hi = min(lo + kCopyVecsPerBlock, n);
  for (int64_t i = lo + threadIdx.x; i < hi; i += 4 * 256) {
    u32x4_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * 256 < hi) v[u] = __builtin_nontemporal_load(src + i + u * 256);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * 256 < hi) __builtin_nontemporal_store(v[u], dst + i + u * 256);
  }
}
__global__ __launch_bounds__(256) void k_copy_tail(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
                                                   int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i];
}
}  // namespace

hipError_t stream_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
  const int64_t vecs = static_cast<int64_t>(bytes / 16);
  if (vecs > 0) {
    const int64_t blocks = (vecs + kCopyVecsPerBlock - 1) / kCopyVecsPerBlock;
    hipLaunchKernelGGL(k_stream_copy, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st,
                       static_cast<const u32x4_t*>(src), static_cast<u32x4_t*>(dst), vecs);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int64_t tail = static_cast<int64_t>(bytes % 16);
  if (tail > 0) {
    hipLaunchKernelGGL(k_copy_tail, dim3(1), dim3(256), 0, st, static_cast<const uint8_t*>(src) + vecs * 16,
                       static_cast<uint8_t*>(dst) + vecs * 16, tail);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t run_adamw(const AdamDesc* d_desc, int n, int64_t blocks, int param_dtype, int grad_dtype,
                     const AdamScalars& sc, double bytes, hipStream_t st, LaunchTimer* timer) {
  if (n <= 0 || blocks <= 0) return hipSuccess;
  Timed tm(timer, KK_ADAMW, st);
  const dim3 grid(static_cast<unsigned>(blocks)), block(256);
  const bool pb = param_dtype == DT_BF16, gb = grad_dtype == DT_BF16;
  if (pb && gb) hipLaunchKernelGGL((k_adamw<uint16_t, uint16_t>), grid, block, 0, st, d_desc, n, sc);
  else if (pb) hipLaunchKernelGGL((k_adamw<uint16_t, float>), grid, block, 0, st, d_desc, n, sc);
  else if (gb) hipLaunchKernelGGL((k_adamw<float, uint16_t>), grid, block, 0, st, d_desc, n, sc);
  else hipLaunchKernelGGL((k_adamw<float, float>), grid, block, 0, st, d_desc, n, sc);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) tm.done(0, 0, bytes);
  return e;
}

}  // namespace muon
