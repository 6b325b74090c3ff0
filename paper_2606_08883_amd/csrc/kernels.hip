// HIP kernels for gfx950 (64-lane wavefronts): the fine five-point operator,
// the batched block-LDL^T box solves of the MRCM-OS apply, the level-scheduled
// coarse interface solve, multiscale reconstruction, Schwarz smoothing and the
// fused Arnoldi vector kernels of GMRES.  Every reduction has a fixed order,
// so results are bit-identical from run to run.
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace mrcm {

namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum over a block of kVecThreads threads; result valid in every thread.
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  const int nw = blockDim.x >> 6;
  for (int k = 0; k < nw; ++k) s += red[k];
  return s;
}

// Store a value where the host waits for it (mailbox.h).
__device__ __forceinline__ void publish(double* place, double v) {
  __hip_atomic_store(place, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Sum of nb partials, identical order in every block.
// Elements a thread handles per round of a grid-stride loop: the loads of a
// round are all issued (indices clamped into range) before any is used, so
// they are in flight together; a thread still visits its elements in
// increasing order, so the reductions keep one fixed order.
constexpr int kRound = 4;

__device__ __forceinline__ double reduce_partials(const double* part, int nb, double* red) {
  double v = 0.0;
  for (int k0 = threadIdx.x; k0 < nb; k0 += kRound * blockDim.x) {
    double a[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const int k = k0 + u * blockDim.x;
      a[u] = part[k < nb ? k : nb - 1];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u)
      if (k0 + u * (int)blockDim.x < nb) v += a[u];
  }
  return block_sum(v, red);
}

// y_c = sum_f t_f (x_c - x_c') over the four faces; boundary faces carry the
// Dirichlet half-transmissibility (coupled to zero) or zero.  Branch-free:
// missing neighbours are read at the cell itself and meet a zero
// coefficient, so all loads are unconditional.
// x(c) gives the vector's value at cell c.
template <typename T, typename X>
__device__ __forceinline__ T stencil_of(const T* __restrict__ tx, const T* __restrict__ ty, int nx,
                                        int ny, int ix, int iy, X x) {
  const long long c = (long long)iy * nx + ix;
  const long long fx = (long long)iy * (nx + 1) + ix;
  const T tW = tx[fx], tE = tx[fx + 1], tS = ty[c], tN = ty[c + nx];
  const T xc = x(c);
  const T xw = x(ix > 0 ? c - 1 : c), xe = x(ix + 1 < nx ? c + 1 : c);
  const T xs = x(iy > 0 ? c - nx : c), xn = x(iy + 1 < ny ? c + nx : c);
  T v = (tW + tE + tS + tN) * xc;
  v -= (ix > 0 ? tW : T(0)) * xw;
  v -= (ix + 1 < nx ? tE : T(0)) * xe;
  v -= (iy > 0 ? tS : T(0)) * xs;
  v -= (iy + 1 < ny ? tN : T(0)) * xn;
  return v;
}
template <typename T>
__device__ __forceinline__ T stencil(const T* __restrict__ tx, const T* __restrict__ ty, int nx,
                                     int ny, int ix, int iy, const T* __restrict__ x) {
  return stencil_of(tx, ty, nx, ny, ix, iy, [&](long long c) { return x[c]; });
}

// y_k = A x_k for K vectors of n values one after the other.  Bound by memory: a
// thread takes kOpRows cells of a grid column, so that what neighbouring rows
// share is loaded once, and the transmissibilities once for the K vectors; a
// workgroup takes a tile of 64 x 4 kOpRows cells, each eighth of the workgroups (one
// L2) a band of consecutive tiles, and y, which no later load of the launch
// needs, is stored past the caches.  2048 x 2048, four columns: 117 us as four
// launches of a thread per cell, 91 in one, 79 with the tiles (76 to 81 with 2 or 8
// rows, 77 without the bands, which one column misses: 20 -> 23 us), 75 with y past
// the caches (54 where x is still cached, 78 without that).  The terms of a cell are
// those of stencil, in its order.
constexpr int kOpColumns = 4, kOpRows = 4;
template <int K>
__global__ void __launch_bounds__(kVecThreads)
    k_op_apply(const double* __restrict__ tx, const double* __restrict__ ty, int nx, int ny,
               int tiles_x, int tiles, const double* __restrict__ x, double* __restrict__ y) {
  constexpr int R = kOpRows;
  const int tile = (blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (tile >= tiles) return;
  const int ix = (tile % tiles_x) * 64 + (threadIdx.x & 63);
  const int y0 = (tile / tiles_x) * 4 * R + (int)(threadIdx.x >> 6) * R;
  if (ix >= nx || y0 >= ny) return;
  const long long n = (long long)nx * ny;
  const bool west = ix > 0, east = ix + 1 < nx;
  double tw[R], te[R], tv[R + 1];
  long long row[R];  // first cells of the rows, clamped into the grid
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int iy = y0 + j < ny ? y0 + j : ny - 1;
    row[j] = (long long)iy * nx;
    tw[j] = tx[row[j] + iy + ix];
    te[j] = tx[row[j] + iy + ix + 1];
  }
#pragma unroll
  for (int j = 0; j <= R; ++j) tv[j] = ty[(long long)(y0 + j < ny ? y0 + j : ny) * nx + ix];
  const long long below = (y0 > 0 ? (long long)(y0 - 1) * nx : row[0]) + ix;
  const long long above = (y0 + R < ny ? (long long)(y0 + R) * nx : row[R - 1]) + ix;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double* xk = x + k * n;
    double xv[R + 2], xw[R], xe[R];
    xv[0] = xk[below];
    xv[R + 1] = xk[above];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      xv[j + 1] = xk[row[j] + ix];
      xw[j] = xk[row[j] + (west ? ix - 1 : ix)];
      xe[j] = xk[row[j] + (east ? ix + 1 : ix)];
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int iy = y0 + j;
      if (iy >= ny) break;
      double v = (tw[j] + te[j] + tv[j] + tv[j + 1]) * xv[j + 1];
      v -= (west ? tw[j] : 0.0) * xw[j];
      v -= (east ? te[j] : 0.0) * xe[j];
      v -= (iy > 0 ? tv[j] : 0.0) * xv[j];
      v -= (iy + 1 < ny ? tv[j + 1] : 0.0) * (iy + 1 < ny ? xv[j + 2] : xv[j + 1]);
      __builtin_nontemporal_store(v, y + k * n + row[j] + ix);
    }
  }
}

__global__ void k_rhs(const double* __restrict__ tx, const double* __restrict__ ty, int nx,
                      int ny, int bcW, int bcE, int bcS, int bcN, const double* __restrict__ f,
                      const double* __restrict__ g, double h, double* __restrict__ b) {
  const long long n = (long long)nx * ny;
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x) {
    const int iy = (int)(c / nx), ix = (int)(c - (long long)iy * nx);
    double v = f ? f[c] * h * h : 0.0;
    if (g) {
      if (ix == 0 && bcW) v += tx[(long long)iy * (nx + 1)] * g[iy];
      if (ix == nx - 1 && bcE) v += tx[(long long)iy * (nx + 1) + nx] * g[ny + iy];
      if (iy == 0 && bcS) v += ty[ix] * g[2 * ny + ix];
      if (iy == ny - 1 && bcN) v += ty[(long long)ny * nx + ix] * g[2 * ny + nx + ix];
    }
    b[c] = v;
  }
}

// Virtual block of a launch: its index and the block count of its grid.  A
// launch over one context uses the hardware grid; a launch over several
// contexts gives every column its own range of workgroups, each of which
// runs as block `id` of a grid of `n`, so that every column's arithmetic and
// reduction order are those of its own launch.
struct Blk {
  int id, n;
};
__device__ __forceinline__ Blk hw_blk() { return Blk{(int)blockIdx.x, (int)gridDim.x}; }

// ---- batched box solves ---------------------------------------------------
// A cell box is solved with the block LDL^T factor of its cell rows
// (setup_jobs.h) by one lane group per end of the elimination: the factors in
// FP64 are two-ended (the group of end 0 eliminates the rows below the middle
// row h upward, the group of end 1 the rows above it downward, both solve row h,
// and each substitutes back from it on its own side), the ones stored in FP32
// one-ended (end 0 only, h the last row):
//   end 0  u_j = D_j^-1 (b_j + T_j u_{j-1}),      x_j = u_j + D_j^-1 (T_{j+1} x_{j+1}),
//   end 1  u_j = D_j^-1 (b_j + T_{j+1} u_{j+1}),  x_j = u_j + D_j^-1 (T_j x_{j-1}),
//   middle x_h = D_h^-1 (b_h + T_h u_{h-1} + T_{h+1} u_{h+1}).
// Two ends halve the chain of dependent row steps, which bounds the solve
// wherever the boxes do not fill the GPU several times over.
// A group is one wave: R row lanes, R = 64 for boxes wider than 32 columns, else
// R = 32 with two lanes per row (halves), which halves
// the instructions of a row step, the other thing a step waits for.  Many boxes of up to
// 16 columns, which fill the GPU, are packed instead: 16 lanes to a group, one per row, four
// groups to a wave, or 32 lanes for up to 20 columns (kPacked16, kPacked20).  Lane r of a
// half owns cell column r of every row.
// The blocks are symmetric and stored as half blocks (setup_jobs.h): row r's
// lanes load the entries D(r, r + k), k = 0 .. NB / 2, of each block and fetch
// D(r, r - k) = D(r - k, r) from the registers of row r - k's lanes.  Exchange
// inside a group is wave-local: the vector of a step goes through the group's
// slot of LDS, the mirrored entries through cross-lane permutes.  The two groups
// of a box meet at two workgroup barriers around the middle row.  The row of a
// step, its addresses and its phase are the same in the whole wave and live in
// scalar registers (unless packed); lanes past the box's width repeat its last column (same
// values to the same addresses), so that a step masks nothing.
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// a * b + c with one rounding, spelled out so that the one-RHS and the
// multi-RHS kernels round every step the same way whatever the optimiser
// would contract.
__device__ __forceinline__ float fmat(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}
__device__ __forceinline__ double fmat(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}

// Four consecutive words of a factor block (16 bytes of FP32 or 32 bytes of
// FP64), as native vectors the optimiser keeps in registers.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <typename S> struct Quad;
template <> struct Quad<float> {
  f32x4 v;
  __device__ float operator[](int i) const { return v[i]; }
};
template <> struct Quad<double> {
  f64x2 lo, hi;
  __device__ double operator[](int i) const { return i < 2 ? lo[i] : hi[i - 2]; }
};
__device__ __forceinline__ void load_quad(Quad<float>& q, const float* p) {
  q.v = *reinterpret_cast<const f32x4*>(p);
}
__device__ __forceinline__ void load_quad(Quad<double>& q, const double* p) {
  q.lo = *reinterpret_cast<const f64x2*>(p);
  q.hi = *reinterpret_cast<const f64x2*>(p + 2);
}

// Make v opaque to the optimiser at this point, so that addresses derived
// from it are recomputed here instead of being hoisted out of the row loop
// into registers for the whole kernel.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Packed forms of boxes of up to 16 and of 17 to 20 columns: the blocks and the arithmetic
// of column widths 16 and 20 (the same bits) with groups of 16 and 32 lanes, one per row,
// four and two groups to a wave.  A wave of its own leaves lanes of a narrow box idle, which
// costs nothing while the boxes do not fill the GPU and up to twice the time once they do
// (launch_cols).  The codes are odd: NB / 2 and the shape of a half block are those of
// NB - 1.
constexpr int kPacked16 = 17, kPacked20 = 21;

// Shape of the half blocks of a launch of column width NB: rows 0 .. H, the
// first K0 of them single words, the others NH quads; R row lanes per half and
// HV halves per group of GL lanes (one wave unless packed).
template <int NB>
struct Half {
  static constexpr bool PACK = NB % 2 == 1;
  static constexpr int H = NB / 2;
  static constexpr int K0 = half_k0(NB);
  static constexpr int NH = half_quads(NB);
  static constexpr int R = NB == kPacked16 ? 16 : NB <= 32 ? 32 : 64;
  static constexpr int HV = PACK ? 1 : 64 / R;
  static constexpr int GL = R * HV;
  static constexpr int NT = (H + 3) / 4;          // steps of four mirrored entries
  static constexpr int NM = HV == 2 ? 2 * NT : H;  // mirrored entries a lane fetches, at most
  // Place of v in the vector slot: H words hold what lies before it; one more where half
  // 1's last mirrored step, which it discards, reaches beyond them (a one-cell row and
  // three words too many: column width 20).
  static constexpr int V0 = HV == 2 && 4 * NT > H + 1 ? H + 1 : H;
  static_assert(HV == 1 || K0 == 1 || K0 == 3, "halves of a row: one or three single words");
  static_assert(HV == 1 || V0 + 1 >= 4 * NT, "mirrored reads stay in the vector slot");
};
// Ends of the factors of storage type S (groups per box).
template <typename S>
constexpr int box_ends() { return sizeof(S) == 8 ? 2 : 1; }

// Two consecutive words of a factor block.
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <typename S> struct PairOf;
template <> struct PairOf<float> { typedef f32x2 type; };
template <> struct PairOf<double> { typedef f64x2 type; };

// A lane's words of one half block.  One lane per row: all of them (row(k) is
// entry D(r, r + k), k a constant after unrolling).  Two lanes per row: words 2 hf
// and 2 hf + 1 of every quad, and the single words that half hf multiplies
// (s[0]: word 2 hf) or passes on (s[1]: word 1).
template <typename S, int NB, int HV = Half<NB>::HV>
struct HalfRow {
  Quad<S> q[Half<NB>::NH];
  S h[Half<NB>::K0 > 0 ? Half<NB>::K0 : 1];
  __device__ S row(int k) const {
    constexpr int K0 = Half<NB>::K0;
    return k < K0 ? h[k] : q[(k - K0) >> 2][(k - K0) & 3];
  }
};
template <typename S, int NB>
struct HalfRow<S, NB, 2> {
  typename PairOf<S>::type p[Half<NB>::NH];
  S s[2];
};

// VGPRs of a lane's words of one block.
template <typename S, int NB>
constexpr int block_regs() {
  return (int)sizeof(S) / 4 *
         (Half<NB>::HV == 1 ? half_rows(NB) : 2 * Half<NB>::NH + (Half<NB>::K0 == 3 ? 2 : 1));
}
// Waves per SIMD the compiler aims for in the box kernels of one box per item, at least and
// at most.  DENSE: launches over several contexts (of 48-wide FP32 factors in FP64
// arithmetic only past a wave per SIMD, box_dense) and, for FP64 boxes of 37 to 48 columns, one
// column past a wave per SIMD.  Left alone the compiler gives up loads in flight for one wave
// more, or takes a few registers too many for two.  Measured, left alone and as here, us:
//   one column of T, FP32 factors in FP64 arithmetic, 512 x 512, 64-wide boxes   271   184
//     (40- and 36-wide boxes, two sweeps)                                        212   182
//   one column, FP64, local: 1024 boxes 40 wide / 576 of 48                  102 129   91 119
//     (144 boxes 48 wide, T: 136, on the DENSE kernels 156)
//   four columns over contexts, local and patch: FP32, 1024 boxes 36 wide    193 153  158 141
//     FP32, 576 of 48 / 256 of 64                            227 196 143 124  190 160  92 77
//     FP64, 1024 of 36 / 576 of 48 (spills 32 bytes)         282 350 381 332  280 277 303 262
//     (FP64 64 wide at two waves: 171 173, left alone 80 72)
// At three waves FP64 24 wide loses (1024 x 1024: 75.2, 77.3, at two 84.5).
template <typename T, typename S, int NB, bool DENSE>
constexpr int box_most_waves() {
  return (sizeof(T) == 8 && sizeof(S) == 4 && NB >= 36) || (DENSE && sizeof(T) == 4 && NB >= 36)
             ? 2
             : 8;
}
template <typename T, typename S, int NB, bool DENSE>
constexpr int box_least_waves() {
  return !DENSE                                                                 ? 1
         : (sizeof(S) == 8 && NB >= 36 && NB <= 48) || (sizeof(T) == 8 && NB == 48) ? 2
         : sizeof(T) == 4 && NB <= 32 && !Half<NB>::PACK                        ? 4
                                                                                : 1;
}
#define MRCM_BOX_KERNEL(T, S, NB, DENSE)                                                \
  __launch_bounds__(kBoxThreads) __attribute__((amdgpu_waves_per_eu(                    \
      box_least_waves<T, S, NB, DENSE>(), box_most_waves<T, S, NB, DENSE>())))
// Blocks in flight per lane, 2 or 4: as many as about 64 VGPRs of rows hold (more
// would cost waves per SIMD; 36-wide FP32 patches with four in flight instead
// of two were a third slower).
constexpr int sweep_depth(int vgprs, int per_block) { return vgprs / per_block >= 4 ? 4 : 2; }
template <typename S, int NB>
constexpr int reg_depth() { return sweep_depth(64, block_regs<S, NB>()); }

// Lane rc's words of one block of a box n cells wide: the quads at words
// (q n + rc) 4, the single words at 4 NH n + k n + rc, so the group reads
// contiguous pieces.  blk is the same in the whole wave; a lane's places in the
// block are 32-bit offsets from it that do not change from block to block.
template <typename S, int NB>
struct BlockPlaces {
  unsigned q, h, n;  // words of the lane's first quad piece and first single word; columns
  __device__ BlockPlaces(int n_, int rc, int hf) : n(n_) {
    q = 4 * rc + 2 * hf;
    h = 4 * Half<NB>::NH * n_ + rc + (Half<NB>::K0 == 3 ? 2 * hf * n_ : 0);
    if constexpr (Half<NB>::HV == 1) {
      // one register each: the places are recomputed from these at every use
      q = opaque(q);
      h = opaque(h);
    }
  }
};
template <typename S, int NB>
__device__ __forceinline__ void load_half(HalfRow<S, NB>& d, const S* __restrict__ blk,
                                          const BlockPlaces<S, NB>& at, int rc) {
  constexpr int NH = Half<NB>::NH, K0 = Half<NB>::K0;
  if constexpr (Half<NB>::HV == 1) {
#pragma unroll
    for (int q = 0; q < NH; ++q) load_quad(d.q[q], blk + (size_t)(at.q + q * 4 * at.n));
#pragma unroll
    for (int k = 0; k < K0; ++k) d.h[k] = blk[(size_t)(at.h + k * at.n)];
  } else {
    typedef typename PairOf<S>::type P;
#pragma unroll
    for (int q = 0; q < NH; ++q)
      d.p[q] = *reinterpret_cast<const P*>(blk + (size_t)(at.q + q * 4 * at.n));
    d.s[0] = blk[(size_t)at.h];
    if constexpr (K0 == 3) d.s[1] = blk[(size_t)(4 * NH * at.n + rc + at.n)];
  }
}

// Value v of the lane whose byte address (4 x lane index) is addr.
__device__ __forceinline__ float lane_fetch(int addr, float v) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double lane_fetch(int addr, double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)b);
  const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum of v over the two halves of the wave (lanes l and l ^ 32), the same in both.
__device__ __forceinline__ float sum_halves(float v) {
  const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}
__device__ __forceinline__ double sum_halves(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// Where a lane's mirrored entries D(rc, rc - k) are held: row lane (rc - k) mod n
// (row lane 0 for k > n, where every lane holds
// a zero row).  One lane per row: k = 1 .. H, byte addresses packed four to a word
// (held unpacked they would fill the registers).  Two lanes per row and one single
// word in a block: half hf takes k = 4 t + 1 + 2 hf + e (e = 0, 1) at [2 t + e], the
// words it holds itself.  Three single words: in FP64 arithmetic (OWN) half hf takes
// the words it holds, k = 3 + 4 q + 2 hf + e at [2 q + e] and k = 1 + hf last; in
// FP32 arithmetic, whose sums keep the order of one lane per row, k = 4 t + 1 + 2 hf
// + e, which the other half holds (its two selects per entry cost 5 us of the 45
// of a 20-wide patch sweep at 1024^2).
template <int NB, bool OWN>
struct Mirror {
  static constexpr int H = Half<NB>::H, HV = Half<NB>::HV, NT = Half<NB>::NT;
  static constexpr int NH = Half<NB>::NH, K0 = Half<NB>::K0;
  int src[HV == 1 ? (H + 3) / 4 : 2 * NT];
  __device__ static int col(int rc, int k, int n) {
    int c = rc - k;
    c = c < 0 ? c + n : c;
    return c < 0 ? 0 : c;
  }
  __device__ Mirror(int rc, int hf, int n) {
    if constexpr (HV == 1) {
      // the group's first lane
      const int g0 = Half<NB>::PACK ? (int)(threadIdx.x & 63) / Half<NB>::GL * Half<NB>::GL : 0;
#pragma unroll
      for (int w = 0; w < (H + 3) / 4; ++w) src[w] = 0;
#pragma unroll
      for (int k = 1; k <= H; ++k)
        src[(k - 1) >> 2] |= (4 * (g0 + col(rc, k, n))) << (8 * ((k - 1) & 3));
    } else if constexpr (K0 == 3 && OWN) {
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i)
        src[i] = 4 * (hf * Half<NB>::R +
                      col(rc, i < 2 * NH ? 3 + 4 * (i >> 1) + 2 * hf + (i & 1) : 1 + hf, n));
    } else {
      const int base = (K0 == 3 ? 1 - hf : hf) * Half<NB>::R;
#pragma unroll
      for (int i = 0; i < 2 * NT; ++i)
        src[i] = 4 * (base + col(rc, 4 * (i >> 1) + 1 + 2 * hf + (i & 1), n));
    }
  }
};

// The mirrored entries of one block (one lane per row: the packed
// addresses are unpacked at each use; opaque keeps the optimiser from
// holding all H of them in registers across the sweep).
template <typename S, int NB, bool OWN>
__device__ __forceinline__ void mirror_rows(S (&rot)[Half<NB>::NM], const HalfRow<S, NB>& d,
                                            const Mirror<NB, OWN>& m, int hf) {
  constexpr int H = Half<NB>::H, NT = Half<NB>::NT, NH = Half<NB>::NH;
  if constexpr (Half<NB>::HV == 1) {
    int w[(H + 3) / 4];
#pragma unroll
    for (int i = 0; i < (H + 3) / 4; ++i) w[i] = opaque(m.src[i]);
#pragma unroll
    for (int k = 1; k <= H; ++k)
      rot[k - 1] = lane_fetch((w[(k - 1) >> 2] >> (8 * ((k - 1) & 3))) & 255, d.row(k));
  } else if constexpr (Half<NB>::K0 == 1) {
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) rot[i] = lane_fetch(m.src[i], d.p[i >> 1][i & 1]);
  } else if constexpr (OWN) {
#pragma unroll
    for (int i = 0; i < 2 * NH; ++i) rot[i] = lane_fetch(m.src[i], d.p[i >> 1][i & 1]);
    rot[2 * NH] = lane_fetch(m.src[2 * NH], hf ? d.s[0] : d.s[1]);
  } else {
    // what this lane passes to the other half: half 1 the single words 1 and 2,
    // then its pair of quad t - 1; half 0 its pair of quad t
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) {
      const int t = i >> 1, e = i & 1;
      const S up = t == 0 ? (e ? d.s[0] : d.s[1]) : d.p[t > 0 ? t - 1 : 0][e];
      const S dn = t < NH ? d.p[t < NH ? t : 0][e] : S(0);
      rot[i] = lane_fetch(m.src[i], hf ? up : dn);
    }
  }
}

// One lane per row: the mirrored entry k that is added i-th (1 .. H) and its partial sum,
// k = 1 .. H in turn, or the order of two lanes per row in FP64 arithmetic with three single
// words (Mirror, OWN): k = 3 .. H, then 1 and 2.
template <typename T, int NB>
constexpr bool own_order() { return Half<NB>::PACK && Half<NB>::K0 == 3 && sizeof(T) == 8; }
template <typename T, int NB>
__device__ constexpr int mirror_k(int i) {
  return !own_order<T, NB>() ? i : i <= Half<NB>::H - 2 ? i + 2 : i - (Half<NB>::H - 2);
}
template <typename T, int NB>
__device__ constexpr int mirror_sum(int i) {
  const int k = mirror_k<T, NB>(i);
  return !own_order<T, NB>() ? (k - 1) & 3 : k >= 3 ? (k - 3) & 3 : 2 * k - 1;
}

// acc = sum_c D(rc, c) v[c]: the rows k against vo[k] = v[(rc + k)
// mod n], the mirrored entries against vr[-k] = v[(rc - k) mod n] (vo and vr
// point into the group's doubled copy of v); four partial sums shorten the
// chain of dependent additions.  Two lanes per row: half hf forms the partial
// sums 2 hf and 2 hf + 1 (vo and vr shifted by 2 hf by the caller), so the result
// is that of one lane, bit for bit, unless half hf takes the mirrored words it holds
// (Mirror).
template <typename T, typename S, int NB, bool DENSE>
__device__ __forceinline__ T half_dot(const HalfRow<S, NB>& d, const S (&rot)[Half<NB>::NM],
                                      const T* vo, const T* vr, int hf) {
  constexpr int NH = Half<NB>::NH, K0 = Half<NB>::K0, H = Half<NB>::H, NT = Half<NB>::NT;
  if constexpr (Half<NB>::HV == 1) {
    T a[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int q = 0; q < NH; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = fmat((T)d.q[q][i], vo[K0 + 4 * q + i], a[i]);
#pragma unroll
    for (int k = 0; k < K0; ++k) a[k] = fmat((T)d.h[k], vo[k], a[k]);
    // fewer vector words in registers at a time, so that two waves fit
    if constexpr (DENSE && sizeof(T) == 8 && sizeof(S) == 4 && NB == 48)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 1; i <= H; ++i) {
      const int k = mirror_k<T, NB>(i), p = mirror_sum<T, NB>(i);
      a[p] = fmat((T)rot[k - 1], vr[-k], a[p]);
    }
    return (a[0] + a[1]) + (a[2] + a[3]);
  } else {
    T a[2] = {T(0), T(0)};
#pragma unroll
    for (int q = 0; q < NH; ++q)
#pragma unroll
      for (int e = 0; e < 2; ++e) a[e] = fmat((T)d.p[q][e], vo[K0 + 4 * q + e], a[e]);
    const T s0 = fmat((T)d.s[0], vo[0], a[0]);
    if constexpr (K0 == 3) {
      const T s1 = fmat((T)d.s[1], vo[1], a[1]);
      a[0] = s0;
      a[1] = hf ? a[1] : s1;
    } else {
      a[0] = hf ? a[0] : s0;
    }
    if constexpr (K0 == 3 && sizeof(T) == 8) {
#pragma unroll
      for (int q = 0; q < NH; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          a[e] = fmat((T)rot[2 * q + e], vr[-(3 + 4 * q + e)], a[e]);
      a[1] = fmat((T)rot[2 * NH], vr[hf - 1], a[1]);
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const T v = fmat((T)rot[2 * t + e], vr[-(4 * t + 1 + e)], a[e]);
          a[e] = 4 * t + 3 + e <= H ? v : hf ? a[e] : v;  // the last step of half 1 may lack it
        }
    }
    return sum_halves(a[0] + a[1]);
  }
}

// One sweep over n row blocks of a box, the first at blk and each next one at
// `dir` words from the one before.  Step s uses its block's words, loaded into
// register set s % DEPTH at step
// s - DEPTH; right after its use the set is refilled with block s + DEPTH (the
// last block past the end), so every block has DEPTH - 1 steps to arrive.  No load
// is conditional, so the
// compiler counts the loads in flight exactly and waits only for the block
// a step uses; the n % DEPTH last steps, which load nothing, run after the loop
// (rounding the count up instead ran 24 steps for the 17 to 20 of a 20-wide patch).
// Packed groups of a wave have different counts: all of them end with the wave's last
// step and one with fewer starts `late` steps later, on its first block until then
// (steps below 0; n < 1: it never starts).
template <typename S, int NB, int DEPTH, typename Step>
__device__ __forceinline__ void pipelined_sweep(int n, int late, const S* __restrict__ blk,
                                                int dir, Step step, int bx, int rc, int hf) {
  const BlockPlaces<S, NB> at(bx, rc, hf);
  HalfRow<S, NB> reg[DEPTH];
  constexpr bool PACK = Half<NB>::PACK;
  int left = n - 1, wait = late;  // blocks after the one at blk; steps before the first
  auto next = [&]() {
    const bool go = !PACK || wait <= 0;
    blk += go && left > 0 ? dir : 0;
    left -= go ? 1 : 0;
    if constexpr (PACK) --wait;
  };
  if constexpr (PACK)
    n = __builtin_amdgcn_readfirstlane((n > 0 ? n : 0) + late);
  else
    late = 0;
#pragma unroll
  for (int u = 0; u < DEPTH; ++u) {
    load_half<S, NB>(reg[u], blk, at, rc);
    next();
  }
  int s0 = 0;
  for (; s0 + DEPTH <= n; s0 += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      step(s0 + u - late, reg[u]);
      load_half<S, NB>(reg[u], blk, at, rc);
      next();
    }
  }
#pragma unroll
  for (int u = 0; u < DEPTH - 1; ++u)
    if (s0 + u < n) step(s0 + u - late, reg[u]);
}

// Words of the group's copy of the step vector for column width NB:
// v at [V0, V0 + n) and again at [V0 + n, V0 + 2 n), zeros around it
// (the lane's rows past the box meet finite values).
template <int NB>
constexpr int vec_words() { return (Half<NB>::V0 + 2 * Half<NB>::R + 3) / 4 * 4; }

// Zero the group's vector slots (count words) before the first step.
template <int GL, typename T>
__device__ __forceinline__ void zero_slots(T* v, int count) {
  for (int i = threadIdx.x % GL; i < count; i += GL) v[i] = T(0);
}

// Meet the other group of the box, if it has two.  The meeting is the workgroup's: every
// wave of a launch has to pass the same number of them (two in a box solve, one where the
// middle row is reached and one when it has been read, whatever the box's rows).
// Packed groups of a box share a wave.
template <typename S, int NB>
__device__ __forceinline__ void pair_sync() {
  if constexpr (box_ends<S>() == 2 && !Half<NB>::PACK)
    __syncthreads();
  else
    wave_sync();
}

// Largest value of v over the 64 lanes of the wave, as a wave-uniform value.
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return __builtin_amdgcn_readfirstlane(v);
}
// Steps by which a group with n steps starts after the one of its wave with the most.
template <int NB>
__device__ __forceinline__ int late_start(int n) {
  if constexpr (Half<NB>::PACK)
    return wave_max(n) - n;
  else
    return 0;
}

// The row steps of one end of a box of by rows: from row first, step by dir rows,
// the elimination up to and with the middle row h (one-ended factors: the last
// row), n of them; then back substitution from the row before it, the other
// way, down to row lo (end 0) or up to row hi (end 1), nb of them.
template <int ENDS>
struct EndSteps {
  int h, first, dir, n, nb;
  bool top;
  __device__ EndSteps(int by, int end, int lo, int hi)
      : h(ENDS == 2 ? by / 2 : by - 1), top(ENDS == 2 && end != 0) {
    first = top ? by - 1 : 0;
    dir = top ? -1 : 1;
    n = (top ? by - 1 - h : h) + 1;
    nb = top ? hi - h : h - lo;
  }
};

// Block LDL^T solve of one box by the group of one end; us holds b on
// entry and x on exit in rows lo .. hi (by rows of bx words, LDS, shared by the
// groups; lo and hi are the first and the last row the caller reads, and
// rows beyond them keep their elimination values); cp holds the couplings T_j
// (LDS); vv is the group's vector slot (vec_words, zeroed); r the row lane and hf
// the half of the lane.  S is the storage
// type of the factors, T the arithmetic and vector type (FP32 factors may be
// applied in FP64 arithmetic).  A step waits for its vector's way through LDS and
// for its sums; what it reads of us and cp is fetched one step ahead.
template <typename T, typename S, int NB, bool DENSE>
__device__ __forceinline__ void box_solve(T* us, T* vv, const S* cp, const S* __restrict__ Dinv,
                                          int bx, int by, int bstride, int r, int hf, int end,
                                          int lo, int hi) {
  constexpr int V0 = Half<NB>::V0, HV = Half<NB>::HV, ENDS = box_ends<S>();
  constexpr int DEPTH = reg_depth<S, NB>();
  const EndSteps<ENDS> st(by, end, lo, hi);
  const int rc = r < bx ? r : bx - 1;
  const Mirror<NB, sizeof(T) == 8> mir(rc, hf, bx);
  const T* vo = vv + V0 + rc + 2 * hf;
  const T* vr = vv + V0 + rc + bx - 2 * hf;
  T* put = vv + V0 + rc + hf * bx;
  T* ur = us + rc;
  const S* cr = cp + rc;
  const int dx = st.dir * bx;
  T xh = T(0);
  auto product = [&](const T& y, const HalfRow<S, NB>& d, const S (&rot)[Half<NB>::NM]) {
    put[0] = y;
    if constexpr (HV == 1) put[bx] = y;
    wave_sync();
    const T acc = half_dot<T, S, NB, DENSE>(d, rot, vo, vr, hf);
    wave_sync();
    return acc;
  };
  // elimination: row j's couplings to the row before it are T_j at end 0 and
  // T_{j+1} at end 1 (none at the first row)
  {
    int at = st.first * bx, ca = (st.top && st.n > 1 ? by : 0) * bx;
    T carry = T(0), b = ur[at], c = T(0);
    pipelined_sweep<S, NB, DEPTH>(
        st.n, late_start<NB>(st.n), Dinv + st.first * bstride, st.dir * bstride,
        [&](int s, const HalfRow<S, NB>& d) {
          S rot[Half<NB>::NM];
          mirror_rows<S, NB>(rot, d, mir, hf);
          T y = fmat(c, carry, b);
          if (ENDS == 2 && s == st.n - 1) {
            pair_sync<S, NB>();  // both ends have reached the middle row
            y = b;
            if (st.h > 0) y = fmat((T)cr[st.h * bx], ur[(st.h - 1) * bx], y);
            if (st.h + 1 < by) y = fmat((T)cr[(st.h + 1) * bx], ur[(st.h + 1) * bx], y);
            pair_sync<S, NB>();  // both have read it and its neighbours
          }
          const bool run = !Half<NB>::PACK || s >= 0;  // the group has started
          // the next step's row (the last step stays on its own)
          const int on = run && s + 1 < st.n ? dx : 0, cur = at;
          at += on;
          ca += on;
          b = ur[at];
          c = run ? (T)cr[ca] : T(0);
          const T u = product(y, d, rot);
          carry = run ? u : T(0);
          if (run && !(st.top && s == st.n - 1)) ur[cur] = u;  // end 0 writes the middle row
        },
        bx, rc, hf);
    xh = carry;
  }
  // substitution: row j's couplings to the row before it are T_{j+1} at end 0 and
  // T_j at end 1
  const int late = late_start<NB>(st.nb > 0 ? st.nb : 0);
  if (st.nb > 0 || late > 0) {
    // (a group without rows stays on the middle one)
    const int row = st.nb > 0 ? st.h - st.dir : st.h;
    int at = row * bx, ca = (st.top ? row : st.h) * bx;
    T carry = xh, b = ur[at], c = (T)cr[ca];
    pipelined_sweep<S, NB, DEPTH>(
        st.nb, late, Dinv + row * bstride, -st.dir * bstride,
        [&](int s, const HalfRow<S, NB>& d) {
          S rot[Half<NB>::NM];
          mirror_rows<S, NB>(rot, d, mir, hf);
          const T y = c * carry, u = b;
          const bool run = !Half<NB>::PACK || s >= 0;
          const int on = run && s + 1 < st.nb ? dx : 0, cur = at;
          at -= on;
          ca -= on;
          b = ur[at];
          c = (T)cr[ca];
          const T x = u + product(y, d, rot);
          carry = run ? x : carry;
          if (run) ur[cur] = x;
        },
        bx, rc, hf);
  }
}

// Stage a box for its solve: rows [0, by) of a grid vector (bx cells wide,
// row lane r: column r) and the box's couplings (by rows of bx words) into LDS,
// the box's NSET sets of row lanes (halves and groups) taking runs of rows in
// turn, both arrays' loads of a run in flight at a time, so that a box of up to
// 32 rows (16 with one set) costs one memory
// latency.  Loads are unconditional (row and column clamped into the box).
template <int NSET, int RUN, typename T, typename G, typename S>
__device__ __forceinline__ void stage_box(T* dst, const G* __restrict__ src, long long origin,
                                          int nx, S* cdst, const S* __restrict__ csrc, int bx,
                                          int by, int r, int set) {
  const int col = r < bx ? r : bx - 1;
  const bool act = r < bx;
  for (int jj = 0; jj < by; jj += RUN * NSET) {
    const int j0 = jj + RUN * set;
    G v[RUN];
    S c[RUN];
#pragma unroll
    for (int u = 0; u < RUN; ++u) {
      const int j = j0 + u < by ? j0 + u : by - 1;
      v[u] = src[origin + (long long)j * nx + col];
      c[u] = csrc[j * bx + col];
    }
#pragma unroll
    for (int u = 0; u < RUN; ++u)
      if (act && j0 + u < by) {
        dst[(j0 + u) * bx + r] = (T)v[u];
        cdst[(j0 + u) * bx + r] = c[u];
      }
  }
}

// Copy count (>= 1) contiguous words from global memory into LDS with a
// box's NL lanes, RUN unconditional loads in flight per lane at a time.
template <typename S, int NL, int RUN>
__device__ __forceinline__ void words_to_lds(S* dst, const S* __restrict__ src, int count,
                                             int lane) {
  for (int q0 = 0; q0 < count; q0 += RUN * NL) {
    S v[RUN];
#pragma unroll
    for (int u = 0; u < RUN; ++u) {
      const int q = q0 + u * NL + lane;
      v[u] = src[q < count ? q : count - 1];
    }
#pragma unroll
    for (int u = 0; u < RUN; ++u) {
      const int q = q0 + u * NL + lane;
      if (q < count) dst[q] = v[u];
    }
  }
}

// LDS slot of one box:
//   vv[ends][vec_words] (T) | cp[max cells] (S) | us[max cells] (T),
// every part 16-byte aligned; cp_words (the coupling area, also the trace
// moments' buffer) is a multiple of 16 bytes.
template <typename T, typename S, int NB>
struct BoxSlot {
  T* vv;
  S* cp;
  T* us;
  __device__ BoxSlot(char* base, int cp_words, int end) {
    constexpr int VW = vec_words<NB>(), ENDS = box_ends<S>();
    vv = reinterpret_cast<T*>(base) + end * VW;
    cp = reinterpret_cast<S*>(base + ENDS * VW * sizeof(T));
    us = reinterpret_cast<T*>(base + ENDS * VW * sizeof(T) + (long long)cp_words * sizeof(S));
  }
};

// The box of a thread in a launch of the box kernels: the box index (clamped:
// groups past the last box, live = false, run along on it in their own slot and
// write nothing outside), the end its group (wave) works on, its row lane r and
// half hf; lane: its index among the box's NL threads, set: among the
// box's sets of row lanes.
template <typename S, int NB>
struct BoxThread {
  static constexpr int R = Half<NB>::R, HV = Half<NB>::HV, GL = Half<NB>::GL;
  static constexpr int ENDS = box_ends<S>(), NL = ENDS * GL, NSET = ENDS * HV;
  // rows that a set stages at a time: 32 in all, with one set or for the narrowest 16
  static constexpr int RUN = NSET == 4 || (NB == kPacked16 && NSET == 2) ? 8 : 16;
  int slot, end, lane, r, hf, set, i;
  bool live;
  __device__ BoxThread(int block, int m) {
    int g = threadIdx.x / GL;
    if constexpr (GL == 64) g = __builtin_amdgcn_readfirstlane(g);
    const int l = threadIdx.x % GL;
    slot = g / ENDS;
    end = g % ENDS;
    lane = end * GL + l;
    r = l % R;
    hf = l / R;
    set = end * HV + hf;
    const int i0 = block * (int)(blockDim.x / NL) + slot;
    live = i0 < m;
    i = live ? i0 : m - 1;
  }
  // The most faces of a subdomain among the workgroup's boxes (the same in every
  // thread, so that loops with workgroup barriers run the same rounds in all waves).
  __device__ int faces(const BoxDesc* __restrict__ boxes, int block, int m) const {
    constexpr bool waves = ENDS == 2 && GL == 64;  // a box is two waves
    const int n = waves ? (int)(blockDim.x / NL) : 1, i0 = waves ? block * n : i;
    int most = 0;
    for (int q = 0; q < n; ++q) {
      const BoxDesc& d = boxes[i0 + q < m ? i0 + q : m - 1];
      const int f = 2 * (d.obx + d.oby);
      most = f > most ? f : most;
    }
    return most;
  }
};
// First and last row of the box that the owned rows' traces read: one beyond
// the owned rows on either side, inside the box.
__device__ __forceinline__ int trace_lo(const BoxDesc& d) { return d.oy > 0 ? d.oy - 1 : 0; }
__device__ __forceinline__ int trace_hi(const BoxDesc& d) {
  return d.oy + d.oby < d.by ? d.oy + d.oby : d.by - 1;
}

// Legendre polynomial P_q at xi (three-term recurrence).
__device__ __forceinline__ double legendre_at(int q, double xi) {
  double pm = 1.0, pq = xi;
  if (q == 0) return 1.0;
  for (int k = 1; k < q; ++k) {
    const double pn = ((2.0 * k + 1.0) * xi * pq - k * pm) / (k + 1.0);
    pm = pq;
    pq = pn;
  }
  return pq;
}

// Box-local indices (row stride d.bx) of the two cells of face j of side
// `side` (W E S N) of the owned subdomain of box d: the subdomain's cell and
// the cell across the face.  A face on the box's boundary (no oversampling)
// has no cell across inside the box; its second index is the first (the
// weights of that cell are zero).
__device__ __forceinline__ void face_cells(const BoxDesc& d, int side, int j, int& cin,
                                           int& cout) {
  int row, col, dr = 0, dc = 0;
  if (side == 0) {
    row = d.oy + j; col = d.ox; dc = -1;
  } else if (side == 1) {
    row = d.oy + j; col = d.ox + d.obx - 1; dc = 1;
  } else if (side == 2) {
    row = d.oy; col = d.ox + j; dr = -1;
  } else {
    row = d.oy + d.oby - 1; col = d.ox + j; dr = 1;
  }
  cin = row * d.bx + col;
  const int r2 = row + dr, c2 = col + dc;
  cout = (r2 < 0 || r2 >= d.by || c2 < 0 || c2 >= d.bx) ? cin : r2 * d.bx + c2;
}

// Flux and pressure moments of the coarse dofs k = (i, side, q) of a subdomain
// over the faces of their sides: sum_j P_q(xi_j) (cUi p_in + cUo p_out) and
// likewise with the pressure weights; face_w: the four weights of each face, the
// subdomain's faces side after side.  v(k, c) reads the solution of column k at
// box-local cell c; the K columns share what a face needs, their moments are nc apart.
// The box's NL threads take a face each (flux, pressure and xi_j into buf,
// 3 NL words of LDS), then one thread per dof adds its side's faces in order:
// the divisions, weights and cells of all faces cost one pass instead of one per
// face and dof (14 of k_local's 89 us at 1024^2 in FP64, 8 of 33 us at 505 x 387,
// were this serial; 768 x 768 in 8-wide subdomains, where all lanes are busy, 269 us of T
// with a search of the dofs for a face's side, 263 with the sides' places).
// The rounds over the faces go to `span`, the workgroup's most (BoxThread::faces): all its
// waves meet at the same barriers, whatever their boxes' sides.  A subdomain has at most
// 36 dofs (four sides, degree 8): one per thread, unless packed.
template <typename S, int NB, int K, typename V>
__device__ __forceinline__ void trace_moments(const BoxDesc& d, int nx, int lane, bool live,
                                              int span, const int* __restrict__ dof_side,
                                              const int* __restrict__ dof_q,
                                              const int* __restrict__ dof_face0, int k0, int nd,
                                              const double* __restrict__ face_w, double* buf,
                                              V v, double* __restrict__ mU,
                                              double* __restrict__ mP, long long nc) {
  constexpr int NL = BoxThread<S, NB>::NL;
  const int f0 = dof_face0[k0];
  const int last = dof_face0[k0 + nd - 1] - f0 +
                   (dof_side[k0 + nd - 1] <= 1 ? d.oby : d.obx);  // faces of the subdomain
  // the sides W, E, S, N that have faces (those inside the grid), one after the other
  const int xw = d.x0 + d.ox, west = xw > 0 ? d.oby : 0;
  const int east = west + (xw + d.obx < nx ? d.oby : 0);
  const int south = east + (d.y0 + d.oy > 0 ? d.obx : 0);
  for (int kb = 0; kb < (NL >= 64 ? 1 : nd); kb += NL) {
    const bool mine = kb + lane < nd;
    const int dof = k0 + (mine ? kb + lane : 0);
    const int side = dof_side[dof], q = dof_q[dof], len = side <= 1 ? d.oby : d.obx;
    const int fa = dof_face0[dof] - f0;
    double su[K], sp[K];
#pragma unroll
    for (int k = 0; k < K; ++k) su[k] = sp[k] = 0.0;
    for (int base = 0; base < span; base += NL) {
      const int f = base + lane;
      f64x2 wu = {0.0, 0.0}, wp = {0.0, 0.0};
      int ci = 0, co = 0;
      if (f < last) {
        const int fs = f < west ? 0 : f < east ? 1 : f < south ? 2 : 3;
        const int fb = fs == 0 ? 0 : fs == 1 ? west : fs == 2 ? east : south;
        const f64x2* w = reinterpret_cast<const f64x2*>(face_w + 4LL * (f0 + f));
        wu = w[0];
        wp = w[1];
        const int j = f - fb;
        face_cells(d, fs, j, ci, co);
        buf[2 * NL + lane] = (2.0 * j + 1.0) / (fs <= 1 ? d.oby : d.obx) - 1.0;
      }
      const int a = fa > base ? fa : base;
      const int b = fa + len < base + NL ? fa + len : base + NL;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (f < last) {
          const double pin = v(k, ci), pout = v(k, co);
          buf[lane] = fmat(wu[1], pout, wu[0] * pin);
          buf[NL + lane] = fmat(wp[1], pout, wp[0] * pin);
        }
        pair_sync<S, NB>();
        if (mine) {
          for (int t = a; t < b; ++t) {
            const double lw = legendre_at(q, buf[2 * NL + t - base]);
            su[k] = fmat(lw, buf[t - base], su[k]);
            sp[k] = fmat(lw, buf[NL + t - base], sp[k]);
          }
        }
        pair_sync<S, NB>();
      }
    }
    if (mine && live) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        mU[k * nc + dof] = su[k];
        mP[k * nc + dof] = sp[k];
      }
    }
  }
}

// Source-driven solves of the apply: the
// oversampled problem on hat-Omega_i (box d) with source r and zero Robin
// data, p = its restriction to Omega_i (the owned cells of d), fused with
// the trace moments of the coarse right-hand side (FP64 sums).
template <typename T, typename S, int NB, bool DENSE>
__device__ __forceinline__ void local_body(
    const Blk blk, const BoxDesc* __restrict__ boxes, int m, int group_bytes, int cp_words,
    const S* __restrict__ dinv, const S* __restrict__ coup, const double* __restrict__ r,
    T* __restrict__ p, int nx, const int* __restrict__ dof_off,
    const int* __restrict__ dof_side, const int* __restrict__ dof_q,
    const int* __restrict__ dof_face0, const double* __restrict__ face_w,
    double* __restrict__ mU, double* __restrict__ mP) {
  extern __shared__ __align__(16) char smem_raw[];
  typedef BoxThread<S, NB> BT;
  const BT t(blk.id, m);
  BoxSlot<T, S, NB> L(smem_raw + (long long)t.slot * group_bytes, cp_words, t.end);
  const BoxDesc d = boxes[t.i];
  const int bx = d.bx, by = d.by;
  const long long origin = (long long)d.y0 * nx + d.x0;
  stage_box<BT::NSET, BT::RUN>(L.us, r, origin, nx, L.cp, coup + d.coff, bx, by, t.r, t.set);
  zero_slots<BT::GL>(L.vv, vec_words<NB>());
  pair_sync<S, NB>();
  if (d.pin) {  // one box covers the grid: the same in every group
    if (t.lane == 0) L.us[0] = T(0);
    pair_sync<S, NB>();
  }
  box_solve<T, S, NB, DENSE>(L.us, L.vv, L.cp, dinv + d.doff, bx, by, d.bs, t.r, t.hf, t.end,
                            trace_lo(d), trace_hi(d));
  pair_sync<S, NB>();
  if (t.live && t.r >= d.ox && t.r < d.ox + d.obx) {
    const long long o2 = origin + (long long)d.oy * nx;
    for (int j = t.set; j < d.oby; j += BT::NSET)
      p[o2 + (long long)j * nx + t.r] = L.us[(d.oy + j) * bx + t.r];
  }
  const int k0 = dof_off[t.i], nd = dof_off[t.i + 1] - k0;
  if (nd > 0)  // none where one subdomain is the grid, the only box then
    trace_moments<S, NB, 1>(d, nx, t.lane, t.live, t.faces(boxes, blk.id, m), dof_side, dof_q,
                            dof_face0, k0, nd, face_w, reinterpret_cast<double*>(L.cp),
                            [&](int, int c) { return (double)L.us[c]; }, mU, mP, 0);
}
template <typename T, typename S, int NB, bool DENSE>
__global__ void MRCM_BOX_KERNEL(T, S, NB, DENSE)
    k_local(const BoxDesc* __restrict__ boxes, int m, int group_bytes, int cp_words,
            const S* __restrict__ dinv, const S* __restrict__ coup,
            const double* __restrict__ r, T* __restrict__ p, int nx,
            const int* __restrict__ dof_off, const int* __restrict__ dof_side,
            const int* __restrict__ dof_q, const int* __restrict__ dof_face0,
            const double* __restrict__ face_w, double* __restrict__ mU,
            double* __restrict__ mP) {
  local_body<T, S, NB, DENSE>(hw_blk(), boxes, m, group_bytes, cp_words, dinv, coup, r, p, nx,
                             dof_off, dof_side, dof_q, dof_face0, face_w, mU, mP);
}

// Interface right-hand side in tree order: for tree position t, gsrc[t] =
// {L, R, kind}: kind 0 a flux row, g = -(mU[L] + mU[R]); 1 a pressure row,
// g = -(mP[L] - mP[R]); 2 the replaced row of an all-no-flow grid, g = 0;
// times the row's equilibration scale gscale[t].
__device__ __forceinline__ void coarse_rhs_body(const Blk blk, const int4* __restrict__ gsrc,
                                                const double* __restrict__ gscale,
                                                const double* __restrict__ mU,
                                                const double* __restrict__ mP,
                                                double* __restrict__ g_nd, int np) {
  const int t = blk.id * blockDim.x + threadIdx.x;
  if (t >= np) return;
  const int4 src = gsrc[t];
  const double v = src.z == 0 ? -(mU[src.x] + mU[src.y]) : -(mP[src.x] - mP[src.y]);
  g_nd[t] = src.z == 2 ? 0.0 : gscale[t] * v;
}
__global__ void k_coarse_rhs(const int4* __restrict__ gsrc, const double* __restrict__ gscale,
                             const double* __restrict__ mU, const double* __restrict__ mP,
                             double* __restrict__ g_nd, int np) {
  coarse_rhs_body(hw_blk(), gsrc, gscale, mU, mP, g_nd, np);
}

// Refinement residual of the interface solve in tree order: r_nd[t] = g_nd[t]
// - sum over the scaled row of position t of v * x (CSR rp / ci / v), one
// thread per row, terms in row order; blockIdx.y selects a column of a
// multi-column solve (vectors of column k at k * np / k * nc).
__device__ __forceinline__ void coarse_resid_body(const Blk blk, int col,
                                                  const int* __restrict__ rp,
                                                  const int* __restrict__ ci,
                                                  const double* __restrict__ v,
                                                  const double* __restrict__ g_nd,
                                                  const double* __restrict__ x,
                                                  double* __restrict__ r_nd, int np, int nc) {
  const int t = blk.id * blockDim.x + threadIdx.x;
  if (t >= np) return;
  const double* xk = x + (long long)col * nc;
  double s = g_nd[(long long)col * np + t];
  for (int q = rp[t]; q < rp[t + 1]; ++q) s = fmat(-v[q], xk[ci[q]], s);
  r_nd[(long long)col * np + t] = s;
}
__global__ void k_coarse_resid(const int* __restrict__ rp, const int* __restrict__ ci,
                               const double* __restrict__ v, const double* __restrict__ g_nd,
                               const double* __restrict__ x, double* __restrict__ r_nd, int np,
                               int nc) {
  coarse_resid_body(hw_blk(), blockIdx.y, rp, ci, v, g_nd, x, r_nd, np, nc);
}

// x += dx over n values (columns of a multi-column solve are consecutive).
__device__ __forceinline__ void coarse_add_body(const Blk blk, double* __restrict__ x,
                                                const double* __restrict__ dx, long long n) {
  const long long q = blk.id * (long long)blockDim.x + threadIdx.x;
  if (q < n) x[q] += dx[q];
}
__global__ void k_coarse_add(double* __restrict__ x, const double* __restrict__ dx, long long n) {
  coarse_add_body(hw_blk(), x, dx, n);
}

// ---- interface solve (level-scheduled nested dissection) -------------------
// One launch per tree level and direction; a workgroup takes one chunk, rows
// [row0, row1) of one node's matrix (see device.h).  Each wave takes groups
// of four rows (wave w: rows row0 + 4 w + 16 k); lanes stride the columns
// eight deep, so a wave has 32 matrix loads in flight.  The first group's
// loads are issued before the right-hand side is gathered, so their latency
// overlaps the gather (except at the root of a large tree, whose long gather
// goes first).

// Entries of a node's vector a thread gathers into LDS at a time: a root
// separator of more than kWideRoot rows (kGatherA), a backward border (up to
// kGatherB, as its length needs).
constexpr int kGatherA = 4;
constexpr int kGatherB = 8;
constexpr int kWideRoot = 1024;

// Issue the loads of one 4 x (8 x 64) tile: rows r .. r + 3 (clipped at
// row1), columns b0 + 64 q (clipped at ncol); missing entries read as zero.
__device__ __forceinline__ void load_tile(double (&m)[4][8], const double* __restrict__ M,
                                          int ncol, int r, int row1, int b0) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int b = b0 + 64 * q;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      m[u][q] = (b < ncol && r + u < row1) ? M[(long long)(r + u) * ncol + b] : 0.0;
  }
}

// s[u] += sum_q m[u][q] vec[b0 + 64 q] (vector in LDS).
__device__ __forceinline__ void fma_tile(double (&s)[4], const double (&m)[4][8],
                                         const double* vec, int ncol, int b0) {
  double x[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) x[q] = b0 + 64 * q < ncol ? vec[b0 + 64 * q] : 0.0;
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] = fmat(m[u][q], x[q], s[u]);
}

// Rows [row0, row1) of M (row-major, ncol columns) times the LDS vector; the
// tile m holds this wave's first tile (rows row0 + 4 wid, columns lane ..),
// and pre(row0 + 4 wid) has already been called.  For every later group of
// four rows r .. r + 3, pre(r) is called first (lane u may fetch what it
// needs for row r + u); then emit(r + u, value) runs in lane u.
template <typename Pre, typename Emit>
__device__ __forceinline__ void gemv_chunk(const double* __restrict__ M, int ncol, int row0,
                                           int row1, const double* vec, double (&m)[4][8],
                                           Pre pre, Emit emit) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int r = row0 + 4 * wid; r < row1; r += 4 * nw) {
    const bool first = r == row0 + 4 * wid;
    if (!first) pre(r);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    fma_tile(s, m, vec, ncol, lane);
    for (int b0 = lane + 64 * 8; b0 < ncol; b0 += 64 * 8) {
      load_tile(m, M, ncol, r, row1, b0);
      fma_tile(s, m, vec, ncol, b0);
    }
    if (r + 4 * nw < row1) load_tile(m, M, ncol, r + 4 * nw, row1, lane);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double t = wave_sum(s[u]);
      if (lane == u && r + u < row1) emit(r + u, t);
    }
  }
}

// Sums of N values (a power of two, 2..64) over the 64 lanes of the wave, all
// at once: at the exchange with lane ^ off (off = 32, 16, ..., 1) a lane
// keeps half of its values, and the sum of each kept value is its own plus
// the partner's, so every value meets the pairs of wave_sum in the same order
// (each result is bit-identical to wave_sum of that value) with 2N - 1 + 6 -
// log2 N exchanges instead of 6 N.  Afterwards v[0] in lane l is the sum of
// value butterfly_index<N>(l).
template <int N>
__device__ __forceinline__ int butterfly_index(int lane) {
  int idx = 0, n = N;
#pragma unroll
  for (int off = 32; off > 0 && n > 1; off >>= 1) {
    n >>= 1;
    if (lane & off) idx += n;
  }
  return idx;
}
template <int N>
__device__ __forceinline__ void butterfly_sum(double (&v)[N], int lane) {
#pragma unroll
  for (int st = 0; st < 6; ++st) {
    const int off = 32 >> st;
    const int n = N >> st;  // values still held (compile-time after unrolling)
    if (n > 1) {
      const int half = n >> 1;
      const bool upper = (lane & off) != 0;
#pragma unroll
      for (int i = 0; i < N / 2; ++i)
        if (i < half) {
          const double send = upper ? v[i] : v[i + half];
          const double keep = upper ? v[i + half] : v[i];
          v[i] = keep + __shfl_xor(send, off, 64);
        }
    } else {
      v[0] += __shfl_xor(v[0], off, 64);
    }
  }
}

// A chunk of at most 16 rows and ncol <= 128 columns taken whole by one
// wave: lane l loads columns l and l + 64 of every row, all at once, and the
// sixteen row sums are reduced together; afterwards lane l holds the sum of
// row row0 + butterfly_index<16>(l).  Each lane's partial sums and the
// reduction tree are those of gemv_chunk, so the results are the same.
__device__ __forceinline__ void load_chunk16(double (&m)[16][2], const double* __restrict__ M,
                                             int ncol, int row0, int row1, int lane) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int b = lane + 64 * q;
#pragma unroll
    for (int u = 0; u < 16; ++u)
      m[u][q] = (b < ncol && row0 + u < row1) ? M[(long long)(row0 + u) * ncol + b] : 0.0;
  }
}
__device__ __forceinline__ double gemv_chunk16(const double (&m)[16][2], const double* vec,
                                               int ncol, int lane) {
  double x[2], s[16];
#pragma unroll
  for (int q = 0; q < 2; ++q) x[q] = lane + 64 * q < ncol ? vec[lane + 64 * q] : 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) s[u] = 0.0;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int u = 0; u < 16; ++u) s[u] = fmat(m[u][q], x[q], s[u]);
  butterfly_sum<16>(s, lane);
  return s[0];
}
// Whether a forward chunk is taken whole, 16 rows per wave (wave w: rows
// row0 + 16 w .. row0 + 16 w + 15) with every row's columns in the wave's
// registers.
__device__ __forceinline__ bool whole_chunk(const CChunk& ch, int ncol) {
  return ncol <= 128 && ch.row1 - ch.row0 <= 16 * (int)(blockDim.x >> 6);
}
// Whether a backward chunk is taken whole by a one-wave workgroup.
__device__ __forceinline__ bool whole_chunk_wave(const CChunk& ch, int ncol) {
  return blockDim.x == 64 && ncol <= 128 && ch.row1 - ch.row0 <= 16;
}

// Forward level: for the separator rows a of the chunk's node (tree
// positions t = yoff + a),
//   v[a] = g_nd[t] - (contributions of the descendants, in slot order),
// with the contributions by destination in contrib[u * np + t] (slot u,
// zero where unused).  Then rows of [W; E] v: y_F into ybuf (straight into
// x through idx for a node without border rows, whose x_F = y_F), each c_n
// row into its destination slot cdest[coff + row - nf].
__device__ __forceinline__ void coarse_fwd_body(
    const CChunk ch, const double* __restrict__ fwd, const double* __restrict__ g_nd,
    double* __restrict__ contrib, int maxp, int np, const int* __restrict__ cdest,
    double* __restrict__ ybuf, const int* __restrict__ idx, double* __restrict__ x) {
  extern __shared__ double v[];
  const int nf = ch.nf, lane = threadIdx.x & 63;
  const double* M = fwd + ch.mat;
  const int yoff = ch.yoff, coff = ch.coff;
  int dst = -1;
  // v[a] = g_nd[t] minus the contributions in slot order; a thread takes
  // its entries A at a time, with all their loads in flight together
  auto gather_rows = [&](auto A) {
    constexpr int kA = decltype(A)::value, kC = kA > 1 ? 4 : 8;
    const int bd = blockDim.x;
    for (int a0 = threadIdx.x; a0 < nf; a0 += kA * bd) {
      long long t[kA];
      double s[kA];
#pragma unroll
      for (int i = 0; i < kA; ++i) {
        const int a = a0 + i * bd;
        t[i] = (long long)yoff + (a < nf ? a : nf - 1);
        s[i] = g_nd[t[i]];
      }
      for (int u0 = 0; u0 < maxp; u0 += kC) {
        double c[kA][kC];
#pragma unroll
        for (int i = 0; i < kA; ++i)
#pragma unroll
          for (int k = 0; k < kC; ++k)
            c[i][k] = u0 + k < maxp ? contrib[(long long)(u0 + k) * np + t[i]] : 0.0;
#pragma unroll
        for (int i = 0; i < kA; ++i)
#pragma unroll
          for (int k = 0; k < kC; ++k)
            if (u0 + k < maxp) s[i] -= c[i][k];
      }
#pragma unroll
      for (int i = 0; i < kA; ++i)
        if (a0 + i * bd < nf) v[a0 + i * bd] = s[i];
    }
    __syncthreads();
  };
  auto gather = [&]() { gather_rows(std::integral_constant<int, 1>()); };
  auto emit = [&](int row, double val) {
    if (row >= nf)
      contrib[dst] = val;
    else if (ch.nu == 0)
      x[idx[ch.fcol + row]] = val;  // a node without border rows: x_F = y_F
    else
      ybuf[yoff + row] = val;
  };
  if (whole_chunk(ch, nf)) {
    const int r0 = ch.row0 + 16 * (int)(threadIdx.x >> 6);
    double m[16][2];
    load_chunk16(m, M, nf, r0, ch.row1, lane);
    const int row = r0 + butterfly_index<16>(lane);
    dst = (row >= nf && row < ch.row1) ? cdest[coff + row - nf] : -1;
    gather();
    const double val = gemv_chunk16(m, v, nf, lane);
    if ((lane & 3) == 0 && row < ch.row1) emit(row, val);
    return;
  }
  auto pre = [&](int r) {
    const int row = r + lane;
    dst = (lane < 4 && row >= nf && row < ch.row1) ? cdest[coff + row - nf] : -1;
  };
  double m[4][8];
  const int rw = ch.row0 + 4 * (threadIdx.x >> 6);
  if (ch.nu == 0 && nf > kWideRoot) {
    // the root of a large tree: few workgroups, each with a long gather,
    // which goes first, kGatherA entries deep (the tile's registers are
    // not live yet, so the kernel's occupancy holds)
    gather_rows(std::integral_constant<int, kGatherA>());
    load_tile(m, M, nf, rw, ch.row1, lane);
    pre(rw);
  } else {
    load_tile(m, M, nf, rw, ch.row1, lane);
    pre(rw);
    gather();
  }
  gemv_chunk(M, nf, ch.row0, ch.row1, v, m, pre, emit);
}
__global__ void __launch_bounds__(kVecThreads)
    k_coarse_fwd(const CChunk* __restrict__ chunks, const double* __restrict__ fwd,
                 const double* __restrict__ g_nd, double* __restrict__ contrib, int maxp, int np,
                 const int* __restrict__ cdest, double* __restrict__ ybuf,
                 const int* __restrict__ idx, double* __restrict__ x) {
  coarse_fwd_body(chunks[blockIdx.x], fwd, g_nd, contrib, maxp, np, cdest, ybuf, idx, x);
}

// Backward level: x_F = y_F - G x_U for the chunk's rows (x_U gathered
// through idx[ucol ..], x_F scattered through idx[fcol ..]; nu > 0).
__device__ __forceinline__ void coarse_bwd_body(const CChunk ch, const double* __restrict__ bwd,
                                                const int* __restrict__ idx,
                                                const double* __restrict__ ybuf,
                                                double* __restrict__ x) {
  extern __shared__ double xu[];
  const int nu = ch.nu, lane = threadIdx.x & 63;
  const double* M = bwd + ch.mat;
  const int yoff = ch.yoff, fcol = ch.fcol;
  int dst = 0;
  double y = 0.0;
  // xu[b] = x[idx[ucol + b]]: a thread takes its entries R at a time, all
  // their loads in flight together, R being 1, 2, 4 or kGatherB as the
  // border needs (it is the same in the whole workgroup)
  auto gather_r = [&](auto R) {
    constexpr int kR = decltype(R)::value;
    const int bd = blockDim.x;
    for (int b0 = threadIdx.x; b0 < nu; b0 += kR * bd) {
      int k[kR];
      double val[kR];
#pragma unroll
      for (int i = 0; i < kR; ++i) {
        const int b = b0 + i * bd;
        k[i] = idx[ch.ucol + (b < nu ? b : nu - 1)];
      }
#pragma unroll
      for (int i = 0; i < kR; ++i) val[i] = x[k[i]];
#pragma unroll
      for (int i = 0; i < kR; ++i)
        if (b0 + i * bd < nu) xu[b0 + i * bd] = val[i];
    }
    __syncthreads();
  };
  auto gather = [&]() {
    const int rounds = (nu + (int)blockDim.x - 1) / (int)blockDim.x;
    if (rounds <= 1)
      gather_r(std::integral_constant<int, 1>());
    else if (rounds <= 2)
      gather_r(std::integral_constant<int, 2>());
    else if (rounds <= 4)
      gather_r(std::integral_constant<int, 4>());
    else
      gather_r(std::integral_constant<int, kGatherB>());
  };
  if (whole_chunk_wave(ch, nu)) {
    double m[16][2];
    load_chunk16(m, M, nu, ch.row0, ch.row1, lane);
    const int row = ch.row0 + butterfly_index<16>(lane);
    if (row < ch.row1) {
      dst = idx[fcol + row];
      y = ybuf[yoff + row];
    }
    gather();
    const double val = gemv_chunk16(m, xu, nu, lane);
    if ((lane & 3) == 0 && row < ch.row1) x[dst] = y - val;
    return;
  }
  auto pre = [&](int r) {
    const int row = r + lane;
    if (lane < 4 && row < ch.row1) {
      dst = idx[fcol + row];
      y = ybuf[yoff + row];
    }
  };
  double m[4][8];
  const int rw = ch.row0 + 4 * (threadIdx.x >> 6);
  load_tile(m, M, nu, rw, ch.row1, lane);
  pre(rw);
  gather();
  gemv_chunk(M, nu, ch.row0, ch.row1, xu, m, pre, [&](int, double val) { x[dst] = y - val; });
}
__global__ void __launch_bounds__(kVecThreads)
    k_coarse_bwd(const CChunk* __restrict__ chunks, const double* __restrict__ bwd,
                 const int* __restrict__ idx, const double* __restrict__ ybuf,
                 double* __restrict__ x) {
  coarse_bwd_body(chunks[blockIdx.x], bwd, idx, ybuf, x);
}

// p[Omega_i] += P_i x_i (multiscale reconstruction; Omega_i is the owned part
// of box d), one workgroup per subdomain.
template <typename T, typename S>
__device__ __forceinline__ void reconstruct_body(const Blk blk, const BoxDesc* __restrict__ boxes,
                                                 const S* __restrict__ mbf,
                                                 const long long* __restrict__ mbf_off,
                                                 const int* __restrict__ dof_off,
                                                 const double* __restrict__ xc,
                                                 T* __restrict__ p, int nx) {
  __shared__ T xs[64];
  const int i = blk.id;
  const BoxDesc d = boxes[i];
  const int k0 = dof_off[i], nk = dof_off[i + 1] - k0, ncell = d.obx * d.oby;
  for (int k = threadIdx.x; k < nk; k += blockDim.x) xs[k] = (T)xc[k0 + k];
  __syncthreads();
  const S* P = mbf + mbf_off[i];
  for (int q = threadIdx.x; q < ncell; q += blockDim.x) {
    const int a = q % d.obx, j = q / d.obx;
    const long long c = (long long)(d.y0 + d.oy + j) * nx + d.x0 + d.ox + a;
    T s = p[c];
    for (int k = 0; k < nk; ++k) s = fmat((T)P[(long long)k * ncell + q], xs[k], s);
    p[c] = s;
  }
}
template <typename T, typename S>
__global__ void __launch_bounds__(kBoxThreads)
    k_reconstruct(const BoxDesc* __restrict__ boxes, const S* __restrict__ mbf,
                  const long long* __restrict__ mbf_off, const int* __restrict__ dof_off,
                  const double* __restrict__ xc, T* __restrict__ p, int nx) {
  reconstruct_body<T, S>(hw_blk(), boxes, mbf, mbf_off, dof_off, xc, p, nx);
}

// Smoothing residual rho = r - A p.
template <typename T>
__device__ __forceinline__ void residual_body(const Blk blk, const T* __restrict__ tx,
                                              const T* __restrict__ ty, int nx, int ny,
                                              const double* __restrict__ r,
                                              const T* __restrict__ p, T* __restrict__ rho) {
  const long long n = (long long)nx * ny;
  for (long long c = blk.id * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)blk.n * blockDim.x) {
    const int iy = (int)(c / nx), ix = (int)(c - (long long)iy * nx);
    rho[c] = (T)r[c] - stencil(tx, ty, nx, ny, ix, iy, p);
  }
}
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_residual(const T* __restrict__ tx, const T* __restrict__ ty, int nx, int ny,
               const double* __restrict__ r, const T* __restrict__ p, T* __restrict__ rho) {
  residual_body<T>(hw_blk(), tx, ty, nx, ny, r, p, rho);
}

// Restricted additive Schwarz: solve A[S_i] e = rho[S_i] on patch i
// and add e on the owned subdomain Omega_i (each cell
// is written by one patch only).
template <typename T, typename S, int NB, bool DENSE>
__device__ __forceinline__ void patch_body(const Blk blk, const BoxDesc* __restrict__ boxes,
                                           int m, int group_bytes, int cp_words,
                                           const S* __restrict__ dinv,
                                           const S* __restrict__ coup,
                                           const T* __restrict__ rho, T* __restrict__ p,
                                           int nx) {
  extern __shared__ __align__(16) char smem_raw[];
  typedef BoxThread<S, NB> BT;
  const BT t(blk.id, m);
  BoxSlot<T, S, NB> L(smem_raw + (long long)t.slot * group_bytes, cp_words, t.end);
  const BoxDesc d = boxes[t.i];
  const int bx = d.bx, by = d.by;
  const long long origin = (long long)d.y0 * nx + d.x0;
  stage_box<BT::NSET, BT::RUN>(L.us, rho, origin, nx, L.cp, coup + d.coff, bx, by, t.r, t.set);
  zero_slots<BT::GL>(L.vv, vec_words<NB>());
  pair_sync<S, NB>();
  if (d.pin) {  // one box covers the grid: the same in every group
    if (t.lane == 0) L.us[0] = T(0);
    pair_sync<S, NB>();
  }
  box_solve<T, S, NB, DENSE>(L.us, L.vv, L.cp, dinv + d.doff, bx, by, d.bs, t.r, t.hf, t.end,
                            d.oy, d.oy + d.oby - 1);
  pair_sync<S, NB>();
  // p += e on the owned cells, each set of row lanes a run of rows in turn, all
  // of a run's read-modify-writes in flight
  constexpr int RUN = BT::RUN == 8 ? 4 : BT::NSET == 2 ? 8 : 16;
  const bool own = t.live && t.r >= d.ox && t.r < d.ox + d.obx;
  const int col = own ? t.r : d.ox;
  const long long o2 = origin + (long long)d.oy * nx;
  const int rows = d.oby;
  for (int jj = 0; jj < rows; jj += RUN * BT::NSET) {
    const int j0 = jj + RUN * t.set;
    T v[RUN];
#pragma unroll
    for (int u = 0; u < RUN; ++u) {
      const int j = j0 + u < d.oby ? j0 + u : d.oby - 1;
      v[u] = p[o2 + (long long)j * nx + col];
    }
#pragma unroll
    for (int u = 0; u < RUN; ++u)
      if (own && j0 + u < d.oby)
        p[o2 + (long long)(j0 + u) * nx + t.r] = v[u] + L.us[(d.oy + j0 + u) * bx + t.r];
  }
}
template <typename T, typename S, int NB, bool DENSE>
__global__ void MRCM_BOX_KERNEL(T, S, NB, DENSE)
    k_patch(const BoxDesc* __restrict__ boxes, int m, int group_bytes, int cp_words,
            const S* __restrict__ dinv, const S* __restrict__ coup, const T* __restrict__ rho,
            T* __restrict__ p, int nx) {
  patch_body<T, S, NB, DENSE>(hw_blk(), boxes, m, group_bytes, cp_words, dinv, coup, rho, p, nx);
}

template <typename T>
__device__ __forceinline__ void sum_body(const Blk blk, const T* __restrict__ p, long long n,
                                         double* __restrict__ partials) {
  __shared__ double red[kVecThreads / 64];
  const long long st = (long long)blk.n * blockDim.x;
  double s = 0.0;
  for (long long c0 = blk.id * (long long)blockDim.x + threadIdx.x; c0 < n;
       c0 += kRound * st) {
    T a[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      a[u] = p[c < n ? c : n - 1];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u)
      if (c0 + u * st < n) s += (double)a[u];
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) partials[blk.id] = s;
}
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_sum(const T* __restrict__ p, long long n, double* __restrict__ partials) {
  sum_body<T>(hw_blk(), p, n, partials);
}

// z = p - mean(p) (no-flow) or z = p, in FP64.  First round loaded before
// the reduction, as in k_mgs_step.
template <typename T>
__device__ __forceinline__ void finalize_body(const Blk blk, const T* __restrict__ p, long long n,
                                              const double* __restrict__ partials, int nb,
                                              double* __restrict__ z) {
  __shared__ double red[kVecThreads / 64];
  const long long st = (long long)blk.n * blockDim.x;
  T a[kRound];
  auto load = [&](long long c0) {
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      a[u] = p[c < n ? c : n - 1];
    }
  };
  const long long start = blk.id * (long long)blockDim.x + threadIdx.x;
  load(start);
  const double mean = partials ? reduce_partials(partials, nb, red) / (double)n : 0.0;
  for (long long c0 = start; c0 < n; c0 += kRound * st) {
    if (c0 != start) load(c0);
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      if (c < n) z[c] = (double)a[u] - mean;
    }
  }
}
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_finalize(const T* __restrict__ p, long long n, const double* __restrict__ partials, int nb,
               double* __restrict__ z) {
  finalize_body<T>(hw_blk(), p, n, partials, nb, z);
}

__global__ void k_convert(const double* __restrict__ s, float* __restrict__ d, long long n) {
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x)
    d[c] = (float)s[c];
}

// ---- GMRES -----------------------------------------------------------------
// (Grid-stride loops in rounds of kRound elements, see reduce_partials.)

// r = b - A p (b when p is null), partial sums of r^2.
__global__ void __launch_bounds__(kVecThreads)
    k_resid_norm(const double* __restrict__ tx, const double* __restrict__ ty, int nx, int ny,
                 const double* __restrict__ b, const double* __restrict__ p,
                 double* __restrict__ r, double* __restrict__ mail) {
  __shared__ double red[kVecThreads / 64];
  const long long n = (long long)nx * ny, st = (long long)gridDim.x * blockDim.x;
  double s = 0.0;
  for (long long c0 = blockIdx.x * (long long)blockDim.x + threadIdx.x; c0 < n;
       c0 += kRound * st) {
    double v[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st, q = c < n ? c : n - 1;
      const int iy = (int)(q / nx), ix = (int)(q - (long long)iy * nx);
      v[u] = p ? b[q] - stencil(tx, ty, nx, ny, ix, iy, p) : b[q];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      if (c < n) {
        r[c] = v[u];
        s += v[u] * v[u];
      }
    }
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) publish(mail + blockIdx.x, s);
}

__global__ void k_zero(double* __restrict__ v, long long n) {
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x)
    v[c] = 0.0;
}

__global__ void k_scale(double* __restrict__ v, long long n, double alpha) {
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x)
    v[c] *= alpha;
}

// w = A z, partial sums of w . v0; z(c) gives the vector's value at cell c, and put
// keeps the value of each cell once.
template <typename Z, typename Put>
__device__ __forceinline__ void arnoldi_start_of(const Blk blk, const double* __restrict__ tx,
                                                   const double* __restrict__ ty, int nx, int ny,
                                                   Z z, Put put, double* __restrict__ w,
                                                   const double* __restrict__ v0,
                                                   double* __restrict__ partials) {
  __shared__ double red[kVecThreads / 64];
  const long long n = (long long)nx * ny, st = (long long)blk.n * blockDim.x;
  double s = 0.0;
  for (long long c0 = blk.id * (long long)blockDim.x + threadIdx.x; c0 < n;
       c0 += kRound * st) {
    double v[kRound], o[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st, q = c < n ? c : n - 1;
      const int iy = (int)(q / nx), ix = (int)(q - (long long)iy * nx);
      v[u] = stencil_of(tx, ty, nx, ny, ix, iy, z);
      o[u] = v0[q];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      if (c < n) {
        put(c);
        w[c] = v[u];
        s += v[u] * o[u];
      }
    }
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) partials[blk.id] = s;
}
__device__ __forceinline__ void arnoldi_start_body(const Blk blk, const double* __restrict__ tx,
                                                   const double* __restrict__ ty, int nx, int ny,
                                                   const double* __restrict__ z,
                                                   double* __restrict__ w,
                                                   const double* __restrict__ v0,
                                                   double* __restrict__ partials) {
  arnoldi_start_of(blk, tx, ty, nx, ny, [&](long long c) { return z[c]; }, [](long long) {}, w, v0,
                   partials);
}
// h = sum(part_in) (= w . v_i); hcol[i] = h; w -= h v_i; partial sums of
// w . v_next, or of w . w when vnext is null.  The vectors' loads do not
// depend on h: every thread issues its first round before the reduction
// that forms h (outside any loop, so its barriers are met by all threads),
// then finishes its remaining rounds.
__device__ __forceinline__ void mgs_step_body(const Blk blk, const double* __restrict__ part_in,
                                              double* __restrict__ part_out, int nb,
                                              double* __restrict__ hcol, int i,
                                              double* __restrict__ w,
                                              const double* __restrict__ vi,
                                              const double* __restrict__ vnext, long long n) {
  __shared__ double red[kVecThreads / 64];
  const bool self = vnext == nullptr;
  const double* vn = self ? vi : vnext;
  const long long st = (long long)blk.n * blockDim.x;
  double a[kRound], b[kRound], d[kRound];
  auto load = [&](long long c0) {
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st, q = c < n ? c : n - 1;
      a[u] = w[q];
      b[u] = vi[q];
      d[u] = vn[q];
    }
  };
  double s = 0.0, h = 0.0;
  auto use = [&](long long c0) {
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      if (c < n) {
        const double v = a[u] - h * b[u];
        w[c] = v;
        s += v * (self ? v : d[u]);
      }
    }
  };
  const long long start = blk.id * (long long)blockDim.x + threadIdx.x;
  load(start);
  h = reduce_partials(part_in, nb, red);
  if (blk.id == 0 && threadIdx.x == 0) hcol[i] = h;
  use(start);
  for (long long c0 = start + kRound * st; c0 < n; c0 += kRound * st) {
    load(c0);
    use(c0);
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) part_out[blk.id] = s;
}
__global__ void __launch_bounds__(kVecThreads)
    k_mgs_step(const double* __restrict__ part_in, double* __restrict__ part_out, int nb,
               double* __restrict__ hcol, int i, double* __restrict__ w,
               const double* __restrict__ vi, const double* __restrict__ vnext, long long n) {
  mgs_step_body(hw_blk(), part_in, part_out, nb, hcol, i, w, vi, vnext, n);
}

// hn = sqrt(sum(part_in)); w /= hn (if hn > 0); block 0 sends the Hessenberg column
// (hcol[0 .. j), hn) to the host as soon as hn is known.  First round
// loaded before the reduction, as in k_mgs_step.
__device__ __forceinline__ void norm_scale_body(const Blk blk, const double* __restrict__ part_in,
                                                int nb, const double* __restrict__ hcol,
                                                double* __restrict__ mail, int j,
                                                double* __restrict__ w, long long n) {
  __shared__ double red[kVecThreads / 64];
  const long long st = (long long)blk.n * blockDim.x;
  double a[kRound];
  auto load = [&](long long c0) {
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      a[u] = w[c < n ? c : n - 1];
    }
  };
  const long long start = blk.id * (long long)blockDim.x + threadIdx.x;
  load(start);
  const double hn = sqrt(reduce_partials(part_in, nb, red));
  if (blk.id == 0) {
    for (int i = threadIdx.x; i < j; i += blockDim.x) publish(mail + i, hcol[i]);
    if (threadIdx.x == 0) publish(mail + j, hn);
  }
  if (!(hn > 0.0)) return;
  const double inv = 1.0 / hn;
  for (long long c0 = start; c0 < n; c0 += kRound * st) {
    if (c0 != start) load(c0);
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      if (c < n) w[c] = a[u] * inv;
    }
  }
}
__global__ void __launch_bounds__(kVecThreads)
    k_norm_scale(const double* __restrict__ part_in, int nb, const double* __restrict__ hcol,
                 double* __restrict__ mail, int j, double* __restrict__ w, long long n) {
  norm_scale_body(hw_blk(), part_in, nb, hcol, mail, j, w, n);
}

// The Arnoldi step after z_j = T v_j for the columns of one context (blockIdx.y):
// each phase one launch over all of them.
__global__ void __launch_bounds__(kVecThreads) k_tail_start(const TailCols cols) {
  const TailCol& c = cols.c[blockIdx.y];
  arnoldi_start_body(hw_blk(), c.tx, c.ty, c.nx, c.ny, c.z, c.V + (long long)(c.j + 1) * c.n, c.V,
                     c.parts);
}
// The same from T's work vector p instead of z (one column): z = p minus its mean
// (sums: nb partial sums of p; null: no mean taken) is formed on the way and
// stored, as k_finalize does, with its values at the neighbours formed again; the
// pass over z and a launch are saved (4096 x 4096 in FP32 arithmetic, 40 steps: 107.1 ->
// 105.6 ms; 64 x 64 479 -> 462 us).
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_tail_finish(const TailCol c, const T* __restrict__ p, const double* __restrict__ sums,
                  double* __restrict__ z) {
  __shared__ double red[kVecThreads / 64];
  const double mean = sums ? reduce_partials(sums, c.nb, red) / (double)c.n : 0.0;
  auto at = [&](long long q) { return (double)p[q] - mean; };
  arnoldi_start_of(hw_blk(), c.tx, c.ty, c.nx, c.ny, at, [&](long long q) { z[q] = at(q); },
                   c.V + (long long)(c.j + 1) * c.n, c.V, c.parts);
}
__global__ void __launch_bounds__(kVecThreads) k_tail_mgs(const TailCols cols, int i) {
  const TailCol& c = cols.c[blockIdx.y];
  if (i > c.j) return;
  mgs_step_body(hw_blk(), c.parts + (i % 2) * kMaxVecBlocks,
                c.parts + ((i + 1) % 2) * kMaxVecBlocks, c.nb, c.hcol, i,
                c.V + (long long)(c.j + 1) * c.n, c.V + (long long)i * c.n,
                i < c.j ? c.V + (long long)(i + 1) * c.n : (const double*)nullptr, c.n);
}
__global__ void __launch_bounds__(kVecThreads) k_tail_norm(const TailCols cols) {
  const TailCol& c = cols.c[blockIdx.y];
  norm_scale_body(hw_blk(), c.parts + ((c.j + 1) % 2) * kMaxVecBlocks, c.nb, c.hcol, c.mail,
                  c.j + 1, c.V + (long long)(c.j + 1) * c.n, c.n);
}

// p += sum_{i < k} y_i Z_i (k <= kMaxUpdate per launch; y travels with the launch).
constexpr int kMaxUpdate = 16;
struct UpdateY {
  double v[kMaxUpdate];
};
__global__ void k_update(double* __restrict__ p, const double* __restrict__ Z,
                         const UpdateY y, int k, long long n) {
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x) {
    double z[kMaxUpdate];
#pragma unroll
    for (int i = 0; i < kMaxUpdate; ++i) z[i] = Z[(long long)(i < k ? i : 0) * n + c];
    double s = p[c];
#pragma unroll
    for (int i = 0; i < kMaxUpdate; ++i)
      if (i < k) s += y.v[i] * z[i];
    p[c] = s;
  }
}

// partial sums of x^2.
__global__ void __launch_bounds__(kVecThreads)
    k_sumsq(const double* __restrict__ x, long long n, double* __restrict__ mail) {
  __shared__ double red[kVecThreads / 64];
  const long long st = (long long)gridDim.x * blockDim.x;
  double s = 0.0;
  for (long long c0 = blockIdx.x * (long long)blockDim.x + threadIdx.x; c0 < n;
       c0 += kRound * st) {
    double a[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      a[u] = x[c < n ? c : n - 1];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u)
      if (c0 + u * st < n) s += a[u] * a[u];
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) publish(mail + blockIdx.x, s);
}

// ---- several right-hand sides per launch ----------------------------------
// The kernels below apply T to K <= kMaxRhs right-hand sides at once (vectors
// given by per-RHS base pointers).  Every per-RHS sum runs in the order of
// the one-RHS kernels above, so the results are those of K separate
// applications, bit for bit; what the K columns share is each load of a
// factor quad, an MBF entry or an interface-matrix tile, and each step of
// the row recurrence of a box.

template <typename T>
struct RhsPtrs {
  T* v[kMaxRhs];
};

// acc[k] = sum_c D(rc, c) v_k[c] for the K vectors of the group (column k's
// doubled copy at vo / vr + k * VW): each factor entry is converted once and
// used for every column; per column, the order of half_dot.  A scheduling
// barrier after each group of four entries keeps the compiler from hoisting
// all the vector reads at once (which would need more registers than a lane
// has).
template <typename T, typename S, int NB, int K, int VW>
__device__ __forceinline__ void half_dot_k(const HalfRow<S, NB>& d,
                                           const S (&rot)[Half<NB>::NM], const T* vo,
                                           const T* vr, T (&acc)[K], int hf) {
  constexpr int NH = Half<NB>::NH, K0 = Half<NB>::K0, H = Half<NB>::H, NT = Half<NB>::NT;
  if constexpr (Half<NB>::HV == 1) {
    T a[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k) a[k][0] = a[k][1] = a[k][2] = a[k][3] = T(0);
#pragma unroll
    for (int q = 0; q < NH; ++q) {
      const T dq[4] = {(T)d.q[q][0], (T)d.q[q][1], (T)d.q[q][2], (T)d.q[q][3]};
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) a[k][i] = fmat(dq[i], vo[k * VW + K0 + 4 * q + i], a[k][i]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = 0; e < K0; ++e) {
      const T de = (T)d.h[e];
#pragma unroll
      for (int k = 0; k < K; ++k) a[k][e] = fmat(de, vo[k * VW + e], a[k][e]);
    }
#pragma unroll
    for (int g = 1; g <= H; g += 4) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = g; i < g + 4 && i <= H; ++i) {
        const int e = mirror_k<T, NB>(i), p = mirror_sum<T, NB>(i);
        const T de = (T)rot[e - 1];
#pragma unroll
        for (int k = 0; k < K; ++k) a[k][p] = fmat(de, vr[k * VW - e], a[k][p]);
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = (a[k][0] + a[k][1]) + (a[k][2] + a[k][3]);
  } else {
    T a[K][2];
#pragma unroll
    for (int k = 0; k < K; ++k) a[k][0] = a[k][1] = T(0);
#pragma unroll
    for (int q = 0; q < NH; ++q) {
      const T dq[2] = {(T)d.p[q][0], (T)d.p[q][1]};
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int e = 0; e < 2; ++e) a[k][e] = fmat(dq[e], vo[k * VW + K0 + 4 * q + e], a[k][e]);
      if (q & 1) __builtin_amdgcn_sched_barrier(0);
    }
    const T s0 = (T)d.s[0], s1 = K0 == 3 ? (T)d.s[1] : T(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const T u = fmat(s0, vo[k * VW], a[k][0]);
      if constexpr (K0 == 3) {
        const T w = fmat(s1, vo[k * VW + 1], a[k][1]);
        a[k][0] = u;
        a[k][1] = hf ? a[k][1] : w;
      } else {
        a[k][0] = hf ? a[k][0] : u;
      }
    }
    if constexpr (K0 == 3 && sizeof(T) == 8) {
#pragma unroll
      for (int q = 0; q < NH; ++q) {
        if (q % 2 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const T de = (T)rot[2 * q + e];
#pragma unroll
          for (int k = 0; k < K; ++k) a[k][e] = fmat(de, vr[k * VW - (3 + 4 * q + e)], a[k][e]);
        }
      }
      const T de = (T)rot[2 * NH];
#pragma unroll
      for (int k = 0; k < K; ++k) a[k][1] = fmat(de, vr[k * VW + hf - 1], a[k][1]);
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t % 2 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const T de = (T)rot[2 * t + e];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const T v = fmat(de, vr[k * VW - (4 * t + 1 + e)], a[k][e]);
            a[k][e] = 4 * t + 3 + e <= H ? v : hf ? a[k][e] : v;
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = sum_halves(a[k][0] + a[k][1]);
  }
}

// Completes this work-item's global stores before its later loads and makes
// them visible to the group (workgroup scope: waits only, no cache flush).
__device__ __forceinline__ void group_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
}

// Block LDL^T solves of one box for K right-hand sides by the group
// of one end (the recurrence of box_solve, K columns per step).  Row j of
// right-hand side k
// is read at in[k] + j * istride (row lane r: column r); the solution is built
// in place at work[k] + j * wstride: the elimination leaves u_j there and
// the substitution overwrites it with x_j.  The next step's rows are loaded
// one step ahead.  vv holds the group's K vector slots (vec_words each,
// zeroed), other those of the box's other group; cp the couplings (LDS); live =
// false writes nothing;
// pin zeroes b_0 in column 0 (a box fixed at its first cell); the other
// arguments as in box_solve.
template <typename T, typename S, int NB, int K, typename In>
__device__ __forceinline__ void box_solve_k(const In* const (&in)[K], long long istride,
                                            T* const (&work)[K], long long wstride, T* vv,
                                            const T* other, const S* cp,
                                            const S* __restrict__ Dinv, int bx, int by,
                                            int bstride, int r, int hf, int end,
                                            bool live, bool pin, int lo, int hi) {
  constexpr int V0 = Half<NB>::V0, HV = Half<NB>::HV, ENDS = box_ends<S>();
  constexpr int VW = vec_words<NB>(), DEPTH = reg_depth<S, NB>();
  const EndSteps<ENDS> st(by, end, lo, hi);
  const int rc = r < bx ? r : bx - 1;
  const Mirror<NB, sizeof(T) == 8> mir(rc, hf, bx);
  const T* vo = vv + V0 + rc + 2 * hf;
  const T* vr = vv + V0 + rc + bx - 2 * hf;
  T* put = vv + V0 + rc + hf * bx;
  const S* cr = cp + rc;
  const int dx = st.dir * bx;
  const bool own = live && hf == 0 && r < bx;
  T xh[K];
  auto product = [&](const T (&y)[K], const HalfRow<S, NB>& d,
                     const S (&rot)[Half<NB>::NM], T (&acc)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      put[k * VW] = y[k];
      if constexpr (HV == 1) put[k * VW + bx] = y[k];
    }
    wave_sync();
    half_dot_k<T, S, NB, K, VW>(d, rot, vo, vr, acc, hf);
    wave_sync();
  };
  {
    int row = st.first, ca = (st.top && st.n > 1 ? by : 0) * bx;
    T carry[K], nxt[K], c = T(0);
    auto fetch = [&]() {
#pragma unroll
      for (int k = 0; k < K; ++k) nxt[k] = (T)in[k][row * istride + rc];
      if (pin && row == 0 && rc == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) nxt[k] = T(0);
    };
#pragma unroll
    for (int k = 0; k < K; ++k) carry[k] = T(0);
    fetch();
    pipelined_sweep<S, NB, DEPTH>(
        st.n, late_start<NB>(st.n), Dinv + st.first * bstride, st.dir * bstride,
        [&](int s, const HalfRow<S, NB>& d) {
          S rot[Half<NB>::NM];
          mirror_rows<S, NB>(rot, d, mir, hf);
          const bool run = !Half<NB>::PACK || s >= 0;  // the group has started
          T b[K], y[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            b[k] = nxt[k];
            y[k] = fmat(c, carry[k], b[k]);
          }
          const int cur = row;
          row += run && s + 1 < st.n ? st.dir : 0;
          ca += run && s + 1 < st.n ? dx : 0;
          fetch();
          c = run ? (T)cr[ca] : T(0);
          if (ENDS == 2 && s == st.n - 1) {
            // both ends have reached the middle row: exchange the rows next to it
#pragma unroll
            for (int k = 0; k < K; ++k) vv[k * VW + V0 + rc] = carry[k];
            pair_sync<S, NB>();
            const T cl = (T)cr[st.h * bx], ch = (T)cr[(st.h + 1 < by ? st.h + 1 : st.h) * bx];
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const T o = other[k * VW + V0 + rc];
              y[k] = b[k];
              if (st.h > 0) y[k] = fmat(cl, st.top ? o : carry[k], y[k]);
              if (st.h + 1 < by) y[k] = fmat(ch, st.top ? carry[k] : o, y[k]);
            }
            pair_sync<S, NB>();
          }
          product(y, d, rot, carry);
          if (own && run && !(st.top && s == st.n - 1))
#pragma unroll
            for (int k = 0; k < K; ++k) work[k][cur * wstride + r] = carry[k];
          if constexpr (Half<NB>::PACK)
#pragma unroll
            for (int k = 0; k < K; ++k) carry[k] = run ? carry[k] : T(0);
        },
        bx, rc, hf);
#pragma unroll
    for (int k = 0; k < K; ++k) xh[k] = carry[k];
  }
  group_fence();  // lanes of the wave read back the rows that others of it wrote
  const int late = late_start<NB>(st.nb > 0 ? st.nb : 0);
  if (st.nb > 0 || late > 0) {
    // (a group without rows stays on the middle one)
    int row = st.nb > 0 ? st.h - st.dir : st.h, ca = (st.top ? row : st.h) * bx;
    T carry[K], nxt[K], c = (T)cr[ca];
    auto fetch = [&]() {
#pragma unroll
      for (int k = 0; k < K; ++k) nxt[k] = work[k][row * wstride + rc];
    };
#pragma unroll
    for (int k = 0; k < K; ++k) carry[k] = xh[k];
    fetch();
    pipelined_sweep<S, NB, DEPTH>(
        st.nb, late, Dinv + row * bstride, -st.dir * bstride,
        [&](int s, const HalfRow<S, NB>& d) {
          S rot[Half<NB>::NM];
          mirror_rows<S, NB>(rot, d, mir, hf);
          const bool run = !Half<NB>::PACK || s >= 0;
          T u[K], y[K], acc[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            u[k] = nxt[k];
            y[k] = c * carry[k];
          }
          const int cur = row;
          row -= run && s + 1 < st.nb ? st.dir : 0;
          ca -= run && s + 1 < st.nb ? dx : 0;
          fetch();
          c = (T)cr[ca];
          product(y, d, rot, acc);
#pragma unroll
          for (int k = 0; k < K; ++k) carry[k] = run ? u[k] + acc[k] : carry[k];
          if (own && run)
#pragma unroll
            for (int k = 0; k < K; ++k) work[k][cur * wstride + r] = carry[k];
        },
        bx, rc, hf);
  }
  group_fence();
  pair_sync<S, NB>();
}

// LDS slot of one box for K right-hand sides:
//   vv[ends][K][vec_words] (T) | cp[max cells] (S, also the moments' buffer).
template <typename T, typename S, int NB, int K>
struct BoxSlotK {
  T *vv, *other;
  S* cp;
  __device__ BoxSlotK(char* base, int end) {
    constexpr int W = K * vec_words<NB>(), ENDS = box_ends<S>();
    vv = reinterpret_cast<T*>(base) + end * W;
    other = reinterpret_cast<T*>(base) + (ENDS - 1 - end) * W;
    cp = reinterpret_cast<S*>(base + ENDS * W * sizeof(T));
  }
};

// k_local for K right-hand sides: the oversampled solve of every column,
// built in the subdomain's slice of the scratch vectors (offset coff, row
// stride bx), p_k = its restriction to Omega_i, and the trace moments of
// every coarse dof of the subdomain for every k (mU[k * nc + dof], mP
// likewise; the arithmetic of k_local per column).
template <typename T, typename S, int NB, int K>
__global__ void __launch_bounds__(kBoxThreads)
    k_local_k(const BoxDesc* __restrict__ boxes, int m, int group_bytes,
              const S* __restrict__ dinv, const S* __restrict__ coup, RhsPtrs<const double> r,
              RhsPtrs<T> p, RhsPtrs<T> e, int nx, const int* __restrict__ dof_off,
              const int* __restrict__ dof_side, const int* __restrict__ dof_q,
              const int* __restrict__ dof_face0, const double* __restrict__ face_w,
              double* __restrict__ mU, double* __restrict__ mP, int nc) {
  extern __shared__ __align__(16) char smem_raw[];
  typedef BoxThread<S, NB> BT;
  const BT t(blockIdx.x, m);
  BoxSlotK<T, S, NB, K> L(smem_raw + (long long)t.slot * group_bytes, t.end);
  const BoxDesc d = boxes[t.i];
  const int bx = d.bx, by = d.by;
  const long long origin = (long long)d.y0 * nx + d.x0;
  const double* in[K];
  T* work[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    in[k] = r.v[k] + origin;
    work[k] = e.v[k] + d.coff;
  }
  words_to_lds<S, BT::NL, (NB == kPacked16 && BT::NSET == 2 ? 4 : 8)>(L.cp, coup + d.coff,
                                                                      bx * by, t.lane);
  zero_slots<BT::GL>(L.vv, K * vec_words<NB>());
  pair_sync<S, NB>();
  box_solve_k<T, S, NB, K, double>(in, nx, work, bx, L.vv, L.other, L.cp, dinv + d.doff, bx, by,
                                   d.bs, t.r, t.hf, t.end, t.live, d.pin != 0,
                                   trace_lo(d), trace_hi(d));
  if (t.live && t.r >= d.ox && t.r < d.ox + d.obx) {
    const long long o2 = origin + (long long)d.oy * nx;
#pragma unroll 1
    for (int k = 0; k < K; ++k)
      for (int j = t.set; j < d.oby; j += BT::NSET)
        p.v[k][o2 + (long long)j * nx + t.r] = work[k][(long long)(d.oy + j) * bx + t.r];
  }
  const int k0 = dof_off[t.i], nd = dof_off[t.i + 1] - k0;
  if (nd > 0)  // as in local_body
    trace_moments<S, NB, K>(d, nx, t.lane, t.live, t.faces(boxes, blockIdx.x, m), dof_side, dof_q,
                            dof_face0, k0, nd, face_w, reinterpret_cast<double*>(L.cp),
                            [&](int k, int c) { return (double)(e.v[k] + d.coff)[c]; }, mU, mP,
                            nc);
}

// k_patch for K right-hand sides: e_k = A[S_i]^-1 rho_k[S_i], built in the
// patch's slice of the scratch vectors (offset coff, row stride bx), then
// p_k += e_k on the owned cells.
template <typename T, typename S, int NB, int K>
__global__ void __launch_bounds__(kBoxThreads)
    k_patch_k(const BoxDesc* __restrict__ boxes, int m, int group_bytes,
              const S* __restrict__ dinv, const S* __restrict__ coup, RhsPtrs<const T> rho,
              RhsPtrs<T> p, RhsPtrs<T> e, int nx) {
  extern __shared__ __align__(16) char smem_raw[];
  typedef BoxThread<S, NB> BT;
  const BT t(blockIdx.x, m);
  BoxSlotK<T, S, NB, K> L(smem_raw + (long long)t.slot * group_bytes, t.end);
  const BoxDesc d = boxes[t.i];
  const int bx = d.bx, by = d.by;
  const long long origin = (long long)d.y0 * nx + d.x0;
  const T* in[K];
  T* work[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    in[k] = rho.v[k] + origin;
    work[k] = e.v[k] + d.coff;
  }
  words_to_lds<S, BT::NL, (NB == kPacked16 && BT::NSET == 2 ? 4 : 8)>(L.cp, coup + d.coff,
                                                                      bx * by, t.lane);
  zero_slots<BT::GL>(L.vv, K * vec_words<NB>());
  pair_sync<S, NB>();
  box_solve_k<T, S, NB, K, T>(in, nx, work, bx, L.vv, L.other, L.cp, dinv + d.doff, bx, by,
                              d.bs, t.r, t.hf, t.end, t.live, d.pin != 0, d.oy,
                              d.oy + d.oby - 1);
  // p += e on the owned cells, each set of row lanes a run of rows in
  // turn, all of a run's read-modify-writes in flight
  constexpr int RUN = NB == kPacked16 && BT::NSET == 2 ? 4 : 8;
  const bool own = t.live && t.r >= d.ox && t.r < d.ox + d.obx;
  const int col = own ? t.r : d.ox;
  const long long o2 = origin + (long long)d.oy * nx;
  const int rows = d.oby;
#pragma unroll 1
  for (int k = 0; k < K; ++k) {
    T* pk = p.v[k];
    const T* ek = work[k] + (long long)d.oy * bx;
    for (int jj = 0; jj < rows; jj += RUN * BT::NSET) {
      const int j0 = jj + RUN * t.set;
      T v[RUN], ev[RUN];
#pragma unroll
      for (int u = 0; u < RUN; ++u) {
        const int j = j0 + u < d.oby ? j0 + u : d.oby - 1;
        v[u] = pk[o2 + (long long)j * nx + col];
        ev[u] = ek[(long long)j * bx + col];
      }
#pragma unroll
      for (int u = 0; u < RUN; ++u)
        if (own && j0 + u < d.oby) pk[o2 + (long long)(j0 + u) * nx + t.r] = v[u] + ev[u];
    }
  }
}

// Interface right-hand sides of K columns (blockIdx.y = column; vectors of
// column k at offset k * nc / k * np).
__global__ void k_coarse_rhs_k(const int4* __restrict__ gsrc, const double* __restrict__ gscale,
                               const double* __restrict__ mU, const double* __restrict__ mP,
                               double* __restrict__ g_nd, int np, int nc) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= np) return;
  const long long ko = (long long)blockIdx.y * nc;
  const int4 src = gsrc[t];
  const double v = src.z == 0 ? -(mU[ko + src.x] + mU[ko + src.y])
                              : -(mP[ko + src.x] - mP[ko + src.y]);
  g_nd[(long long)blockIdx.y * np + t] = src.z == 2 ? 0.0 : gscale[t] * v;
}

// s[u][k] += sum_q m[u][q] vec_k[b0 + 64 q] for the K columns vec + k * ld
// (LDS): per (u, k) the order of fma_tile.  One column at a time (a
// scheduling barrier after each keeps the LDS reads of later columns from
// being hoisted into registers).
template <int K>
__device__ __forceinline__ void fma_tile_k(double (&s)[4][K], const double (&m)[4][8],
                                           const double* vec, int ld, int ncol, int b0) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = b0 + 64 * q < ncol ? vec[k * ld + b0 + 64 * q] : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u][k] = fmat(m[u][q], x[q], s[u][k]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// gemv_chunk for K columns of the LDS matrix vec (column k at vec + k * ld).
// After the butterfly, lane l holds output (row r + u_l, column k_l) with
// u_l * K + k_l = butterfly_index(l); pre(row, k) runs in every lane for its
// own output before that group's tile loads, and emit(row, k, value) in one
// lane per output.
template <int K, typename Pre, typename Emit>
__device__ __forceinline__ void gemv_chunk_k(const double* __restrict__ M, int ncol, int row0,
                                             int row1, const double* vec, int ld,
                                             double (&m)[4][8], Pre pre, Emit emit) {
  constexpr int N = 4 * K;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int bi = butterfly_index<N>(lane);
  const int ul = bi / K, kl = bi % K;
  const bool emitter = (lane & (64 / N - 1)) == 0;
  for (int r = row0 + 4 * wid; r < row1; r += 4 * nw) {
    const bool first = r == row0 + 4 * wid;
    if (!first) pre(r + ul, kl);
    double s[4][K];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) s[u][k] = 0.0;
    fma_tile_k<K>(s, m, vec, ld, ncol, lane);
    for (int b0 = lane + 64 * 8; b0 < ncol; b0 += 64 * 8) {
      load_tile(m, M, ncol, r, row1, b0);
      fma_tile_k<K>(s, m, vec, ld, ncol, b0);
    }
    if (r + 4 * nw < row1) load_tile(m, M, ncol, r + 4 * nw, row1, lane);
    double v[N];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) v[u * K + k] = s[u][k];
    butterfly_sum<N>(v, lane);
    if (emitter && r + ul < row1) emit(r + ul, kl, v[0]);
  }
}

// k_coarse_fwd for K columns (column k of g_nd, contrib, ybuf and x at
// offsets k * np, k * maxp * np, k * np and k * nc).
template <int K>
__global__ void __launch_bounds__(kVecThreads)
    k_coarse_fwd_k(const CChunk* __restrict__ chunks, const double* __restrict__ fwd,
                   const double* __restrict__ g_nd, double* __restrict__ contrib, int maxp,
                   int np, const int* __restrict__ cdest, double* __restrict__ ybuf,
                   const int* __restrict__ idx, double* __restrict__ x, int nc) {
  extern __shared__ double v[];
  const CChunk ch = chunks[blockIdx.x];
  const int nf = ch.nf;
  const double* M = fwd + ch.mat;
  const int yoff = ch.yoff, coff = ch.coff;
  const long long cstride = (long long)maxp * np;
  int dst = -1;
  auto pre = [&](int row, int) {
    dst = (row >= nf && row < ch.row1) ? cdest[coff + row - nf] : -1;
  };
  double m[4][8];
  const int rw = ch.row0 + 4 * (threadIdx.x >> 6);
  load_tile(m, M, nf, rw, ch.row1, threadIdx.x & 63);
  {
    const int bi = butterfly_index<4 * K>(threadIdx.x & 63);
    pre(rw + bi / K, bi % K);
  }
  for (int e = threadIdx.x; e < nf * K; e += blockDim.x) {
    const int k = e / nf, a = e - k * nf;
    const long long t = (long long)yoff + a;
    double s = g_nd[(long long)k * np + t];
    const double* ck = contrib + k * cstride;
    for (int u0 = 0; u0 < maxp; u0 += 8) {
      double c[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) c[q] = u0 + q < maxp ? ck[(long long)(u0 + q) * np + t] : 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (u0 + q < maxp) s -= c[q];
    }
    v[k * nf + a] = s;
  }
  __syncthreads();
  gemv_chunk_k<K>(M, nf, ch.row0, ch.row1, v, nf, m, pre, [&](int row, int k, double val) {
    if (row >= nf)
      contrib[k * cstride + dst] = val;
    else if (ch.nu == 0)
      x[(long long)k * nc + idx[ch.fcol + row]] = val;
    else
      ybuf[(long long)k * np + yoff + row] = val;
  });
}

// k_coarse_bwd for K columns (column k of ybuf and x at offsets k * np and
// k * nc).
template <int K>
__global__ void __launch_bounds__(kVecThreads)
    k_coarse_bwd_k(const CChunk* __restrict__ chunks, const double* __restrict__ bwd,
                   const int* __restrict__ idx, const double* __restrict__ ybuf,
                   double* __restrict__ x, int np, int nc) {
  extern __shared__ double xu[];
  const CChunk ch = chunks[blockIdx.x];
  const int nu = ch.nu;
  const double* M = bwd + ch.mat;
  const int yoff = ch.yoff, fcol = ch.fcol;
  int dst = 0;
  double y = 0.0;
  auto pre = [&](int row, int k) {
    if (row < ch.row1) {
      dst = idx[fcol + row];
      y = ybuf[(long long)k * np + yoff + row];
    }
  };
  double m[4][8];
  const int rw = ch.row0 + 4 * (threadIdx.x >> 6);
  load_tile(m, M, nu, rw, ch.row1, threadIdx.x & 63);
  {
    const int bi = butterfly_index<4 * K>(threadIdx.x & 63);
    pre(rw + bi / K, bi % K);
  }
  for (int e = threadIdx.x; e < nu * K; e += blockDim.x) {
    const int k = e / nu, b = e - k * nu;
    xu[k * nu + b] = x[(long long)k * nc + idx[ch.ucol + b]];
  }
  __syncthreads();
  gemv_chunk_k<K>(M, nu, ch.row0, ch.row1, xu, nu, m, pre,
                  [&](int, int k, double val) { x[(long long)k * nc + dst] = y - val; });
}

// k_reconstruct for K columns: p_k[Omega_i] += P_i x_i^k, each MBF entry
// loaded once for all k.
template <typename T, typename S, int K>
__global__ void __launch_bounds__(kBoxThreads)
    k_reconstruct_k(const BoxDesc* __restrict__ boxes, const S* __restrict__ mbf,
                    const long long* __restrict__ mbf_off, const int* __restrict__ dof_off,
                    const double* __restrict__ xc, int nc, RhsPtrs<T> p, int nx) {
  __shared__ T xs[K][64];
  const int i = blockIdx.x;
  const BoxDesc d = boxes[i];
  const int k0 = dof_off[i], nk = dof_off[i + 1] - k0, ncell = d.obx * d.oby;
  for (int e = threadIdx.x; e < nk * K; e += blockDim.x) {
    const int k = e / nk, j = e - k * nk;
    xs[k][j] = (T)xc[(long long)k * nc + k0 + j];
  }
  __syncthreads();
  const S* P = mbf + mbf_off[i];
  for (int q = threadIdx.x; q < ncell; q += blockDim.x) {
    const int a = q % d.obx, j = q / d.obx;
    const long long c = (long long)(d.y0 + d.oy + j) * nx + d.x0 + d.ox + a;
    T s[K];
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = p.v[k][c];
    for (int j2 = 0; j2 < nk; ++j2) {
      const T pv = (T)P[(long long)j2 * ncell + q];
#pragma unroll
      for (int k = 0; k < K; ++k) s[k] = fmat(pv, xs[k][j2], s[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) p.v[k][c] = s[k];
  }
}

// k_reconstruct_k for 8 right-hand sides on the matrix cores: per
// subdomain, P_i^T (cells x nk, nk <= 8 basis functions) times X (nk x 8
// columns) is added to the 8 columns of p[Omega_i] in tiles of 16 cells, one
// wave per tile, as a 16 x 16 x 8 product (columns 8..15 and basis functions
// past nk are zero).  MfmaRecon selects the instruction: 0 the FP32 or FP64
// 16x16x4 MFMA of the arithmetic type (two steps of four basis functions);
// 1 the BF16 16x16x16 MFMA with FP32 accumulation (P and X rounded to BF16,
// nearest even; FP32 arithmetic only).  The sums are those of the MFMA, not
// of k_reconstruct_k's FMA chain, so results differ from it in rounding.
// MFMA 16 x 16 operand layout: lane l holds A[l % 16][l / 16] (cells x
// basis functions), B[l / 16][l % 16] (basis functions x columns), and in
// accumulator register r row 4 (l / 16) + r of column l % 16 (FP32 and
// BF16 forms) or row 4 r + l / 16 (FP64 form); the BF16 form holds four
// consecutive k per lane (k = 4 (l / 16) .. + 3).
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));
typedef double mfma_f64x4 __attribute__((ext_vector_type(4)));
typedef short mfma_s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ short bf16_rne(float f) {
  const unsigned u = __float_as_uint(f);
  return (short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
template <typename T, int MODE> struct MfmaAcc;
template <> struct MfmaAcc<float, 0> { typedef mfma_f32x4 type; };
template <> struct MfmaAcc<float, 1> { typedef mfma_f32x4 type; };
template <> struct MfmaAcc<double, 0> { typedef mfma_f64x4 type; };

template <typename T, typename S, int MODE>
__global__ void __launch_bounds__(kBoxThreads)
    k_reconstruct_mfma(const BoxDesc* __restrict__ boxes, const S* __restrict__ mbf,
                       const long long* __restrict__ mbf_off, const int* __restrict__ dof_off,
                       const double* __restrict__ xc, int nc, RhsPtrs<T> p, int nx) {
  typedef typename MfmaAcc<T, MODE>::type Acc;
  __shared__ T xs[16][16];
  const int i = blockIdx.x;
  const BoxDesc d = boxes[i];
  const int k0 = dof_off[i], nk = dof_off[i + 1] - k0, ncell = d.obx * d.oby;
  for (int e = threadIdx.x; e < 16 * 16; e += blockDim.x) {
    const int k = e / 16, j = e % 16;
    xs[k][j] = (k < nk && k < 8 && j < 8) ? (T)xc[(long long)j * nc + k0 + k] : T(0);
  }
  __syncthreads();
  const S* P = mbf + mbf_off[i];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  T* pj = p.v[li < 8 ? li : 0];
  const long long base = (long long)(d.y0 + d.oy) * nx + d.x0 + d.ox;
  for (int t = wid; t * 16 < ncell; t += nw) {
    const int q = 16 * t + li;
    long long addr[4];
    bool ok[4];
    Acc c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qq = 16 * t + (sizeof(T) == 8 ? 4 * r + lk : 4 * lk + r);
      ok[r] = li < 8 && qq < ncell;
      const int qc = qq < ncell ? qq : 0;
      const int row = qc / d.obx, col = qc - row * d.obx;
      addr[r] = base + (long long)row * nx + col;
      c[r] = ok[r] ? pj[addr[r]] : T(0);
    }
    if constexpr (MODE == 0) {
#pragma unroll
      for (int s4 = 0; s4 < 2; ++s4) {
        const int k = 4 * s4 + lk;
        const T a = (k < nk && q < ncell) ? (T)P[(long long)k * ncell + q] : T(0);
        const T b = xs[k][li];
        if constexpr (sizeof(T) == 4)
          c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
        else
          c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
      }
    } else {
      mfma_s16x4 a, b;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 4 * lk + u;
        a[u] = bf16_rne((k < nk && q < ncell) ? (float)P[(long long)k * ncell + q] : 0.0f);
        b[u] = bf16_rne((float)xs[k][li]);
      }
      c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (ok[r]) pj[addr[r]] = c[r];
  }
}

// Smoothing residuals rho_k = r_k - A p_k (blockIdx.y = k).
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_residual_k(const T* __restrict__ tx, const T* __restrict__ ty, int nx, int ny,
                 RhsPtrs<const double> r, RhsPtrs<const T> p, RhsPtrs<T> rho) {
  const long long n = (long long)nx * ny;
  const double* rk = r.v[blockIdx.y];
  const T* pk = p.v[blockIdx.y];
  T* ok = rho.v[blockIdx.y];
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x) {
    const int iy = (int)(c / nx), ix = (int)(c - (long long)iy * nx);
    ok[c] = (T)rk[c] - stencil(tx, ty, nx, ny, ix, iy, pk);
  }
}

// k_sum for K vectors (blockIdx.y = k; partials of k at k * kMaxVecBlocks).
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_sum_k(RhsPtrs<const T> p, long long n, double* __restrict__ partials) {
  __shared__ double red[kVecThreads / 64];
  const T* pk = p.v[blockIdx.y];
  const long long st = (long long)gridDim.x * blockDim.x;
  double s = 0.0;
  for (long long c0 = blockIdx.x * (long long)blockDim.x + threadIdx.x; c0 < n;
       c0 += kRound * st) {
    T a[kRound];
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      a[u] = pk[c < n ? c : n - 1];
    }
#pragma unroll
    for (int u = 0; u < kRound; ++u)
      if (c0 + u * st < n) s += (double)a[u];
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) partials[(long long)blockIdx.y * kMaxVecBlocks + blockIdx.x] = s;
}

// k_finalize for K vectors (blockIdx.y = k).
template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_finalize_k(RhsPtrs<const T> p, long long n, const double* __restrict__ partials, int nb,
                 RhsPtrs<double> z) {
  __shared__ double red[kVecThreads / 64];
  const T* pk = p.v[blockIdx.y];
  double* zk = z.v[blockIdx.y];
  const double* part = partials ? partials + (long long)blockIdx.y * kMaxVecBlocks : nullptr;
  const long long st = (long long)gridDim.x * blockDim.x;
  T a[kRound];
  auto load = [&](long long c0) {
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      a[u] = pk[c < n ? c : n - 1];
    }
  };
  const long long start = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  load(start);
  const double mean = part ? reduce_partials(part, nb, red) / (double)n : 0.0;
  for (long long c0 = start; c0 < n; c0 += kRound * st) {
    if (c0 != start) load(c0);
#pragma unroll
    for (int u = 0; u < kRound; ++u) {
      const long long c = c0 + u * st;
      if (c < n) zk[c] = (double)a[u] - mean;
    }
  }
}

inline int grid_for(long long n) {
  long long b = (n + kVecThreads - 1) / kVecThreads;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

void launch_op_apply(const double* tx, const double* ty, int nx, int ny, const double* x,
                     double* y, int nrhs, hipStream_t s) {
  const long long n = (long long)nx * ny;
  const int tiles_x = (nx + 63) / 64, tiles = tiles_x * ((ny + 4 * kOpRows - 1) / (4 * kOpRows));
  const dim3 grid((tiles + 7) / 8 * 8), block(kVecThreads);
  for (int k = 0; k < nrhs; k += kOpColumns) {
    auto run = [&](auto* kernel) {
      hipLaunchKernelGGL(kernel, grid, block, 0, s, tx, ty, nx, ny, tiles_x, tiles, x + k * n,
                         y + k * n);
    };
    switch (nrhs - k < kOpColumns ? nrhs - k : kOpColumns) {
      case 1: run(k_op_apply<1>); break;
      case 2: run(k_op_apply<2>); break;
      case 3: run(k_op_apply<3>); break;
      default: run(k_op_apply<4>);
    }
  }
}

void launch_rhs(const double* tx, const double* ty, int nx, int ny, const int* bc,
                const double* f, const double* g, double h, double* b, hipStream_t s) {
  const long long n = (long long)nx * ny;
  hipLaunchKernelGGL(k_rhs, dim3(grid_for(n)), dim3(kVecThreads), 0, s, tx, ty, nx, ny, bc[0],
                     bc[1], bc[2], bc[3], f, g, h, b);
}

// Column width (registers) for boxes up to max_bx cells wide; ends of a factor; threads of
// one box of column width code nb (a wave per end of its factor, fewer lanes packed);
// w: bytes of the factor storage type.
inline int col_width(int max_bx) { return box_cols(max_bx); }
inline int ends_of(size_t w) { return w == 8 ? 2 : 1; }
inline int box_threads(int nb, size_t w) {
  return (nb == kPacked16 ? 16 : nb == kPacked20 ? 32 : 64) * ends_of(w);
}
// Words of a group's vector slot (vec_words of the kernels).
inline int vec_slot_words(int nb) {
  switch (nb) {
    case 16: return vec_words<16>();
    case kPacked16: return vec_words<kPacked16>();
    case kPacked20: return vec_words<kPacked20>();
    case 20: return vec_words<20>();
    case 24: return vec_words<24>();
    case 32: return vec_words<32>();
    case 36: return vec_words<36>();
    case 40: return vec_words<40>();
    case 48: return vec_words<48>();
    default: return vec_words<64>();
  }
}
// Words of S in 16 bytes; x rounded up to a multiple of them.
inline int round16(long long x, size_t w) {
  const long long e = 16 / (long long)w;
  return (int)((x + e - 1) / e * e);
}
// Words of a box's coupling area: the couplings, or the trace moments' buffer
// (three FP64 words per thread of the box) where that is larger.
inline int coupling_words(int nb, int max_cells, size_t w) {
  const long long buf = 3LL * box_threads(nb, w) * (8 / (long long)w);
  return round16(max_cells > buf ? max_cells : buf, w);
}
// LDS bytes of one box: the vector slots of its groups and the box
// (arithmetic words t) and the coupling area (storage words w), rounded to 16
// bytes.
inline size_t group_bytes(int nb, int max_cells, size_t t, size_t w) {
  const size_t b = (size_t)ends_of(w) * vec_slot_words(nb) * t +
                   (size_t)coupling_words(nb, max_cells, w) * w + (size_t)max_cells * t;
  return (b + 15) / 16 * 16;
}
// Boxes are accepted up to kBoxLds bytes for one vector slot of whole lane groups (16
// lanes for boxes of up to 16 columns), the couplings and the box, which is not what a
// launch takes: with the second slot, wider slots and the moments' buffer the largest
// accepted boxes ask for up to kBoxLdsMax (16 x 254 in FP64: 66 176 bytes).
constexpr size_t kBoxLds = 64 * 1024, kBoxLdsMax = kBoxLds + 8192, kCuLds = 160 * 1024;
bool box_fits(int max_bx, int max_cells, size_t t, size_t w) {
  const int lanes = max_bx <= 16 ? 16 : max_bx <= 32 ? 32 : 64;
  const size_t slot = (col_width(max_bx) / 2 + 2 * lanes + 3) / 4 * 4;
  const size_t b = slot * t + (size_t)round16(max_cells, w) * w + (size_t)max_cells * t;
  return (b + 15) / 16 * 16 <= kBoxLds;
}
// Column width code of a launch over m boxes.  Boxes of up to 16 columns are packed where
// one wave per end gives the GPU more than two waves per SIMD (256 CUs of four).  One column
// of T, a wave per end and packed: 256 x 256 in 8-wide subdomains, 1024 boxes, FP64 (2048
// waves) 74, 75 us; 480 x 480, 12-wide, 1600 boxes, FP64 106, 98, FP32 storage (1600 waves)
// 102, 109; 256 x 256, 4-wide, 4096 boxes, FP32 storage 117, 111; 768 x 768, 8-wide, 9216
// boxes, FP64 309, 263 (278 with one-ended factors, four boxes to a wave).
// Boxes of 17 to 20 columns are packed past kPack20Boxes where that measured faster: FP32
// arithmetic over several contexts (four columns of T, 16-wide subdomains: 5184 boxes 239,
// 228 us, 16 384 boxes 522, 468; 1296 boxes 121, 124), and several columns unless FP32
// factors are applied in FP64 arithmetic (four columns, 4096 boxes, FP64 628, 593, FP32 430, 415;
// 2304 boxes 399, 421 and 272, 294).  One column gains nothing (4096 boxes, FP64 102, 103 in
// the box kernels), FP64 over several contexts neither (16 384 boxes 677, 674).
constexpr long long kPackWaves = 2 * 4 * 256, kPack20Boxes = 3072;
constexpr bool pack20_many(size_t t) { return t == 4; }
constexpr bool pack20_columns(size_t t, size_t w) { return t == w; }
inline int launch_cols(long long m, int max_bx, size_t w, bool pack20) {
  const int nb = col_width(max_bx);
  if (nb == 20 && pack20 && m > kPack20Boxes) return kPacked20;
  return nb == 16 && m * ends_of(w) > kPackWaves ? kPacked16 : nb;
}
// Whether a launch over m boxes has more waves than the GPU has SIMDs, so that kernels of one
// wave per SIMD would take a second round (box_least_waves).
inline bool box_dense(long long m, size_t w) { return m * ends_of(w) > 4 * 256; }
// The most boxes a workgroup of up to 256 threads takes in whole waves, `bytes` of LDS each
// (0: not one wave's).
inline int most_groups(int nb, size_t w, size_t bytes) {
  const int bt = box_threads(nb, w);
  for (int groups = kBoxThreads / bt; groups * bt >= 64 && groups > 0; groups /= 2)
    if (groups * bytes <= kBoxLds) return groups;
  return 0;
}
BoxGrid box_grid(long long m, int max_bx, int max_cells, size_t t, size_t w, bool many) {
  int nb = launch_cols(m, max_bx, w, many && pack20_many(t));
  const bool dense = box_dense(m, w);
  if (nb % 2 == 1) {
    const int groups = most_groups(nb, w, group_bytes(nb, max_cells, t, w));
    if (groups > 0) return BoxGrid{nb, groups, 64 / box_threads(nb, w), false};
    --nb;  // tall boxes: not a wave's worth of them in LDS
  }
  // up to 256 threads per CU a box is a workgroup, so that they spread over the CUs (T, packed
  // into workgroups of four waves and spread: 512 x 512, 40-wide boxes in FP64 124, 105 us, 256
  // boxes 20 wide 63, 60; 1024 of them, FP32 storage, 93 both ways; 2500 of 32 in FP64 231, 240)
  if (!many && m * box_threads(nb, w) <= 4LL * 64 * 256) return BoxGrid{nb, 1, 1, dense};
  const size_t bytes = group_bytes(nb, max_cells, t, w);
  int groups = most_groups(nb, w, bytes);
  // more large boxes over several contexts than run at once: as many on a CU as its 160 KB
  // hold (48 x 48 with FP32 factors, 29 KB each: two to a workgroup are four on a CU, one is
  // five; four columns of 960 x 960 1042, 948 us; without the condition 512 x 512 in 40-wide
  // boxes 243, 251; 24-wide boxes are held by registers, not LDS: a server's three grids 3057 us,
  // 3182)
  if (many && nb >= 36 && groups > 1 && m > 256 * (long long)(kCuLds / (groups * bytes) * groups))
    for (int g = groups / 2; g >= 1; g /= 2)
      if (kCuLds / (g * bytes) * g > kCuLds / (groups * bytes) * groups) groups = g;
  return BoxGrid{nb, groups > 0 ? groups : 1, 1, dense};
}
// Launch a box kernel with shm bytes of LDS (past 64 KB gfx950 has to be asked).
template <typename... A, typename... B>
void launch_box(void (*kernel)(A...), dim3 grid, dim3 block, size_t shm, hipStream_t s,
                B... args) {
  if (shm > kBoxLds &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBoxLdsMax) != hipSuccess)
    throw Error(MRCM_EDEVICE, "no workgroup with the LDS of a box");
  hipLaunchKernelGGL(kernel, grid, block, shm, s, args...);
}
#define MRCM_BOX_CASE(KERNEL, T, S, NB, ...) \
  case NB: launch_box(KERNEL<T, S, NB, false>, __VA_ARGS__); break;
#define MRCM_BOX_CASE_DENSE(KERNEL, T, S, NB, dense, ...)     \
  case NB:                                                    \
    if constexpr (sizeof(S) == 8) {                           \
      if (dense) {                                            \
        launch_box(KERNEL<T, S, NB, true>, __VA_ARGS__);      \
        break;                                                \
      }                                                       \
    }                                                         \
    launch_box(KERNEL<T, S, NB, false>, __VA_ARGS__);         \
    break;
#define MRCM_BOX_DISPATCH(KERNEL, T, S, nb, dense, ...)            \
  do {                                                             \
    switch (nb) {                                                  \
      MRCM_BOX_CASE(KERNEL, T, S, 16, __VA_ARGS__)                 \
      MRCM_BOX_CASE(KERNEL, T, S, kPacked16, __VA_ARGS__)          \
      MRCM_BOX_CASE(KERNEL, T, S, 20, __VA_ARGS__)                 \
      MRCM_BOX_CASE(KERNEL, T, S, 24, __VA_ARGS__)                 \
      MRCM_BOX_CASE(KERNEL, T, S, 32, __VA_ARGS__)                 \
      MRCM_BOX_CASE(KERNEL, T, S, 36, __VA_ARGS__)                 \
      MRCM_BOX_CASE_DENSE(KERNEL, T, S, 40, dense, __VA_ARGS__)    \
      MRCM_BOX_CASE_DENSE(KERNEL, T, S, 48, dense, __VA_ARGS__)    \
      MRCM_BOX_CASE(KERNEL, T, S, 64, __VA_ARGS__)                 \
    }                                                              \
  } while (0)
#define MRCM_MANY_CASE(KERNEL, T, S, NB, ...) \
  case NB: launch_box(KERNEL<T, S, NB, true>, __VA_ARGS__); break;
#define MRCM_MANY_DISPATCH(KERNEL, T, S, nb, dense, ...)               \
  do {                                                          \
    switch (nb) {                                               \
      MRCM_MANY_CASE(KERNEL, T, S, 16, __VA_ARGS__)             \
      MRCM_MANY_CASE(KERNEL, T, S, kPacked16, __VA_ARGS__)      \
      MRCM_MANY_CASE(KERNEL, T, S, 20, __VA_ARGS__)             \
      case kPacked20:                                           \
        if constexpr (pack20_many(sizeof(T)))                   \
          launch_box(KERNEL<T, S, kPacked20, true>, __VA_ARGS__); \
        break;                                                  \
      MRCM_MANY_CASE(KERNEL, T, S, 24, __VA_ARGS__)             \
      MRCM_MANY_CASE(KERNEL, T, S, 32, __VA_ARGS__)             \
      MRCM_MANY_CASE(KERNEL, T, S, 36, __VA_ARGS__)             \
      MRCM_MANY_CASE(KERNEL, T, S, 40, __VA_ARGS__)             \
      case 48:                                                  \
        if constexpr (sizeof(T) == 8 && sizeof(S) == 4) {       \
          if (!(dense)) {                                       \
            launch_box(KERNEL<T, S, 48, false>, __VA_ARGS__);   \
            break;                                              \
          }                                                     \
        }                                                       \
        launch_box(KERNEL<T, S, 48, true>, __VA_ARGS__);        \
        break;                                                  \
      MRCM_MANY_CASE(KERNEL, T, S, 64, __VA_ARGS__)             \
    }                                                           \
  } while (0)
// The grid of a launch over m boxes, capped at groups_cap boxes per workgroup, and its
// LDS: bytes of a box and words of its coupling area.
struct BoxLaunch {
  int nb, gb, cp_words;
  bool dense;
  dim3 grid, block;
  size_t shm;
  BoxLaunch(int m, int max_bx, int max_cells, size_t t, size_t w, int groups_cap) {
    const BoxGrid g = box_grid(m, max_bx, max_cells, t, w, false);
    nb = g.cols;
    dense = g.dense;
    int groups = g.groups;
    if (groups_cap > 0 && groups_cap < groups) groups = groups_cap > g.least ? groups_cap : g.least;
    gb = (int)group_bytes(nb, max_cells, t, w);
    cp_words = coupling_words(nb, max_cells, w);
    grid = dim3((m + groups - 1) / groups);
    block = dim3(groups * box_threads(nb, w));
    shm = (size_t)groups * gb;
  }
};
template <typename T, typename S>
void launch_local(const BoxDesc* boxes, int m, int max_cells, int max_bx, const S* dinv,
                  const S* coup, const double* r, T* p, int nx, const int* dof_off,
                  const int* dof_side, const int* dof_q, const int* dof_face0,
                  const double* face_w, double* mU, double* mP, hipStream_t s, int groups_cap) {
  const BoxLaunch l(m, max_bx, max_cells, sizeof(T), sizeof(S), groups_cap);
  MRCM_BOX_DISPATCH(k_local, T, S, l.nb, l.dense, l.grid, l.block, l.shm, s, boxes, m, l.gb,
                    l.cp_words, dinv, coup, r, p, nx, dof_off, dof_side, dof_q, dof_face0,
                    face_w, mU, mP);
}

void launch_coarse_rhs(const int4* gsrc, const double* gscale, const double* mU,
                       const double* mP, double* g_nd, int np, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_coarse_rhs, dim3((np + 255) / 256), dim3(256), 0, s, gsrc, gscale, mU, mP,
                     g_nd, np);
}
void launch_coarse_resid(int k, const int* rp, const int* ci, const double* v,
                         const double* g_nd, const double* x, double* r_nd, int np, int nc,
                         hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_coarse_resid, dim3((np + 255) / 256, k), dim3(256), 0, s, rp, ci, v, g_nd,
                     x, r_nd, np, nc);
}
void launch_coarse_add(double* x, const double* dx, long long n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_coarse_add, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, dx, n);
}

// Threads per chunk of an interface level: levels with very many chunks
// (the leaves: small fronts) take one wave per chunk, which takes its chunk
// whole, so that every chunk of the level is resident at once; the other
// levels take four waves per chunk (a sweep of the threshold over 0, 1024,
// 2048 and never found 2048 best at 1024^2 and 4096^2).
int coarse_threads(int nchunks, bool forward) {
  return forward || nchunks < 2048 ? kVecThreads : 64;
}

void launch_coarse_fwd(const CChunk* chunks, int nchunks, const double* fwd, const double* g_nd,
                       double* contrib, int maxp, int np, const int* cdest, double* ybuf,
                       const int* idx, double* x, int max_nf, hipStream_t s, int threads) {
  if (nchunks <= 0) return;
  if (threads != 64 && threads != kVecThreads) threads = coarse_threads(nchunks, true);
  hipLaunchKernelGGL(k_coarse_fwd, dim3(nchunks), dim3(threads),
                     sizeof(double) * (size_t)(max_nf > 0 ? max_nf : 1), s, chunks, fwd, g_nd,
                     contrib, maxp, np, cdest, ybuf, idx, x);
}
void launch_coarse_bwd(const CChunk* chunks, int nchunks, const double* bwd, const int* idx,
                       const double* ybuf, double* x, int max_nu, hipStream_t s, int threads) {
  if (nchunks <= 0) return;
  if (threads != 64 && threads != kVecThreads) threads = coarse_threads(nchunks, false);
  hipLaunchKernelGGL(k_coarse_bwd, dim3(nchunks), dim3(threads),
                     sizeof(double) * (size_t)(max_nu > 0 ? max_nu : 1), s, chunks, bwd, idx,
                     ybuf, x);
}
template <typename T, typename S>
void launch_reconstruct(const BoxDesc* boxes, int m, const S* mbf, const long long* mbf_off,
                        const int* dof_off, const double* xc, T* p, int nx, hipStream_t s) {
  hipLaunchKernelGGL((k_reconstruct<T, S>), dim3(m), dim3(kBoxThreads), 0, s, boxes, mbf,
                     mbf_off, dof_off, xc, p, nx);
}

template <typename T>
void launch_residual(const T* tx, const T* ty, int nx, int ny, const double* r, const T* p,
                     T* rho, hipStream_t s) {
  const long long n = (long long)nx * ny;
  hipLaunchKernelGGL(k_residual<T>, dim3(grid_for(n)), dim3(kVecThreads), 0, s, tx, ty, nx, ny,
                     r, p, rho);
}

template <typename T, typename S>
void launch_patch(const BoxDesc* boxes, int m, int max_cells, int max_bx, const S* dinv,
                  const S* coup, const T* rho, T* p, int nx, hipStream_t s, int groups_cap) {
  const BoxLaunch l(m, max_bx, max_cells, sizeof(T), sizeof(S), groups_cap);
  MRCM_BOX_DISPATCH(k_patch, T, S, l.nb, l.dense, l.grid, l.block, l.shm, s, boxes, m, l.gb,
                    l.cp_words, dinv, coup, rho, p, nx);
}

// ---- K right-hand sides per launch ----
namespace {
template <typename T>
RhsPtrs<T> rhs_ptrs(int k, T* const* v) {
  RhsPtrs<T> out{};
  for (int i = 0; i < k; ++i) out.v[i] = v[i];
  return out;
}
void check_k(int k) {
  if (k != 2 && k != 4 && k != 8)
    throw Error(MRCM_EINVAL, "multi-RHS launch of unsupported width");
}
inline size_t group_bytes_k(int k, int nb, int max_cells, size_t t, size_t w) {
  const size_t b = (size_t)ends_of(w) * k * vec_slot_words(nb) * t +
                   (size_t)coupling_words(nb, max_cells, w) * w;
  return (b + 15) / 16 * 16;
}
// As BoxLaunch, for k columns.
struct BoxLaunchK {
  int nb, gb;
  dim3 grid, block;
  size_t shm;
  BoxLaunchK(int k, int m, int max_bx, int max_cells, size_t t, size_t w) {
    nb = launch_cols(m, max_bx, w, pack20_columns(t, w));
    int groups = most_groups(nb, w, group_bytes_k(k, nb, max_cells, t, w));
    if (nb % 2 == 1 && groups <= 0) {
      --nb;
      groups = most_groups(nb, w, group_bytes_k(k, nb, max_cells, t, w));
    }
    if (groups <= 0) throw Error(MRCM_EINVAL, "boxes too large for a multi-RHS launch");
    gb = (int)group_bytes_k(k, nb, max_cells, t, w);
    grid = dim3((m + groups - 1) / groups);
    block = dim3(groups * box_threads(nb, w));
    shm = (size_t)groups * gb;
  }
};
}  // namespace

// Right-hand sides one box launch takes at most, by column width; 1 = the one-RHS kernels,
// once per column.  The bounds of unpacked boxes are what the registers of a lane that owns a
// whole row hold without spilling; with two lanes to a row FP64 boxes of 20 to 32 columns would
// hold four (212 to 256 registers), which has not been timed.  Packed, a lane holds a whole
// row: eight columns spill 148 bytes and four in FP64 leave one wave per SIMD
// (768 x 768 in 4-wide subdomains, four columns of T: 2342 us, two at a time 2260).
constexpr int box_width_k(int nb, size_t w) {
  if (nb % 2 == 1) return w == 8 ? 2 : 4;
  if (w == 8) return nb <= 16 ? 4 : nb <= 48 ? 2 : 1;
  return nb <= 16 ? 8 : nb <= 32 ? 4 : nb <= 48 ? 2 : 1;
}

inline int columns_width(int m, int max_bx, size_t t, size_t w) {
  return box_width_k(launch_cols(m, max_bx, w, pack20_columns(t, w)), w);
}

#define MRCM_BOX_CASE_K(KERNEL, T, S, NB, K, ...)            \
  case 16 * NB + K:                                          \
    if constexpr (K <= box_width_k(NB, sizeof(S)) &&         \
                  (NB != kPacked20 || pack20_columns(sizeof(T), sizeof(S)))) \
      launch_box(KERNEL<T, S, NB, K>, __VA_ARGS__);          \
    break;
#define MRCM_BOX_DISPATCH_K(KERNEL, T, S, nb, kk, ...)       \
  do {                                                       \
    switch (16 * (nb) + (kk)) {                              \
      MRCM_BOX_CASE_K(KERNEL, T, S, 16, 8, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 16, 4, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 16, 2, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, kPacked16, 4, __VA_ARGS__) \
      MRCM_BOX_CASE_K(KERNEL, T, S, kPacked16, 2, __VA_ARGS__) \
      MRCM_BOX_CASE_K(KERNEL, T, S, kPacked20, 4, __VA_ARGS__) \
      MRCM_BOX_CASE_K(KERNEL, T, S, kPacked20, 2, __VA_ARGS__) \
      MRCM_BOX_CASE_K(KERNEL, T, S, 20, 4, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 20, 2, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 24, 4, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 24, 2, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 32, 4, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 32, 2, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 36, 2, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 40, 2, __VA_ARGS__)      \
      MRCM_BOX_CASE_K(KERNEL, T, S, 48, 2, __VA_ARGS__)      \
    }                                                        \
  } while (0)
#define MRCM_K_DISPATCH(k, CALL) \
  do {                           \
    if ((k) == 2) {              \
      constexpr int K = 2;       \
      CALL;                      \
    } else if ((k) == 4) {       \
      constexpr int K = 4;       \
      CALL;                      \
    } else {                     \
      constexpr int K = 8;       \
      CALL;                      \
    }                            \
  } while (0)

template <typename T, typename S>
void launch_local_k(int k, const BoxDesc* boxes, int m, int max_cells, int max_bx, const S* dinv,
                    const S* coup, const double* const* r, T* const* p, T* const* e, int nx,
                    const int* dof_off, const int* dof_side, const int* dof_q,
                    const int* dof_face0, const double* face_w, double* mU, double* mP, int nc,
                    hipStream_t s) {
  check_k(k);
  const int kk = std::min(k, columns_width(m, max_bx, sizeof(T), sizeof(S)));
  for (int k0 = 0; k0 < k; k0 += kk) {
    double* u = mU + (long long)k0 * nc;
    double* v = mP + (long long)k0 * nc;
    if (kk == 1) {
      launch_local<T, S>(boxes, m, max_cells, max_bx, dinv, coup, r[k0], p[k0], nx, dof_off,
                         dof_side, dof_q, dof_face0, face_w, u, v, s);
      continue;
    }
    const BoxLaunchK l(kk, m, max_bx, max_cells, sizeof(T), sizeof(S));
    const RhsPtrs<const double> rp = rhs_ptrs(kk, r + k0);
    const RhsPtrs<T> pp = rhs_ptrs(kk, p + k0), ep = rhs_ptrs(kk, e + k0);
    MRCM_BOX_DISPATCH_K(k_local_k, T, S, l.nb, kk, l.grid, l.block, l.shm, s, boxes, m, l.gb,
                        dinv, coup, rp, pp, ep, nx, dof_off, dof_side, dof_q, dof_face0, face_w, u,
                        v, nc);
  }
}

void launch_coarse_rhs_k(int k, const int4* gsrc, const double* gscale, const double* mU,
                         const double* mP, double* g_nd, int np, int nc, hipStream_t s) {
  check_k(k);
  if (np <= 0) return;
  hipLaunchKernelGGL(k_coarse_rhs_k, dim3((np + 255) / 256, k), dim3(256), 0, s, gsrc, gscale,
                     mU, mP, g_nd, np, nc);
}

// Columns go in groups of at most 4 (wider ones spill registers) whose LDS
// vector (group width x the largest front) fits in 64 KB.
static int coarse_width(int k, int max_dim) {
  int w = k < 4 ? k : 4;
  while (w > 1 && (size_t)w * (max_dim > 0 ? max_dim : 1) * sizeof(double) > 64 * 1024) w /= 2;
  return w;
}

void launch_coarse_fwd_k(int k, const CChunk* chunks, int nchunks, const double* fwd,
                         const double* g_nd, double* contrib, int maxp, int np, const int* cdest,
                         double* ybuf, const int* idx, double* x, int nc, int max_nf,
                         hipStream_t s) {
  check_k(k);
  if (nchunks <= 0) return;
  const int w = coarse_width(k, max_nf);
  for (int k0 = 0; k0 < k; k0 += w) {
    const double* g = g_nd + (long long)k0 * np;
    double* c = contrib + (long long)k0 * maxp * np;
    double* y = ybuf + (long long)k0 * np;
    double* xk = x + (long long)k0 * nc;
    const size_t shm = sizeof(double) * (size_t)w * (max_nf > 0 ? max_nf : 1);
    const dim3 grid(nchunks), block(coarse_threads(nchunks, true));
    if (w == 1)
      hipLaunchKernelGGL(k_coarse_fwd, grid, block, shm, s, chunks, fwd, g, c, maxp, np, cdest, y,
                         idx, xk);
    else if (w == 2)
      hipLaunchKernelGGL(k_coarse_fwd_k<2>, grid, block, shm, s, chunks, fwd, g, c, maxp, np, cdest,
                         y, idx, xk, nc);
    else
      hipLaunchKernelGGL(k_coarse_fwd_k<4>, grid, block, shm, s, chunks, fwd, g, c, maxp, np, cdest,
                         y, idx, xk, nc);
  }
}

void launch_coarse_bwd_k(int k, const CChunk* chunks, int nchunks, const double* bwd,
                         const int* idx, const double* ybuf, double* x, int max_nu, int np, int nc,
                         hipStream_t s) {
  check_k(k);
  if (nchunks <= 0) return;
  const int w = coarse_width(k, max_nu);
  for (int k0 = 0; k0 < k; k0 += w) {
    const double* y = ybuf + (long long)k0 * np;
    double* xk = x + (long long)k0 * nc;
    const size_t shm = sizeof(double) * (size_t)w * (max_nu > 0 ? max_nu : 1);
    const dim3 grid(nchunks), block(coarse_threads(nchunks, false));
    if (w == 1)
      hipLaunchKernelGGL(k_coarse_bwd, grid, block, shm, s, chunks, bwd, idx, y, xk);
    else if (w == 2)
      hipLaunchKernelGGL(k_coarse_bwd_k<2>, grid, block, shm, s, chunks, bwd, idx, y, xk, np, nc);
    else
      hipLaunchKernelGGL(k_coarse_bwd_k<4>, grid, block, shm, s, chunks, bwd, idx, y, xk, np, nc);
  }
}

template <typename T, typename S>
void launch_reconstruct_k(int k, const BoxDesc* boxes, int m, const S* mbf,
                          const long long* mbf_off, const int* dof_off, const double* xc, int nc,
                          T* const* p, int nx, hipStream_t s) {
  check_k(k);
  const RhsPtrs<T> pp = rhs_ptrs(k, p);
  MRCM_K_DISPATCH(k, hipLaunchKernelGGL((k_reconstruct_k<T, S, K>), dim3(m), dim3(kBoxThreads), 0,
                                        s, boxes, mbf, mbf_off, dof_off, xc, nc, pp, nx));
}

template <typename T, typename S>
void launch_reconstruct_mfma(int mode, const BoxDesc* boxes, int m, const S* mbf,
                             const long long* mbf_off, const int* dof_off, const double* xc,
                             int nc, T* const* p, int nx, hipStream_t s) {
  const RhsPtrs<T> pp = rhs_ptrs(8, p);
  if constexpr (sizeof(T) == 4) {
    if (mode == 2) {
      hipLaunchKernelGGL((k_reconstruct_mfma<T, S, 1>), dim3(m), dim3(kBoxThreads), 0, s, boxes,
                         mbf, mbf_off, dof_off, xc, nc, pp, nx);
      return;
    }
  }
  hipLaunchKernelGGL((k_reconstruct_mfma<T, S, 0>), dim3(m), dim3(kBoxThreads), 0, s, boxes, mbf,
                     mbf_off, dof_off, xc, nc, pp, nx);
}

template <typename T>
void launch_residual_k(int k, const T* tx, const T* ty, int nx, int ny, const double* const* r,
                       const T* const* p, T* const* rho, hipStream_t s) {
  check_k(k);
  const long long n = (long long)nx * ny;
  hipLaunchKernelGGL(k_residual_k<T>, dim3(grid_for(n), k), dim3(kVecThreads), 0, s, tx, ty, nx,
                     ny, rhs_ptrs(k, r), rhs_ptrs(k, p), rhs_ptrs(k, rho));
}

template <typename T, typename S>
void launch_patch_k(int k, const BoxDesc* boxes, int m, int max_cells, int max_bx, const S* dinv,
                    const S* coup, const T* const* rho, T* const* p, T* const* e, int nx,
                    hipStream_t s) {
  check_k(k);
  const int kk = std::min(k, columns_width(m, max_bx, sizeof(T), sizeof(S)));
  for (int k0 = 0; k0 < k; k0 += kk) {
    if (kk == 1) {
      launch_patch<T, S>(boxes, m, max_cells, max_bx, dinv, coup, rho[k0], p[k0], nx, s);
      continue;
    }
    const BoxLaunchK l(kk, m, max_bx, max_cells, sizeof(T), sizeof(S));
    const RhsPtrs<const T> rp = rhs_ptrs(kk, rho + k0);
    const RhsPtrs<T> pp = rhs_ptrs(kk, p + k0), ep = rhs_ptrs(kk, e + k0);
    MRCM_BOX_DISPATCH_K(k_patch_k, T, S, l.nb, kk, l.grid, l.block, l.shm, s, boxes, m, l.gb,
                        dinv, coup, rp, pp, ep, nx);
  }
}

template <typename T>
void launch_finalize_k(int k, const T* const* p, long long n, int noflow, double* const* z,
                       double* partials, hipStream_t s) {
  check_k(k);
  const int nb = vec_blocks(n);
  const RhsPtrs<const T> pp = rhs_ptrs(k, p);
  if (noflow)
    hipLaunchKernelGGL(k_sum_k<T>, dim3(nb, k), dim3(kVecThreads), 0, s, pp, n, partials);
  hipLaunchKernelGGL(k_finalize_k<T>, dim3(nb, k), dim3(kVecThreads), 0, s, pp, n,
                     noflow ? partials : (const double*)nullptr, nb, rhs_ptrs(k, z));
}

template <typename T>
void launch_finalize(const T* p, long long n, int noflow, double* z, double* partials,
                     hipStream_t s) {
  const int nb = vec_blocks(n);
  if (noflow) hipLaunchKernelGGL(k_sum<T>, dim3(nb), dim3(kVecThreads), 0, s, p, n, partials);
  hipLaunchKernelGGL(k_finalize<T>, dim3(nb), dim3(kVecThreads), 0, s, p, n,
                     noflow ? partials : (const double*)nullptr, nb, z);
}

void launch_convert(const double* src, float* dst, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_convert, dim3(grid_for(n)), dim3(kVecThreads), 0, s, src, dst, n);
}

void launch_resid_norm(const double* tx, const double* ty, int nx, int ny, const double* b,
                       const double* p, double* r, double* mail, int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_resid_norm, dim3(nb), dim3(kVecThreads), 0, s, tx, ty, nx, ny, b, p, r,
                     mail);
}

void launch_zero(double* v, long long n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_zero, dim3(grid_for(n)), dim3(kVecThreads), 0, s, v, n);
}

void launch_scale(double* v, long long n, double alpha, hipStream_t s) {
  hipLaunchKernelGGL(k_scale, dim3(grid_for(n)), dim3(kVecThreads), 0, s, v, n, alpha);
}

namespace {
void launch_tail_rest(const TailCols& cols, int k, hipStream_t s) {
  int maxj = 0;
  for (int i = 0; i < k; ++i) maxj = cols.c[i].j > maxj ? cols.c[i].j : maxj;
  const dim3 grid(cols.c[0].nb, k), block(kVecThreads);
  for (int i = 0; i <= maxj; ++i) hipLaunchKernelGGL(k_tail_mgs, grid, block, 0, s, cols, i);
  hipLaunchKernelGGL(k_tail_norm, grid, block, 0, s, cols);
}
}  // namespace

void launch_tail(const TailCols& cols, int k, hipStream_t s) {
  if (k < 1 || k > kMaxRhs) throw Error(MRCM_EINVAL, "launch of unsupported width");
  hipLaunchKernelGGL(k_tail_start, dim3(cols.c[0].nb, k), dim3(kVecThreads), 0, s, cols);
  launch_tail_rest(cols, k, s);
}

template <typename T>
void launch_tail_finish(const TailCol& col, const T* p, int noflow, double* z, double* partials,
                        hipStream_t s) {
  if (noflow)
    hipLaunchKernelGGL(k_sum<T>, dim3(col.nb), dim3(kVecThreads), 0, s, p, col.n, partials);
  hipLaunchKernelGGL(k_tail_finish<T>, dim3(col.nb), dim3(kVecThreads), 0, s, col, p,
                     noflow ? partials : (const double*)nullptr, z);
  TailCols cols{};
  cols.c[0] = col;
  launch_tail_rest(cols, 1, s);
}
template void launch_tail_finish<float>(const TailCol&, const float*, int, double*, double*,
                                        hipStream_t);
template void launch_tail_finish<double>(const TailCol&, const double*, int, double*, double*,
                                         hipStream_t);

void launch_mgs_step(const double* part_in, double* part_out, int nb, double* hcol, int i,
                     double* w, const double* vi, const double* vnext, long long n,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_mgs_step, dim3(nb), dim3(kVecThreads), 0, s, part_in, part_out, nb, hcol, i,
                     w, vi, vnext, n);
}

void launch_norm_scale(const double* part_in, int nb, const double* hcol, double* mail, int j,
                       double* w, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_norm_scale, dim3(nb), dim3(kVecThreads), 0, s, part_in, nb, hcol, mail, j,
                     w, n);
}

void launch_update(double* p, const double* Z, const double* y, int k, long long n,
                   hipStream_t s) {
  // in slices of kMaxUpdate vectors: p is updated in the same order
  for (int i0 = 0; i0 < k; i0 += kMaxUpdate) {
    const int ki = k - i0 < kMaxUpdate ? k - i0 : kMaxUpdate;
    UpdateY u{};
    for (int i = 0; i < ki; ++i) u.v[i] = y[i0 + i];
    hipLaunchKernelGGL(k_update, dim3(grid_for(n)), dim3(kVecThreads), 0, s, p,
                       Z + (long long)i0 * n, u, ki, n);
  }
}

void launch_sumsq(const double* x, long long n, double* mail, int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_sumsq, dim3(nb), dim3(kVecThreads), 0, s, x, n, mail);
}

// ---- launches over several contexts ----------------------------------------
namespace {

// The column whose workgroup range [pre[c], pre[c + 1]) holds workgroup b
// (the largest c with pre[c] <= b; empty ranges are skipped).
__device__ __forceinline__ int many_col(const int* __restrict__ pre, int ncol, int b) {
  int lo = 0, hi = ncol - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ Blk many_blk(const int* __restrict__ pre, int c) {
  return Blk{(int)blockIdx.x - pre[c], pre[c + 1] - pre[c]};
}

template <typename T, typename S, int NB, bool DENSE>
__global__ void MRCM_BOX_KERNEL(T, S, NB, DENSE)
    k_local_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol,
                 int group_bytes, int cp_words) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  local_body<T, S, NB, DENSE>(many_blk(pre, c), a.lbox, a.m, group_bytes, cp_words,
                           static_cast<const S*>(a.ldinv), static_cast<const S*>(a.lcoup), a.r,
                           static_cast<T*>(a.p), a.nx, a.dof_off, a.dof_side, a.dof_q,
                           a.dof_face0, a.face_w, a.mU, a.mP);
}

__global__ void k_coarse_rhs_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre,
                                  int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  coarse_rhs_body(many_blk(pre, c), a.gsrc, a.gscale, a.mU, a.mP, a.g_nd, a.np);
}

__global__ void __launch_bounds__(kVecThreads)
    k_coarse_fwd_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre,
                      const int* __restrict__ first, int ncol, int refine) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  const int q = first[c] + (int)blockIdx.x - pre[c];
  coarse_fwd_body(a.chunks[q], a.cfwd, refine ? a.rnd : a.g_nd, a.contrib, a.maxp, a.np,
                  a.cdest, a.ybuf, a.cidx, refine ? a.dx : a.xc);
}

__global__ void __launch_bounds__(kVecThreads)
    k_coarse_bwd_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre,
                      const int* __restrict__ first, int ncol, int refine) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  const int q = first[c] + (int)blockIdx.x - pre[c];
  coarse_bwd_body(a.chunks[q], a.cbwd, a.cidx, a.ybuf, refine ? a.dx : a.xc);
}

__global__ void k_coarse_resid_many(const ManyCol* __restrict__ cols,
                                    const int* __restrict__ pre, int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  coarse_resid_body(many_blk(pre, c), 0, a.crp, a.cci, a.cv, a.g_nd, a.xc, a.rnd, a.np, a.nc);
}

__global__ void k_coarse_add_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre,
                                  int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  coarse_add_body(many_blk(pre, c), a.xc, a.dx, a.nc);
}

template <typename T, typename S>
__global__ void __launch_bounds__(kBoxThreads)
    k_reconstruct_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  reconstruct_body<T, S>(many_blk(pre, c), a.lbox, static_cast<const S*>(a.mbf), a.mbf_off,
                         a.dof_off, a.xc, static_cast<T*>(a.p), a.nx);
}

template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_residual_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  residual_body<T>(many_blk(pre, c), static_cast<const T*>(a.txT), static_cast<const T*>(a.tyT),
                   a.nx, a.ny, a.r, static_cast<const T*>(a.p), static_cast<T*>(a.rho));
}

template <typename T, typename S, int NB, bool DENSE>
__global__ void MRCM_BOX_KERNEL(T, S, NB, DENSE)
    k_patch_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol,
                 int group_bytes, int cp_words) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  patch_body<T, S, NB, DENSE>(many_blk(pre, c), a.pbox, a.m, group_bytes, cp_words,
                           static_cast<const S*>(a.pdinv), static_cast<const S*>(a.pcoup),
                           static_cast<const T*>(a.rho), static_cast<T*>(a.p), a.nx);
}

template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_sum_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  sum_body<T>(many_blk(pre, c), static_cast<const T*>(a.p), a.n, a.partials);
}

template <typename T>
__global__ void __launch_bounds__(kVecThreads)
    k_finalize_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  finalize_body<T>(many_blk(pre, c), static_cast<const T*>(a.p), a.n,
                   a.noflow ? a.partials : (const double*)nullptr, a.nb, a.z);
}

__global__ void __launch_bounds__(kVecThreads)
    k_arnoldi_start_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre,
                         int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  arnoldi_start_body(many_blk(pre, c), a.tx, a.ty, a.nx, a.ny, a.Z + (long long)a.j * a.n,
                     a.V + (long long)(a.j + 1) * a.n, a.V, a.parts);
}

__global__ void __launch_bounds__(kVecThreads)
    k_mgs_step_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol,
                    int i) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  const long long n = a.n;
  mgs_step_body(many_blk(pre, c), a.parts + (i % 2) * kMaxVecBlocks,
                a.parts + ((i + 1) % 2) * kMaxVecBlocks, a.nb, a.hcol, i,
                a.V + (long long)(a.j + 1) * n, a.V + (long long)i * n,
                i < a.j ? a.V + (long long)(i + 1) * n : (const double*)nullptr, n);
}

__global__ void __launch_bounds__(kVecThreads)
    k_norm_scale_many(const ManyCol* __restrict__ cols, const int* __restrict__ pre, int ncol) {
  const int c = many_col(pre, ncol, blockIdx.x);
  const ManyCol& a = cols[c];
  norm_scale_body(many_blk(pre, c), a.parts + ((a.j + 1) % 2) * kMaxVecBlocks, a.nb, a.hcol,
                  a.mail, a.j + 1, a.V + (long long)(a.j + 1) * a.n, a.n);
}

}  // namespace

template <typename T, typename S>
void launch_local_many(const ManyCol* cols, const int* pre, int ncol, int blocks, int max_cells,
                       BoxGrid g, hipStream_t s) {
  if (blocks <= 0) return;
  const int gb = (int)group_bytes(g.cols, max_cells, sizeof(T), sizeof(S));
  const int cp_words = coupling_words(g.cols, max_cells, sizeof(S));
  MRCM_MANY_DISPATCH(k_local_many, T, S, g.cols, g.dense, dim3(blocks),
                    dim3(g.groups * box_threads(g.cols, sizeof(S))), (size_t)g.groups * gb, s, cols,
                    pre, ncol, gb, cp_words);
}
void launch_coarse_rhs_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                            hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_coarse_rhs_many, dim3(blocks), dim3(256), 0, s, cols, pre, ncol);
}
void launch_coarse_fwd_many(const ManyCol* cols, const int* pre, const int* first, int ncol,
                            int blocks, int refine, int max_nf, hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_coarse_fwd_many, dim3(blocks), dim3(coarse_threads(blocks, true)),
                     sizeof(double) * (size_t)(max_nf > 0 ? max_nf : 1), s, cols, pre, first,
                     ncol, refine);
}
void launch_coarse_bwd_many(const ManyCol* cols, const int* pre, const int* first, int ncol,
                            int blocks, int refine, int max_nu, hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_coarse_bwd_many, dim3(blocks), dim3(coarse_threads(blocks, false)),
                     sizeof(double) * (size_t)(max_nu > 0 ? max_nu : 1), s, cols, pre, first,
                     ncol, refine);
}
void launch_coarse_resid_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                              hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_coarse_resid_many, dim3(blocks), dim3(256), 0, s, cols, pre, ncol);
}
void launch_coarse_add_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                            hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_coarse_add_many, dim3(blocks), dim3(256), 0, s, cols, pre, ncol);
}
template <typename T, typename S>
void launch_reconstruct_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                             hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL((k_reconstruct_many<T, S>), dim3(blocks), dim3(kBoxThreads), 0, s, cols,
                     pre, ncol);
}
template <typename T>
void launch_residual_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                          hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_residual_many<T>, dim3(blocks), dim3(kVecThreads), 0, s, cols, pre, ncol);
}
template <typename T, typename S>
void launch_patch_many(const ManyCol* cols, const int* pre, int ncol, int blocks, int max_cells,
                       BoxGrid g, hipStream_t s) {
  if (blocks <= 0) return;
  const int gb = (int)group_bytes(g.cols, max_cells, sizeof(T), sizeof(S));
  const int cp_words = coupling_words(g.cols, max_cells, sizeof(S));
  MRCM_MANY_DISPATCH(k_patch_many, T, S, g.cols, g.dense, dim3(blocks),
                    dim3(g.groups * box_threads(g.cols, sizeof(S))), (size_t)g.groups * gb, s, cols,
                    pre, ncol, gb, cp_words);
}
template <typename T>
void launch_sum_many(const ManyCol* cols, const int* pre, int ncol, int blocks, hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_sum_many<T>, dim3(blocks), dim3(kVecThreads), 0, s, cols, pre, ncol);
}
template <typename T>
void launch_finalize_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                          hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_finalize_many<T>, dim3(blocks), dim3(kVecThreads), 0, s, cols, pre, ncol);
}
void launch_arnoldi_start_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                               hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_arnoldi_start_many, dim3(blocks), dim3(kVecThreads), 0, s, cols, pre,
                     ncol);
}
void launch_mgs_step_many(const ManyCol* cols, const int* pre, int ncol, int blocks, int i,
                          hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_mgs_step_many, dim3(blocks), dim3(kVecThreads), 0, s, cols, pre, ncol, i);
}
void launch_norm_scale_many(const ManyCol* cols, const int* pre, int ncol, int blocks,
                            hipStream_t s) {
  if (blocks <= 0) return;
  hipLaunchKernelGGL(k_norm_scale_many, dim3(blocks), dim3(kVecThreads), 0, s, cols, pre, ncol);
}
#define MRCM_INSTANTIATE_TS(T, S)                                                              \
  template void launch_local<T, S>(const BoxDesc*, int, int, int, const S*, const S*,          \
                                   const double*, T*, int, const int*, const int*, const int*,   \
                                   const int*, const double*, double*, double*, hipStream_t,     \
                                   int);                                                        \
  template void launch_reconstruct<T, S>(const BoxDesc*, int, const S*, const long long*,       \
                                         const int*, const double*, T*, int, hipStream_t);      \
  template void launch_patch<T, S>(const BoxDesc*, int, int, int, const S*, const S*,          \
                                   const T*, T*, int, hipStream_t, int);                         \
  template void launch_local_k<T, S>(int, const BoxDesc*, int, int, int, const S*, const S*,    \
                                     const double* const*, T* const*, T* const*, int,           \
                                     const int*, const int*, const int*, const int*,            \
                                     const double*, double*, double*, int, hipStream_t);        \
  template void launch_reconstruct_k<T, S>(int, const BoxDesc*, int, const S*,                  \
                                           const long long*, const int*, const double*, int,    \
                                           T* const*, int, hipStream_t);                        \
  template void launch_reconstruct_mfma<T, S>(int, const BoxDesc*, int, const S*,               \
                                              const long long*, const int*, const double*, int, \
                                              T* const*, int, hipStream_t);                     \
  template void launch_patch_k<T, S>(int, const BoxDesc*, int, int, int, const S*, const S*,    \
                                     const T* const*, T* const*, T* const*, int, hipStream_t); \
  template void launch_local_many<T, S>(const ManyCol*, const int*, int, int, int, BoxGrid,     \
                                        hipStream_t);                                           \
  template void launch_reconstruct_many<T, S>(const ManyCol*, const int*, int, int, hipStream_t); \
  template void launch_patch_many<T, S>(const ManyCol*, const int*, int, int, int, BoxGrid,     \
                                        hipStream_t);
#define MRCM_INSTANTIATE_T(T)                                                                  \
  template void launch_residual<T>(const T*, const T*, int, int, const double*, const T*, T*,   \
                                   hipStream_t);                                                \
  template void launch_finalize<T>(const T*, long long, int, double*, double*, hipStream_t);    \
  template void launch_residual_k<T>(int, const T*, const T*, int, int, const double* const*,   \
                                     const T* const*, T* const*, hipStream_t);                  \
  template void launch_finalize_k<T>(int, const T* const*, long long, int, double* const*,      \
                                     double*, hipStream_t);                                     \
  template void launch_residual_many<T>(const ManyCol*, const int*, int, int, hipStream_t);     \
  template void launch_sum_many<T>(const ManyCol*, const int*, int, int, hipStream_t);          \
  template void launch_finalize_many<T>(const ManyCol*, const int*, int, int, hipStream_t);

MRCM_INSTANTIATE_TS(double, double)
MRCM_INSTANTIATE_TS(float, float)
MRCM_INSTANTIATE_TS(double, float)
MRCM_INSTANTIATE_T(double)
MRCM_INSTANTIATE_T(float)

}  // namespace mrcm
