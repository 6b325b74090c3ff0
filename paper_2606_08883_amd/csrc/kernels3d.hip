// HIP kernels of the 3-D path (include/mrcm3d.h), FP64: plane-block LDL^T
// box solves (one workgroup per box, tiled symmetric plane products), trace
// moments with tensor Legendre test functions, reconstruction, and the
// seven-point operator in its forms for smoothing and GMRES (the interface
// solve runs the level kernels of the 2-D path on the 3-D factor).  Every
// reduction has a fixed order.
#include "device3d.h"

namespace mrcm3d {

namespace {

constexpr int kVec3Threads = 256;

__device__ __forceinline__ double legendre_face3(int q, int j, int n) {
  const double xi = (2.0 * j + 1.0) / n - 1.0;
  if (q == 0) return 1.0;
  double pm = 1.0, pq = xi;
  for (int k = 1; k < q; ++k) {
    const double pn = ((2.0 * k + 1.0) * xi * pq - k * pm) / (k + 1.0);
    pm = pq;
    pq = pn;
  }
  return pq;
}

// Global cell of box-local cell q (x fastest, then y, then z).
__device__ __forceinline__ long long global_cell(const Box3& d, int q, int nx, int ny) {
  const int x = q % d.n[0], y = (q / d.n[0]) % d.n[1], z = q / (d.n[0] * d.n[1]);
  return ((long long)(d.lo[2] + z) * ny + (d.lo[1] + y)) * nx + (d.lo[0] + x);
}

// Four consecutive words of a tile, in FP64.
struct Quad3 {
  double v[4];
};
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void load_words(f64x2 (&d)[2], const double* p) {
  d[0] = *reinterpret_cast<const f64x2*>(p);
  d[1] = *reinterpret_cast<const f64x2*>(p + 2);
}
__device__ __forceinline__ void load_words(f32x4 (&d)[1], const float* p) {
  d[0] = *reinterpret_cast<const f32x4*>(p);
}
__device__ __forceinline__ Quad3 words(const f64x2 (&d)[2]) {
  return Quad3{{d[0][0], d[0][1], d[1][0], d[1][1]}};
}
__device__ __forceinline__ Quad3 words(const f32x4 (&d)[1]) {
  return Quad3{{(double)d[0][0], (double)d[0][1], (double)d[0][2], (double)d[0][3]}};
}
template <typename S> struct TileRegs;
template <> struct TileRegs<double> { f64x2 d[2]; };
template <> struct TileRegs<float> { f32x4 d[1]; };

// Sum of v over the four lanes of a quad, in every lane.
template <int CTRL>
__device__ __forceinline__ double quad_perm(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double quad_sum(double v) {
  v += quad_perm<0xB1>(v);  // lanes 1 0 3 2
  return v + quad_perm<0x4E>(v);  // lanes 2 3 0 1
}

// Block LDL^T solve of the box in LDS: us holds b on entry and x on exit in
// planes stop .. bz - 1 (planes below keep their forward values).
//
// A plane's symmetric block D_j^-1 is stored as its 16 x 16 tiles (I, J), J <= I
// (device3d.h).  One wave takes a tile: lane 4 r + c holds words 4 c .. 4 c + 3 of
// row r, which give row r's part of D v (from v_J, summed over the quad of lanes)
// and, off the diagonal, the columns' part (from v_I, summed over the rows once
// per tile column).  Wave w takes the tile columns w and nt - 1 - w, together
// nt + 1 tiles in every wave, so the waves of a box are evenly loaded; every part
// goes to a slot of its own in LDS and row t's thread adds its parts in a fixed
// order.  A wave has the next TR tiles of its stream (which runs on over the
// planes and over the turn of the sweep) in flight in registers, across the
// barriers: the HBM rate, not the latency of a plane step, is what this waits for.
// One thread per row of the block over its cyclic diagonals, as before, read every
// word twice through L1 and waited for each pass of loads (96^3 cube, FP64 / FP32
// words: local 806 / 471 us, patch 737 / 418 us).
template <typename S>
__device__ __forceinline__ void plane_solve(double* us, double* v, const Box3& d,
                                            const S* __restrict__ dinv,
                                            const double* __restrict__ coup, int stop) {
  constexpr int TR = sizeof(S) == 4 ? 10 : 5;
  const int P = d.P, bz = d.n[2], t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nt = (P + 15) / 16;                     // tile rows
  const int rows_last = P - 16 * (nt - 1);
  const int HP = block_words(P);
  double* rp = v + 16 * nt;                         // [tile (I, J)][row]: row parts
  double* cp = rp + 8 * nt * (nt + 1);              // [J][row]: column parts
  const S* D = dinv + d.doff;
  const double* T = coup + d.coff;
  const int na = nt - w, wb = nt - 1 - w;           // tiles of column w; the second column
  const int mine = 2 * w > nt - 1 ? 0 : wb == w ? na : nt + 1;
  const int np = bz + (bz - 1 - stop > 0 ? bz - 1 - stop : 0);
  const int r = lane >> 2, c4 = 4 * (lane & 3);
  auto tile = [&](int q, int& I, int& J) {
    const bool first = q < na;
    J = first ? w : wb;
    I = first ? w + q : wb + (q - na);
  };
  auto plane = [&](int p) { return p < bz ? p : 2 * (bz - 1) - p; };
  auto load = [&](TileRegs<S>& reg, int p, int q) {
    int I, J;
    tile(q < mine ? q : mine - 1, I, J);
    const int nr = I == nt - 1 ? rows_last : 16;
    const int off = 128 * I * (I + 1) + J * nr * 16;
    const S* at = D + (long long)plane(p < np ? p : np - 1) * HP + off;
    load_words(reg.d, at + (unsigned)((r < nr ? r : nr - 1) * 16 + c4));
  };
  TileRegs<S> reg[TR];
  if (mine > 0)
#pragma unroll
    for (int u = 0; u < TR; ++u) load(reg[u], 0, u);
  // v of plane 0 (rows past P stay zero)
  if (t < 16 * nt) v[t] = t < P ? us[t] : 0.0;
  __syncthreads();
  for (int p = 0; p < np; ++p) {
    const int j = plane(p);
    double cs[4] = {0.0, 0.0, 0.0, 0.0}, x[4] = {0.0, 0.0, 0.0, 0.0};
    // the sums over the rows of tile column J's words, into cp
    auto flush = [&](int J) {
      const bool b5 = lane & 32, b4 = lane & 16;
      double k0 = b5 ? cs[2] : cs[0], k1 = b5 ? cs[3] : cs[1];
      k0 += __shfl_xor(b5 ? cs[0] : cs[2], 32, 64);
      k1 += __shfl_xor(b5 ? cs[1] : cs[3], 32, 64);
      double k = b4 ? k1 : k0;
      k += __shfl_xor(b4 ? k0 : k1, 16, 64);
      k += __shfl_xor(k, 8, 64);
      k += __shfl_xor(k, 4, 64);
      if ((lane & 12) == 0) cp[16 * J + c4 + (b5 ? 2 : 0) + (b4 ? 1 : 0)] = k;
    };
    for (int q0 = 0; q0 < mine; q0 += TR) {
#pragma unroll
      for (int u = 0; u < TR; ++u) {
        const int q = q0 + u;
        if (q < mine) {
          int I, J;
          tile(q, I, J);
          if (I == J) {
            if (q > 0) flush(w);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              x[i] = v[16 * J + c4 + i];
              cs[i] = 0.0;
            }
          }
          const Quad3 m = words(reg[u].d);
          double s = m.v[0] * x[0];
#pragma unroll
          for (int i = 1; i < 4; ++i) s = fma(m.v[i], x[i], s);
          s = quad_sum(s);
          if ((lane & 3) == 0) rp[8 * I * (I + 1) + 16 * J + r] = s;
          if (I != J) {
            const double vi = v[16 * I + r];
#pragma unroll
            for (int i = 0; i < 4; ++i) cs[i] = fma(m.v[i], vi, cs[i]);
          }
        }
        const bool wrap = q0 + TR >= mine;
        load(reg[u], wrap ? p + 1 : p, wrap ? u : q + TR);
      }
    }
    if (mine > 0) flush(mine > na ? wb : w);
    __syncthreads();
    if (t < P) {
      const int I = t >> 4, rt = t & 15;
      double s = I + 1 < nt ? cp[t] : 0.0;
      const double* part = rp + 8 * I * (I + 1) + rt;
      for (int J = 0; J <= I; J += 4) {
        double e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = part[16 * (J + i <= I ? J + i : I)];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (J + i <= I) s += e[i];
      }
      const double xj = p < bz ? s : us[j * P + t] + s;
      us[j * P + t] = xj;
      if (p + 1 < np) {
        const int jn = plane(p + 1);
        v[t] = p + 1 < bz ? fma(T[(long long)jn * P + t], xj, us[jn * P + t])
                          : T[(long long)(jn + 1) * P + t] * xj;
      }
    }
    __syncthreads();
  }
}

// LDS: us[cells] | v, rp, cp of plane_solve.  S: the storage type of the plane
// blocks (FP64 or FP32); the arithmetic is FP64.
template <typename S>
__global__ void __launch_bounds__(kBox3MaxThreads)
    k_local3(const Box3* __restrict__ boxes, const S* __restrict__ dinv,
             const double* __restrict__ coup, const double* __restrict__ r,
             double* __restrict__ p, int nx, int ny, const int* __restrict__ dof_off,
             const Dof3* __restrict__ dofs, const int* __restrict__ fin,
             const int* __restrict__ fout, const double* __restrict__ fw,
             double* __restrict__ mU, double* __restrict__ mP) {
  extern __shared__ double sm3[];
  const int i = blockIdx.x;
  const Box3 d = boxes[i];
  const int cells = d.P * d.n[2];
  double* us = sm3;
  double* v = sm3 + cells;
  for (int q = threadIdx.x; q < cells; q += blockDim.x) us[q] = r[global_cell(d, q, nx, ny)];
  __syncthreads();
  if (d.pin && threadIdx.x == 0) us[0] = 0.0;
  __syncthreads();
  plane_solve(us, v, d, dinv, coup, d.olo[2] > 0 ? d.olo[2] - 1 : 0);
  // p on the owned cells
  const int oc = d.on[0] * d.on[1] * d.on[2];
  for (int q = threadIdx.x; q < oc; q += blockDim.x) {
    const int x = q % d.on[0], y = (q / d.on[0]) % d.on[1], z = q / (d.on[0] * d.on[1]);
    const int lq = ((d.olo[2] + z) * d.n[1] + d.olo[1] + y) * d.n[0] + d.olo[0] + x;
    p[global_cell(d, lq, nx, ny)] = us[lq];
  }
  // trace moments of every dof of the subdomain, eight lanes to a dof (the 64
  // faces of a dof one after the other, with a division or two each, took as long
  // as the solve)
  const int sub = threadIdx.x & 7;
  for (int k0 = dof_off[i]; k0 < dof_off[i + 1]; k0 += blockDim.x / 8) {
    const int k = k0 + (threadIdx.x >> 3);
    const bool on = k < dof_off[i + 1];
    const Dof3 q = dofs[on ? k : k0];
    double su = 0.0, sp = 0.0;
    for (int f = sub; f < q.nf; f += 8) {
      const int ff = q.f0 + f;
      const double pin = us[fin[ff]], pout = us[fout[ff]];
      const double bv = legendre_face3(q.a, f % q.n0, q.n0) * legendre_face3(q.b, f / q.n0, q.n1);
      const double U = fma(fw[4LL * ff + 1], pout, fw[4LL * ff] * pin);
      const double Pi = fma(fw[4LL * ff + 3], pout, fw[4LL * ff + 2] * pin);
      su = fma(bv, U, su);
      sp = fma(bv, Pi, sp);
    }
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) {
      su += __shfl_xor(su, off, 64);
      sp += __shfl_xor(sp, off, 64);
    }
    if (on && sub == 0) {
      mU[k] = su;
      mP[k] = sp;
    }
  }
}

template <typename S>
__global__ void __launch_bounds__(kBox3MaxThreads)
    k_patch3(const Box3* __restrict__ boxes, const S* __restrict__ dinv,
             const double* __restrict__ coup, const double* __restrict__ rho,
             double* __restrict__ p, int nx, int ny) {
  extern __shared__ double sm3[];
  const Box3 d = boxes[blockIdx.x];
  const int cells = d.P * d.n[2];
  double* us = sm3;
  double* v = sm3 + cells;
  for (int q = threadIdx.x; q < cells; q += blockDim.x) us[q] = rho[global_cell(d, q, nx, ny)];
  __syncthreads();
  if (d.pin && threadIdx.x == 0) us[0] = 0.0;
  __syncthreads();
  plane_solve(us, v, d, dinv, coup, d.olo[2]);
  const int oc = d.on[0] * d.on[1] * d.on[2];
  for (int q = threadIdx.x; q < oc; q += blockDim.x) {
    const int x = q % d.on[0], y = (q / d.on[0]) % d.on[1], z = q / (d.on[0] * d.on[1]);
    const int lq = ((d.olo[2] + z) * d.n[1] + d.olo[1] + y) * d.n[0] + d.olo[0] + x;
    const long long c = global_cell(d, lq, nx, ny);
    p[c] += us[lq];
  }
}

__device__ __forceinline__ double wave_sum3(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// p[Omega_i] += P_i x_i, a thread per owned cell (blockIdx.y: cells kBox3Threads at a
// time), eight basis functions in flight: a cell's sum is a chain of loads otherwise
// (60 x 44 x 36 in 8 x 8 x 8 subdomains: 16.6 -> 6.1 us; 96^3 42.0 -> 41.1, 4.1 TB/s).
__global__ void __launch_bounds__(kBox3Threads)
    k_reconstruct3(const Box3* __restrict__ boxes, const double* __restrict__ mbf,
                   const long long* __restrict__ mbf_off, const int* __restrict__ dof_off,
                   const double* __restrict__ x, double* __restrict__ p, int nx, int ny) {
  const int i = blockIdx.x;
  const Box3 d = boxes[i];
  const int k0 = dof_off[i], nk = dof_off[i + 1] - k0;
  const int oc = d.on[0] * d.on[1] * d.on[2];
  const int q = blockIdx.y * kBox3Threads + threadIdx.x;
  if (q >= oc) return;
  const double* Pm = mbf + mbf_off[i] + q;
  const int xx = q % d.on[0], y = (q / d.on[0]) % d.on[1], z = q / (d.on[0] * d.on[1]);
  const int lq = ((d.olo[2] + z) * d.n[1] + d.olo[1] + y) * d.n[0] + d.olo[0] + xx;
  const long long c = global_cell(d, lq, nx, ny);
  double s = p[c];
  for (int kb = 0; kb < nk; kb += 8) {
    double m[8], v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = kb + e < nk ? kb + e : nk - 1;
      m[e] = Pm[(long long)k * oc];
      v[e] = x[k0 + k];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) s = kb + e < nk ? fma(m[e], v[e], s) : s;
  }
  p[c] = s;
}

// The seven-point stencil at cell c: sum over the faces of t_f (x_c - x_c'),
// boundary faces coupled to zero.  A missing neighbour is read at the cell itself and
// its term left out, so that no load waits for a branch; one division gives the
// row, one the plane (with the sums of A z: 60 x 44 x 36 10.2 -> 5.6 us, 96^3 17.0 ->
// 13.7; with branches around the neighbours and three divisions before).
__device__ __forceinline__ double stencil3(const double* __restrict__ tx,
                                           const double* __restrict__ ty,
                                           const double* __restrict__ tz, int nx, int ny, int nz,
                                           long long c, const double* __restrict__ x) {
  const long long row = c / nx, plane = (long long)nx * ny;
  const int ix = (int)(c - row * nx), iz = (int)(row / ny), iy = (int)(row - (long long)iz * ny);
  const long long fx = c + row, fy = c + (long long)iz * nx;
  const double tW = tx[fx], tE = tx[fx + 1], tS = ty[fy], tN = ty[fy + nx], tB = tz[c],
               tT = tz[c + plane];
  const bool hw = ix > 0, he = ix + 1 < nx, hs = iy > 0, hn = iy + 1 < ny, hb = iz > 0,
             ht = iz + 1 < nz;
  const double xc = x[c], xw = x[hw ? c - 1 : c], xe = x[he ? c + 1 : c],
               xs = x[hs ? c - nx : c], xn = x[hn ? c + nx : c], xb = x[hb ? c - plane : c],
               xt = x[ht ? c + plane : c];
  double v = (tW + tE + tS + tN + tB + tT) * xc;
  v = hw ? fma(-tW, xw, v) : v;
  v = he ? fma(-tE, xe, v) : v;
  v = hs ? fma(-tS, xs, v) : v;
  v = hn ? fma(-tN, xn, v) : v;
  v = hb ? fma(-tB, xb, v) : v;
  v = ht ? fma(-tT, xt, v) : v;
  return v;
}

__global__ void __launch_bounds__(kVec3Threads)
    k_op3(const double* __restrict__ tx, const double* __restrict__ ty,
          const double* __restrict__ tz, int nx, int ny, int nz, const double* __restrict__ x,
          double* __restrict__ y, const double* __restrict__ r, int mode) {
  const long long n = (long long)nx * ny * nz;
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x) {
    const double a = stencil3(tx, ty, tz, nx, ny, nz, c, x);
    y[c] = mode == 0 ? a : r[c] - a;
  }
}

__device__ __forceinline__ double block_sum3(double v, double* red) {
  v = wave_sum3(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += red[k];
  return s;
}

// mode 0: w = A z, partials of w . v0 (v0 = aux); mode 1: r = b - A p (b when
// p is NULL; b = aux), partials of r^2, which the host waits for (mailbox.h).
__global__ void __launch_bounds__(kVec3Threads)
    k_op_reduce3(const double* __restrict__ tx, const double* __restrict__ ty,
                 const double* __restrict__ tz, int nx, int ny, int nz,
                 const double* __restrict__ x, double* __restrict__ out,
                 const double* __restrict__ aux, double* __restrict__ partials, int mode) {
  __shared__ double red[kVec3Threads / 64];
  const long long n = (long long)nx * ny * nz;
  double s = 0.0;
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x) {
    if (mode == 0) {
      const double w = stencil3(tx, ty, tz, nx, ny, nz, c, x);
      out[c] = w;
      s = fma(w, aux[c], s);
    } else {
      const double rr = x ? aux[c] - stencil3(tx, ty, tz, nx, ny, nz, c, x) : aux[c];
      out[c] = rr;
      s = fma(rr, rr, s);
    }
  }
  s = block_sum3(s, red);
  if (threadIdx.x == 0) {
    if (mode == 0)
      partials[blockIdx.x] = s;
    else
      __hip_atomic_store(partials + blockIdx.x, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// b = f h^2 plus t_f g_f on every Dirichlet boundary face (t_f = 2 K_c
// there), sides in the order W, E, S, N, B, T; g: the six sides' face values
// concatenated (W, E: z ny + y; S, N: z nx + x; B, T: y nx + x).
__global__ void __launch_bounds__(kVec3Threads)
    k_rhs3(const double* __restrict__ tx, const double* __restrict__ ty,
           const double* __restrict__ tz, int nx, int ny, int nz, int bcmask,
           const double* __restrict__ f, const double* __restrict__ g, double h,
           double* __restrict__ b) {
  const long long n = (long long)nx * ny * nz;
  const long long oW = 0, oE = (long long)ny * nz, oS = 2LL * ny * nz,
                  oN = oS + (long long)nx * nz, oB = oN + (long long)nx * nz,
                  oT = oB + (long long)nx * ny;
  for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n;
       c += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(c % nx), iy = (int)((c / nx) % ny), iz = (int)(c / ((long long)nx * ny));
    double v = f ? f[c] * h * h : 0.0;
    if (g) {
      const long long fx = ((long long)iz * ny + iy) * (nx + 1) + ix;
      const long long fy = ((long long)iz * (ny + 1) + iy) * nx + ix;
      const long long fz = ((long long)iz * ny + iy) * nx + ix;
      if (ix == 0 && (bcmask & 1)) v += tx[fx] * g[oW + (long long)iz * ny + iy];
      if (ix == nx - 1 && (bcmask & 2)) v += tx[fx + 1] * g[oE + (long long)iz * ny + iy];
      if (iy == 0 && (bcmask & 4)) v += ty[fy] * g[oS + (long long)iz * nx + ix];
      if (iy == ny - 1 && (bcmask & 8)) v += ty[fy + nx] * g[oN + (long long)iz * nx + ix];
      if (iz == 0 && (bcmask & 16)) v += tz[fz] * g[oB + (long long)iy * nx + ix];
      if (iz == nz - 1 && (bcmask & 32))
        v += tz[fz + (long long)nx * ny] * g[oT + (long long)iy * nx + ix];
    }
    b[c] = v;
  }
}

inline int grid3(long long n) {
  long long b = (n + kVec3Threads - 1) / kVec3Threads;
  return (int)(b < 1 ? 1 : b > 4096 ? 4096 : b);
}

}  // namespace

// Threads of a box launch: a wave per two tile columns of the largest plane
// (which is at least one thread per cell of it), and the LDS of its boxes.
inline int tile_rows(int max_plane) { return (max_plane + 15) / 16; }
inline int box3_threads(int max_plane) { return 64 * ((tile_rows(max_plane) + 1) / 2); }
inline size_t box3_lds(int max_cells, int max_plane) {
  const int nt = tile_rows(max_plane);
  return sizeof(double) * ((size_t)max_cells + 16 * nt + 8 * nt * (nt + 1) + 16 * nt);
}

template <typename S>
void launch_local3(const Box3* boxes, int m, int max_cells, int max_plane, const S* dinv,
                   const double* coup, const double* r, double* p, int nx, int ny,
                   const int* dof_off, const Dof3* dofs, const int* fin, const int* fout,
                   const double* fw, double* mU, double* mP, hipStream_t s) {
  if (m <= 0) return;
  const size_t shm = box3_lds(max_cells, max_plane);
  hipLaunchKernelGGL(k_local3<S>, dim3(m), dim3(box3_threads(max_plane)), shm, s, boxes, dinv,
                     coup, r, p, nx, ny, dof_off, dofs, fin, fout, fw, mU, mP);
}
template <typename S>
void launch_patch3(const Box3* boxes, int m, int max_cells, int max_plane, const S* dinv,
                   const double* coup, const double* rho, double* p, int nx, int ny,
                   hipStream_t s) {
  if (m <= 0) return;
  const size_t shm = box3_lds(max_cells, max_plane);
  hipLaunchKernelGGL(k_patch3<S>, dim3(m), dim3(box3_threads(max_plane)), shm, s, boxes, dinv,
                     coup, rho, p, nx, ny);
}
#define MRCM3D_INSTANTIATE(S)                                                                  \
  template void launch_local3<S>(const Box3*, int, int, int, const S*, const double*,          \
                                 const double*, double*, int, int, const int*, const Dof3*,    \
                                 const int*, const int*, const double*, double*, double*,      \
                                 hipStream_t);                                                 \
  template void launch_patch3<S>(const Box3*, int, int, int, const S*, const double*,          \
                                 const double*, double*, int, int, hipStream_t);
MRCM3D_INSTANTIATE(double)
MRCM3D_INSTANTIATE(float)
#undef MRCM3D_INSTANTIATE
void launch_reconstruct3(const Box3* boxes, int m, int max_owned, const double* mbf,
                         const long long* mbf_off, const int* dof_off, const double* x, double* p,
                         int nx, int ny, hipStream_t s) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_reconstruct3, dim3(m, (max_owned + kBox3Threads - 1) / kBox3Threads),
                     dim3(kBox3Threads), 0, s, boxes, mbf, mbf_off, dof_off, x, p, nx, ny);
}
void launch_op3(const double* tx, const double* ty, const double* tz, int nx, int ny, int nz,
                const double* x, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_op3, dim3(grid3((long long)nx * ny * nz)), dim3(kVec3Threads), 0, s, tx,
                     ty, tz, nx, ny, nz, x, y, (const double*)nullptr, 0);
}
void launch_residual3(const double* tx, const double* ty, const double* tz, int nx, int ny,
                      int nz, const double* r, const double* p, double* rho, hipStream_t s) {
  hipLaunchKernelGGL(k_op3, dim3(grid3((long long)nx * ny * nz)), dim3(kVec3Threads), 0, s, tx,
                     ty, tz, nx, ny, nz, p, rho, r, 1);
}
void launch_rhs3(const double* tx, const double* ty, const double* tz, int nx, int ny, int nz,
                 int bcmask, const double* f, const double* g, double h, double* b,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_rhs3, dim3(grid3((long long)nx * ny * nz)), dim3(kVec3Threads), 0, s, tx,
                     ty, tz, nx, ny, nz, bcmask, f, g, h, b);
}
void launch_arnoldi_start3(const double* tx, const double* ty, const double* tz, int nx, int ny,
                           int nz, const double* z, double* w, const double* v0,
                           double* partials, int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_op_reduce3, dim3(nb), dim3(kVec3Threads), 0, s, tx, ty, tz, nx, ny, nz, z,
                     w, v0, partials, 0);
}
void launch_resid_norm3(const double* tx, const double* ty, const double* tz, int nx, int ny,
                        int nz, const double* b, const double* p, double* r, double* mail,
                        int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_op_reduce3, dim3(nb), dim3(kVec3Threads), 0, s, tx, ty, tz, nx, ny, nz, p,
                     r, b, mail, 1);
}

}  // namespace mrcm3d
