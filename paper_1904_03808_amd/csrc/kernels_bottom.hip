// The two coarsest levels of a V-cycle in two launches (Sec. 3.6, gfx950).
//
// The cycle on the level above the coarsest (smoothing from a zero guess, the
// coarsest solve, the correction and smoothing again) is one fixed linear map
// from that level's right-hand side b to its correction x.  Its colours have
// period 2 in x and y and the coarsest operator is the same at every column,
// so the map commutes with shifts by two columns or rows: Fourier modes over
// the cx * cy shifts (cx, cy the coarsest sizes) split it into independent
// blocks of n = 12 (nz - 1) unknowns (component, plane, y parity, x parity).
// The blocks are computed at setup in FP64 (k_bottom_build), for whatever sweeps
// and colour order the handle has, and are held and applied in FP64 in both
// precisions, as the coarsest inverse is.
//
// The map commutes with the reflections in x and y as well, which keep every
// node's colour.  Taken about the nodes' own positions (half a shift for the odd
// columns and rows) and with the z component times i, a block is therefore real,
// and the blocks of (mx, my) and (mx, -my) differ in the y component's sign only:
// 6.5 MB at 8^3 under 16^3 where complex blocks of every mode are 17.6 MB.
//
// What bounds it: the cycle it stands for is 16 colour-pair launches, residual,
// restriction, coarsest solve and correction, each a fixed cost of 3 to 7 us
// and next to no work (8^3 under 16^3: 20 launches, about 75 us).  The map costs
// about what the coarsest inverse's product alone did.
#include <hip/hip_runtime.h>

#include "device.h"

namespace qs {

namespace {

constexpr int kThreads = 512;              // of the kernels that transform b
constexpr int kRows = 32;                  // rows of a block per workgroup
constexpr int kGroups = kThreads / kRows;  // column groups per workgroup
constexpr int kBatch = 8;                  // loads in flight per thread in the transform
constexpr size_t kMaxLds = 64ull << 10;    // bytes a workgroup may take

// Modes (mx, my) kept: one of each conjugate pair.  mx = 0 and 2 mx = cx pair
// (mx, my) with (mx, -my), the other mx with cx - mx.
__host__ __device__ inline int half_y(int cy) { return cy / 2 + 1; }

__host__ __device__ inline int mode_count(int cx, int cy) {
  int n = 0;
  for (int mx = 0; 2 * mx <= cx; ++mx) n += (mx == 0 || 2 * mx == cx) ? half_y(cy) : cy;
  return n;
}

__device__ __forceinline__ void mode_of(int m, int cx, int cy, int* mx, int* my) {
  const int h = half_y(cy);
  if (m < h) {
    *mx = 0;
    *my = m;
  } else {
    *mx = 1 + (m - h) / cy;
    *my = (m - h) % cy;
  }
}

// Position of mode (mx, my), 2 mx <= cx, and whether it is stored conjugated.
__device__ __forceinline__ int mode_index(int mx, int my, int cx, int cy, bool* conj) {
  const int h = half_y(cy);
  *conj = (mx == 0 || 2 * mx == cx) && my >= h;
  if (*conj) my = cy - my;
  return mx == 0 ? my : h + (mx - 1) * cy + my;
}

__host__ __device__ inline int block_count(int cx, int cy) { return (cx / 2 + 1) * half_y(cy); }

// Position of the block that serves mode (mx, my).
__device__ __forceinline__ int block_of(int mx, int my, int cx, int cy) {
  return mx + (cx / 2 + 1) * (2 * my <= cy ? my : cy - my);
}

// Unknown u's factor between the transform at mode (mx, my) and the real blocks.
__device__ __forceinline__ double2 real_factor(int u, int nz, int mx, int my, int cx, int cy) {
  const int ex = u & 1, ey = (u >> 1) & 1, c = u / (4 * (nz - 1));
  const int sy = 2 * my <= cy ? my : my - cy;
  double sn, cs;
  sincospi(static_cast<double>(mx * ex) / cx + static_cast<double>(sy * ey) / cy, &sn, &cs);
  if (c == 2) return make_double2(sn, cs);  // i exp(-i a)
  return c == 1 && sy < 0 ? make_double2(-cs, sn) : make_double2(cs, -sn);
}

// The transform of the node vector f (level dims nx, ny, nz) at mode (mx, my):
// out[(c (nz-1) + k-1) 4 + 2 ey + ex] = sum over shifts of
// f[c][k][2 sy + ey][2 sx + ex] exp(-2 pi i (mx sx / cx + my sy / cy)),
// times the factor of the real blocks.
// y first (rows are read whole, coalesced in x), then x from LDS (part).
template <typename T>
__device__ __forceinline__ void forward_mode(const T* __restrict__ f, int nx, int ny, int nz, int mx,
                                             int my, const double2* __restrict__ twx,
                                             const double2* __restrict__ twy,
                                             double2* __restrict__ part, double2* __restrict__ out) {
  const int cx = nx / 2, cy = ny / 2, P = nx * ny, per = 2 * nx * (nz - 1);
  const size_t C = static_cast<size_t>(nz + 1) * P;
  for (int t = threadIdx.x; t < 3 * per; t += blockDim.x) {
    const int c = t / per, r = t - c * per;
    const int i = r % nx, q = r / nx, ey = q & 1, k = 1 + (q >> 1);
    const T* p = f + c * C + static_cast<size_t>(k) * P + ey * nx + i;
    double2 s = make_double2(0.0, 0.0);
    int ph = 0;  // (my sy) mod cy
    for (int s0 = 0; s0 < cy; s0 += kBatch) {
      T v[kBatch];
#pragma unroll
      for (int q = 0; q < kBatch; ++q) v[q] = p[2 * min(s0 + q, cy - 1) * nx];
#pragma unroll
      for (int q = 0; q < kBatch; ++q)
        if (s0 + q < cy) {
          s.x += static_cast<double>(v[q]) * twy[ph].x;
          s.y -= static_cast<double>(v[q]) * twy[ph].y;
          ph += my;
          if (ph >= cy) ph -= cy;
        }
    }
    part[t] = s;
  }
  __syncthreads();
  const int n = 12 * (nz - 1);
  for (int u = threadIdx.x; u < n; u += blockDim.x) {
    const double2* row = part + (u >> 1) * nx + (u & 1);
    double2 s = make_double2(0.0, 0.0);
    int ph = 0;
    for (int sx = 0; sx < cx; ++sx) {
      const double2 v = row[2 * sx], w = twx[ph];
      s.x += v.x * w.x + v.y * w.y;
      s.y += v.y * w.x - v.x * w.y;
      ph += mx;
      if (ph >= cx) ph -= cx;
    }
    const double2 w = real_factor(u, nz, mx, my, cx, cy);
    out[u] = make_double2(s.x * w.x - s.y * w.y, s.x * w.y + s.y * w.x);
  }
  __syncthreads();
}

__device__ __forceinline__ void load_twiddles(const double2* __restrict__ tw, int cx, int cy,
                                              double2* __restrict__ l) {
  for (int t = threadIdx.x; t < cx + cy; t += blockDim.x) l[t] = tw[t];
  __syncthreads();
}

// One row slice of one mode's block applied to the transform of b, which every
// slice forms itself (b is a few hundred KB and comes from L2): yh[mode][row].
// A workgroup of 512 threads takes 32 rows and splits the columns over sixteen
// groups; 32 consecutive rows of a column are one 256-byte access.  The
// transform's loads go out eight at a time (10.5 us at 8^3 under 16^3 in FP64
// with one load after the other and 256 threads).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_bottom_modes(const double* __restrict__ M,
                                                      const T* __restrict__ b, int nx, int ny, int nz,
                                                      const double2* __restrict__ tw,
                                                      double2* __restrict__ yh) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int cx = nx / 2, cy = ny / 2, n = 12 * (nz - 1);
  double2* ltw = reinterpret_cast<double2*>(smem);
  double2* bh = ltw + cx + cy;
  double2* part = bh + n;  // 6 (nz-1) nx values, later the partial sums
  int mx, my;
  mode_of(blockIdx.x, cx, cy, &mx, &my);
  load_twiddles(tw, cx, cy, ltw);
  forward_mode<T>(b, nx, ny, nz, mx, my, ltw, ltw + cx, part, bh);
  const int rr = threadIdx.x % kRows, g = threadIdx.x / kRows;
  const int row = blockIdx.y * kRows + rr;
  double2 s = make_double2(0.0, 0.0);
  if (row < n) {
    const double* __restrict__ col = M + static_cast<size_t>(block_of(mx, my, cx, cy)) * n * n + row;
#pragma unroll 8
    for (int q = g; q < n; q += kGroups) {
      const double a = col[static_cast<size_t>(q) * n];
      const double2 v = bh[q];
      s.x += a * v.x;
      s.y += a * v.y;
    }
  }
  part[threadIdx.x] = s;
  __syncthreads();
  if (g == 0 && row < n) {
#pragma unroll
    for (int q = 1; q < kGroups; ++q) {
      s.x += part[q * kRows + rr].x;
      s.y += part[q * kRows + rr].y;
    }
    const double2 w = real_factor(row, nz, mx, my, cx, cy);
    yh[static_cast<size_t>(blockIdx.x) * n + row] = make_double2(s.x * w.x + s.y * w.y, s.y * w.x - s.x * w.y);
  }
}

// Back to the nodes, one workgroup per component and plane: y modes first into
// LDS, then x modes straight into x.
template <typename T>
__global__ __launch_bounds__(256) void k_bottom_back(const double2* __restrict__ yh, T* __restrict__ x,
                                                     int nx, int ny, int nz,
                                                     const double2* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int cx = nx / 2, cy = ny / 2, n = 12 * (nz - 1), hx = cx / 2 + 1;
  double2* ltw = reinterpret_cast<double2*>(smem);
  double2* part = ltw + cx + cy;  // [4 parities][cy][hx]
  const int c = blockIdx.x / (nz - 1), k = 1 + blockIdx.x - c * (nz - 1);
  load_twiddles(tw, cx, cy, ltw);
  const int base = (c * (nz - 1) + k - 1) * 4;
  for (int t = threadIdx.x; t < 4 * cy * hx; t += blockDim.x) {
    const int mx = t % hx, q = t / hx, sy = q % cy, par = q / cy;
    double2 s = make_double2(0.0, 0.0);
    int ph = 0;
    for (int my = 0; my < cy; ++my) {
      bool conj;
      const double2 v = yh[static_cast<size_t>(mode_index(mx, my, cx, cy, &conj)) * n + base + par];
      const double vy = conj ? -v.y : v.y;
      const double2 w = ltw[cx + ph];
      s.x += v.x * w.x - vy * w.y;
      s.y += vy * w.x + v.x * w.y;
      ph += sy;
      if (ph >= cy) ph -= cy;
    }
    part[t] = s;
  }
  __syncthreads();
  const double norm = 1.0 / (static_cast<double>(cx) * cy);
  const int P = nx * ny;
  T* px = x + (static_cast<size_t>(c) * (nz + 1) + k) * P;
  for (int t = threadIdx.x; t < P; t += blockDim.x) {
    const int i = t % nx, j = t / nx;
    const int sx = i >> 1;
    const double2* g = part + ((2 * (j & 1) + (i & 1)) * cy + (j >> 1)) * hx;
    double s = g[0].x;
    int ph = 0;
    for (int mx = 1; mx < hx; ++mx) {
      ph += sx;
      if (ph >= cx) ph -= cx;
      const double2 v = g[mx], w = ltw[ph];
      const double re = v.x * w.x - v.y * w.y;
      s += 2 * mx == cx ? re : 2.0 * re;
    }
    px[t] = static_cast<T>(s * norm);
  }
}

// A stencil entry between components c and d, at the phase a between the two
// nodes, as it enters the real blocks (f_c conj(f_d) exp(i a), f = 1, 1, i, whose
// imaginary part cancels against the mirrored entry's).
__device__ __forceinline__ double real_phase(int c, int d, double sn, double cs) {
  return (c == 2) == (d == 2) ? cs : (c == 2 ? -sn : sn);
}

// The map's blocks, one column per wavefront.  In the real basis the level's
// operator couples plane k to k - 1, k, k + 1 and each (y, x) parity to the same
// or the other one by 108 numbers a plane (G, the stencil summed over its mirrored
// entries at the mode's phases), the transfers are products of cosines, and the
// coarsest inverse is a matrix B of 3 (nzc - 1) unknowns: a column is the cycle run
// on one unit vector of 12 (nz - 1) values in LDS.  Everything is a fixed cost of
// about forty short phases, and all columns of all blocks are one launch.  Running
// the level kernels on every unit right-hand side instead took 20 launches each:
// setup of 16^3 (map of 8^3 over 4^3, 84 unknowns) 6.9 -> 0.74 ms, of 96^3 36.3 ->
// 25.5 ms, of 256^3 474 -> 457 ms, the rest of it on the host.
__global__ __launch_bounds__(256) void k_bottom_build(const double* __restrict__ S,
                                                      const double* __restrict__ Dinv,
                                                      const double* __restrict__ Ainv, int ncoarse, int nx,
                                                      int ny, int nz, const double2* __restrict__ tw,
                                                      unsigned order, int n_pre, int n_post,
                                                      double* __restrict__ M) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int cx = nx / 2, cy = ny / 2, Z = nz - 1, ZC = nz / 2 - 1, n = 12 * Z, m = 3 * ZC;
  const int mx = blockIdx.x % (cx / 2 + 1), my = blockIdx.x / (cx / 2 + 1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  double* G = reinterpret_cast<double*>(smem);  // [plane][oz][parity change][c][d]
  double* B = G + 108 * Z;                      // [c, K][d, K']
  double* y = B + m * m + 2 * n * wave;         // this wavefront's column
  double* r = y + n;                            // its residual, then the coarse vectors
  double sx, cosx, sy, cosy;                    // of the phase of one column, one row
  sincospi(static_cast<double>(mx) / cx, &sx, &cosx);
  sincospi(static_cast<double>(my) / cy, &sy, &cosy);
  for (int e = threadIdx.x; e < 108 * Z; e += blockDim.x) {
    const int d = e % 3, c = e / 3 % 3, par = e / 9 % 4, oz = e / 36 % 3, k = 1 + e / 108;
    const int px = par & 1, py = par >> 1;
    double g = 0.0;
    for (int oy = -py; oy <= py; oy += 2)
      for (int ox = -px; ox <= px; ox += 2) {
        const double c1 = ox ? cosx : 1.0, s1 = ox * sx, c2 = oy ? cosy : 1.0, s2 = oy * sy;
        g += S[(k * 27 + oz * 9 + (oy + 1) * 3 + ox + 1) * 9 + c * 3 + d] *
             real_phase(c, d, s1 * c2 + c1 * s2, c1 * c2 - s1 * s2);
      }
    G[e] = g;
  }
  for (int e = threadIdx.x; e < m * m; e += blockDim.x) {
    const int q = e % m, row = e / m;
    const double* a = Ainv + static_cast<size_t>(row) * cx * cy * ncoarse + q * cx * cy;
    double g = 0.0;
    for (int J = 0; J < cy; ++J) {
      const double2 wy = tw[cx + my * J % cy];
      for (int I = 0; I < cx; ++I) {
        const double2 wx = tw[mx * I % cx];
        g += a[J * cx + I] * real_phase(row / ZC, q / ZC, wx.y * wy.x + wx.x * wy.y,
                                        wx.x * wy.x - wx.y * wy.y);
      }
    }
    B[e] = g;
  }
  const int u = blockIdx.y * waves + wave;  // a wavefront past the last column runs along
  for (int t = lane; t < n; t += 64) y[t] = 0.0;
  __syncthreads();
  // sum of the operator's row (c, k, par) times y, with or without the node itself
  auto row_sum = [&](int c, int k, int par, bool own) {
    double s = 0.0;
    for (int oz = 0; oz < 3; ++oz) {
      const int kk = k + oz - 1;
      if (kk < 1 || kk > Z) continue;
      const double* g = G + ((k - 1) * 3 + oz) * 36 + c * 3;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (oz == 1 && q == 0 && !own) continue;
#pragma unroll
        for (int d = 0; d < 3; ++d) s += g[q * 9 + d] * y[(d * Z + kk - 1) * 4 + (par ^ q)];
      }
    }
    return s;
  };
  auto smooth = [&](int sweeps, bool reverse) {
    for (int q = 0; q < 8 * sweeps; ++q) {
      const int col = order >> (4 * (reverse ? 7 - q % 8 : q % 8)) & 7;
      const int par = col & 3, first = col & 4 ? 1 : 2;
      // lane: a component and plane of the colour (at most 48)
      const int c = lane % 3, k = first + 2 * (lane / 3);
      const int t = (c * Z + k - 1) * 4 + par;
      double v = 0.0;
      if (k <= Z) v = Dinv[k * 9 + c * 4] * ((t == u ? 1.0 : 0.0) - row_sum(c, k, par, false));
      if (k <= Z) y[t] = v;  // nodes of one colour do not couple
      __syncthreads();
    }
  };
  smooth(n_pre, false);
  for (int t = lane; t < n; t += 64)
    r[t] = (t == u ? 1.0 : 0.0) - row_sum(t / (4 * Z), 1 + t / 4 % Z, t & 3, true);
  __syncthreads();
  const int c = lane / ZC, K = 1 + lane % ZC;  // coarse unknown of this lane (m <= 45)
  double v = 0.0;
  if (lane < m)
    for (int dz = -1; dz <= 1; ++dz) {
      const double* p = r + (c * Z + 2 * K + dz - 1) * 4;
      v += (dz ? 0.5 : 1.0) * (p[0] + cosx * p[1] + cosy * (p[2] + cosx * p[3]));
    }
  __syncthreads();
  if (lane < m) r[lane] = v;
  __syncthreads();
  v = 0.0;
  if (lane < m)
    for (int q = 0; q < m; ++q) v += B[lane * m + q] * r[q];
  __syncthreads();
  if (lane < m) r[lane] = v;
  __syncthreads();
  for (int t = lane; t < n; t += 64) {
    const int ct = t / (4 * Z), k = 1 + t / 4 % Z, K0 = k >> 1, K1 = (k + 1) >> 1;
    const double lo = K0 >= 1 ? r[ct * ZC + K0 - 1] : 0.0, hi = K1 <= ZC ? r[ct * ZC + K1 - 1] : 0.0;
    y[t] += 0.5 * (lo + hi) * (t & 1 ? cosx : 1.0) * (t & 2 ? cosy : 1.0);
  }
  __syncthreads();
  smooth(n_post, true);
  if (u >= n) return;
  double* col = M + (static_cast<size_t>(blockIdx.x) * n + u) * n;
  for (int t = lane; t < n; t += 64) col[t] = y[t];
}

size_t build_lds(Dims d, int waves) {
  const size_t Z = d.nz - 1, m = 3 * (d.nz / 2 - 1);
  return (108 * Z + m * m + 24 * Z * waves) * sizeof(double);
}

size_t modes_lds(Dims d) {
  const size_t part = 6ull * (d.nz - 1) * d.nx;
  return (d.nx / 2 + d.ny / 2 + 12ull * (d.nz - 1) + (part > kThreads ? part : kThreads)) * sizeof(double2);
}

size_t back_lds(Dims d) {
  const int cx = d.nx / 2, cy = d.ny / 2;
  return (cx + cy + 4ull * cy * (cx / 2 + 1)) * sizeof(double2);
}

}  // namespace

int bottom_unknowns(Dims d) { return 12 * (d.nz - 1); }

size_t bottom_matrix_values(Dims d) {
  const size_t n = static_cast<size_t>(bottom_unknowns(d));
  return n * n * block_count(d.nx / 2, d.ny / 2);
}

size_t bottom_vector_values(Dims d) {
  return 2ull * bottom_unknowns(d) * mode_count(d.nx / 2, d.ny / 2);
}

// Where the map is used.  The bounds are of space, not of time: the 20 launches it
// stands for cost 60 to 80 us, in which 4 TB/s read some 300 MB, and the map won
// wherever it was tried, V-cycle without and with it 115 -> 55 us at 16^3 over
// 4^3, 124.5 -> 62 at 32^3 over 8^3, 174 -> 93.5 at 36 x 36 x 64 over 9 x 9 x 16
// (45 MB read a cycle, 28 held).  The transforms stage their sums in 64 KB of LDS
// (40 x 40 x 64 over 10 x 10 x 16 does not fit and stays at 184 us); 48 MB read a
// cycle, a block for every mode, bounds what the workspace holds, where reflected
// modes share theirs; and up to 384 unknowns k_bottom_build has a lane for every
// coarse unknown and for every component and plane of a colour.
bool bottom_supported(Dims d) {
  constexpr size_t kMaxBytes = 48ull << 20;
  const size_t n = static_cast<size_t>(bottom_unknowns(d));
  return n <= 384 && n * n * mode_count(d.nx / 2, d.ny / 2) * sizeof(double) <= kMaxBytes &&
         modes_lds(d) <= kMaxLds && back_lds(d) <= kMaxLds;
}

void launch_bottom_build(const double* S, const double* Dinv, const double* Ainv, int ncoarse, Dims d,
                         const double* tw, const int order[8], int n_pre, int n_post, double* M,
                         hipStream_t s) {
  unsigned packed = 0;
  for (int q = 0; q < 8; ++q) packed |= static_cast<unsigned>(order[q]) << (4 * q);
  // four columns per workgroup, fewer where 64 KB do not hold them (the deepest levels)
  int waves = 4;
  while (waves > 1 && build_lds(d, waves) > kMaxLds) --waves;
  const int n = bottom_unknowns(d);
  hipLaunchKernelGGL(k_bottom_build, dim3(block_count(d.nx / 2, d.ny / 2), (n + waves - 1) / waves),
                     dim3(64 * waves), build_lds(d, waves), s, S, Dinv, Ainv, ncoarse, d.nx, d.ny, d.nz,
                     reinterpret_cast<const double2*>(tw), packed, n_pre, n_post, M);
}

template <typename T>
void launch_bottom(const double* M, const double* tw, const T* b, T* x, double* yh, Dims d,
                   hipStream_t s) {
  const int n = bottom_unknowns(d);
  hipLaunchKernelGGL(k_bottom_modes<T>, dim3(mode_count(d.nx / 2, d.ny / 2), (n + kRows - 1) / kRows),
                     dim3(kThreads), modes_lds(d), s, M, b, d.nx, d.ny, d.nz,
                     reinterpret_cast<const double2*>(tw), reinterpret_cast<double2*>(yh));
  hipLaunchKernelGGL(k_bottom_back<T>, dim3(3 * (d.nz - 1)), dim3(256), back_lds(d), s,
                     reinterpret_cast<const double2*>(yh), x, d.nx, d.ny, d.nz,
                     reinterpret_cast<const double2*>(tw));
}

template void launch_bottom<double>(const double*, const double*, const double*, double*, double*,
                                    Dims, hipStream_t);
template void launch_bottom<float>(const double*, const double*, const float*, float*, double*, Dims,
                                   hipStream_t);

}  // namespace qs
