// The two coarsest levels of a V-cycle in two launches (Sec. 3.6, gfx950).
//
// The cycle on the level above the coarsest (smoothing from a zero guess, the
// coarsest solve, the correction and smoothing again) is one fixed linear map
// from that level's right-hand side b to its correction x.  Its colours have
// period 2 in x and y and the coarsest operator is the same at every column,
// so the map commutes with shifts by two columns or rows: Fourier modes over
// the cx * cy shifts (cx, cy the coarsest sizes) split it into independent
// blocks of n = 12 (nz - 1) unknowns (component, plane, y parity, x parity).
// The blocks are computed at setup by running that cycle in FP64 on the n unit
// right-hand sides (bottom_column), for whatever sweeps and colour order the
// handle has, and are held and applied in FP64 in both precisions, as the
// coarsest inverse is.
//
// The map commutes with the reflections in x and y as well, which keep every
// node's colour.  Taken about the nodes' own positions (half a shift for the odd
// columns and rows) and with the z component times i, a block is therefore real,
// and the blocks of (mx, my) and (mx, -my) differ in the y component's sign only:
// 6.5 MB at 8^3 under 16^3 where complex blocks of every mode are 17.6 MB.
//
// What bounds it: the cycle it stands for is 16 colour-pair launches, residual,
// restriction, coarsest solve and correction, each a fixed cost of 3 to 7 us
// and next to no work (8^3 under 16^3: 21 launches, 90 us).  The map costs about
// what the coarsest inverse's product alone did.
#include <hip/hip_runtime.h>

#include "device.h"

namespace qs {

namespace {

constexpr int kThreads = 512;              // of the kernels that transform b
constexpr int kRows = 32;                  // rows of a block per workgroup
constexpr int kGroups = kThreads / kRows;  // column groups per workgroup
constexpr int kBatch = 8;                  // loads in flight per thread in the transform

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

// Unit right-hand side of unknown u at shift 0: b = 0 but for one node.
__global__ __launch_bounds__(256) void k_bottom_unit(double* __restrict__ b, double* __restrict__ x,
                                                     int total, int at) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  b[t] = t == at ? 1.0 : 0.0;
  x[t] = 0.0;
}

// Column u of every block from the response x to unit u.
__global__ __launch_bounds__(kThreads) void k_bottom_column(const double* __restrict__ x, int nx, int ny,
                                                       int nz, const double2* __restrict__ tw, int u,
                                                       double* __restrict__ M) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int cx = nx / 2, cy = ny / 2, n = 12 * (nz - 1);
  double2* ltw = reinterpret_cast<double2*>(smem);
  double2* xh = ltw + cx + cy;
  double2* part = xh + n;
  int mx, my;
  mode_of(blockIdx.x, cx, cy, &mx, &my);
  if (2 * my > cy) return;  // the block of (mx, cy - my) serves
  load_twiddles(tw, cx, cy, ltw);
  forward_mode<double>(x, nx, ny, nz, mx, my, ltw, ltw + cx, part, xh);
  double* col = M + (static_cast<size_t>(block_of(mx, my, cx, cy)) * n + u) * n;
  const double2 w = real_factor(u, nz, mx, my, cx, cy);
  for (int t = threadIdx.x; t < n; t += blockDim.x) col[t] = xh[t].x * w.x + xh[t].y * w.y;
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

// The blocks pay as long as reading them costs less than the launches they
// stand for: 22 launches of about 4 us against kMaxBytes at the 4 to 5 TB/s at
// which the coarsest inverse streams.  The block size also bounds the setup
// (one cycle per unknown).  The transforms stage their sums in LDS (64 KB).
bool bottom_supported(Dims d) {
  constexpr size_t kMaxBytes = 48ull << 20, kMaxLds = 64ull << 10;
  const size_t n = static_cast<size_t>(bottom_unknowns(d));
  return n <= 384 && n * n * mode_count(d.nx / 2, d.ny / 2) * sizeof(double) <= kMaxBytes &&
         modes_lds(d) <= kMaxLds && back_lds(d) <= kMaxLds;
}

void launch_bottom_unit(double* b, double* x, Dims d, int u, hipStream_t s) {
  const int ex = u & 1, ey = (u >> 1) & 1, q = u >> 2, c = q / (d.nz - 1), k = 1 + q % (d.nz - 1);
  const int total = static_cast<int>(d.elems());
  const int at = c * d.comp() + k * d.plane() + ey * d.nx + ex;
  hipLaunchKernelGGL(k_bottom_unit, dim3((total + 255) / 256), dim3(256), 0, s, b, x, total, at);
}

void launch_bottom_column(const double* x, Dims d, const double* tw, int u, double* M, hipStream_t s) {
  hipLaunchKernelGGL(k_bottom_column, dim3(mode_count(d.nx / 2, d.ny / 2)), dim3(kThreads), modes_lds(d), s,
                     x, d.nx, d.ny, d.nz, reinterpret_cast<const double2*>(tw), u, M);
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
