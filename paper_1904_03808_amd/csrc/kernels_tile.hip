// Gauss-Seidel sweep of the fine level by tiles held in LDS, for small and
// medium grids (smoother of Sec. 3.6 on the operator of Sec. 3.4, gfx950).
//
// What bounds such a grid is not bytes but the chain of dependent steps: the
// row sweep (kernels_sweep.hip) marches a few workgroups up the planes, one
// step of loads and barriers after the other, and takes 12 to 20 us per half
// sweep however small the grid is.  Here a workgroup owns a tile of `tr` rows by
// kTP planes (all of x, so the wrap stays inside) and loads, in one round, every
// row and plane its colour phases can reach.  Rows are updated in the order
// first parity, second parity, and within each the planes of the first and then
// of the second parity, so the last values of a whole sweep depend on three more
// rows and up to seven more planes, those of a half sweep (one row parity) on
// one more row and three more planes.  It then runs the phases from LDS, each on
// the part of the tile that the later ones still need, and writes what it owns.
// Values outside are recomputed by several workgroups from the same old values
// in the same order, so the result does not depend on the tiling; the sweep
// reads one buffer and writes another.
//
// Measured, us per sweep, row sweep before -> now: 32^3 36.5 -> 8.2 (FP64),
// 29.3 -> 8.6 (FP32); 64 x 64 x 32 37.1 -> 10.7, 29.8 -> 8.0; 96^3 42.8 -> 34.0,
// 32.1 -> 17.2; 128^3 67.2 -> 61.4, 38.3 -> 31.7.  At 32^3 that is about three
// launches' worth: the fill (two rounds of loads) and eight phases of 42 LDS
// reads per node (18 along the axes, 24 mixed).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.h"

namespace qs {

namespace {

template <typename T>
struct W2;
template <>
struct W2<float> {
  using type = float2;
};
template <>
struct W2<double> {
  using type = double2;
};

constexpr int kTP = 4;           // planes a workgroup owns
constexpr int kTileThreads = 512;
constexpr int kFill = 6;         // row-planes a thread has in flight while the tile is filled
constexpr int kNodes = 2;        // nodes per thread and phase at most
constexpr int kFullStride = 100; // widest rows (LDS stride) of the whole sweep
constexpr int kNone = 1 << 20;   // rounds of a tile that does not fit

struct TileArgs {
  int nx, ny, nz;
  int row_first, plane_first, x_first;  // parities updated first
  int tr;                               // rows a workgroup owns (even)
  int slots;                            // rows of threads: threads / (nx / 2)
  int ntr, ntp;                         // tiles in y and z
};

// Planes a workgroup holds at most: those it owns and what the phases reach.
constexpr int planes_held(int H) { return kTP + (H == 2 ? 7 : 3); }

// [lo, hi) cut to the planes or rows of parity `par`: first one and count.
__device__ __forceinline__ void of_parity(int lo, int hi, int par, int* first, int* n) {
  const int f = lo + ((lo ^ par) & 1);
  *first = f;
  *n = f < hi ? (hi - f + 1) / 2 : 0;
}

// H = 2: a whole sweep, every row from src (nbr is src).  H = 1: the rows of
// parity row_first alone, those from src and the rows between them from nbr;
// only the former are written.
// Z = 0: rows as stored; Z = 1 (H = 1): the rows updated are known to be zero
// and not read; Z = 2: all rows are.
template <typename T, int NXP, int H, int Z>
__global__ __launch_bounds__(kTileThreads) void k_sweep_tile(const T* __restrict__ src,
                                                             const T* __restrict__ nbr,
                                                             T* __restrict__ dst,
                                                             const T* __restrict__ b,
                                                             TileArgs a, FineCoef<T> cf) {
  using V = typename W2<T>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  // [row][kPL][3][NXP]: the even columns of a row, a copy of column 0 after
  // them, then (from kOdd on) the odd columns after a copy of the last one, so
  // that the lanes of a phase, which updates every other column, read
  // consecutive words
  T* tile = reinterpret_cast<T*>(smem);
  constexpr int kOdd = NXP / 2 + 1, kPL = planes_held(H), NU = 2 * H;
  const int nx = a.nx, ny = a.ny, nz = a.nz, W = nx >> 1;
  const int ty = blockIdx.x % a.ntr, tz = blockIdx.x / a.ntr;
  const int j0 = ty * a.tr, k0 = 1 + tz * kTP, k1 = min(k0 + kTP, nz);
  const int pair = threadIdx.x % W, slot = threadIdx.x / W;
  const bool works = slot < a.slots;
  const int c0 = 2 * pair;
  const int P = nx * ny, C = (nz + 1) * P;

  // planes and rows each pair of phases updates, from the last back to the
  // first: what it updates needs the planes and rows next to it
  int kf[NU], kn[NU], jf[H], jn[H];
  int klo = k0, khi = k1, jlo = j0, jhi = j0 + a.tr;
#pragma unroll
  for (int h = H - 1; h >= 0; --h) {
    of_parity(jlo, jhi, h ? 1 - a.row_first : a.row_first, &jf[h], &jn[h]);
#pragma unroll
    for (int q = 1; q >= 0; --q) {
      const int u = 2 * h + q;
      of_parity(max(klo, 1), min(khi, nz), q ? 1 - a.plane_first : a.plane_first, &kf[u], &kn[u]);
      if (kn[u] > 0) {
        klo = min(klo, kf[u] - 1);
        khi = max(khi, kf[u] + 2 * kn[u]);
      }
    }
    jlo = min(jlo, jf[h] - 1);
    jhi = max(jhi, jf[h] + 2 * jn[h]);
  }
  const int np = khi - klo, nr = jhi - jlo;  // np <= kPL

  // fill: thread (pair, slot) takes every slots-th (row, plane), kFill of them
  // with their three components in flight at once
  if (works) {
    const int total = nr * np, dr = a.slots / np, dp = a.slots - dr * np;
    int r = slot / np, p = slot - r * np;
    for (int m0 = slot; m0 < total; m0 += kFill * a.slots) {
      V v[kFill][3];
      int at[kFill];
#pragma unroll
      for (int u = 0; u < kFill; ++u) {
        at[u] = m0 + u * a.slots < total ? (r * kPL + p) * 3 * NXP : -1;
        int j = jlo + min(r, nr - 1);
        j = j < 0 ? j + ny : (j >= ny ? j - ny : j);
        const int k = klo + p, o = __mul24(k, P) + __mul24(j, nx) + c0;
        // rows of the other parity in a half sweep
        const bool between = H == 1 && ((j ^ a.row_first) & 1);
        const T* __restrict__ from = between ? nbr : src;
        const bool zero = Z == 2 || (Z == 1 && !between);
#pragma unroll
        for (int c = 0; c < 3; ++c)
          v[u][c] = zero ? V{T(0), T(0)} : *reinterpret_cast<const V*>(from + c * C + o);
        r += dr;
        p += dp;
        if (p >= np) {
          p -= np;
          ++r;
        }
      }
#pragma unroll
      for (int u = 0; u < kFill; ++u)
        if (at[u] >= 0) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            T* row = tile + at[u] + c * NXP;
            row[pair] = v[u][c].x;
            row[kOdd + pair] = v[u][c].y;
            if (pair == 0) row[W] = v[u][c].x;
            if (pair == W - 1) row[kOdd - 1] = v[u][c].y;
          }
        }
    }
  }

  // The nodes of a pair of phases (both columns of the pair): their place in
  // the tile (-1: none) and b.
  auto fetch = [&](int u, int at[kNodes], V out[kNodes][3]) {
    const int n = jn[u >> 1];
#pragma unroll
    for (int it = 0; it < kNodes; ++it) {
      const int m = slot + it * a.slots;
      at[it] = -1;
      if (!works || m >= n * kn[u]) continue;
      const int q = m / n, r = jf[u >> 1] + 2 * (m - q * n) - jlo, p = kf[u] + 2 * q - klo;
      int j = jlo + r;
      j = j < 0 ? j + ny : (j >= ny ? j - ny : j);
      at[it] = (r * kPL + p) * 3 * NXP;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        out[it][c] = *reinterpret_cast<const V*>(b + c * C + (klo + p) * P + j * nx + c0);
    }
  };
  V bn[kNodes][3];
  int an[kNodes];
  fetch(0, an, bn);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    V bc[kNodes][3];
    int at[kNodes];
#pragma unroll
    for (int it = 0; it < kNodes; ++it) {
      at[it] = an[it];
#pragma unroll
      for (int c = 0; c < 3; ++c) bc[it][c] = bn[it][c];
    }
    if (u < NU - 1) fetch(u + 1, an, bn);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      // column 2 pair + xp: its own place, the column left of it (x[side]) and
      // right of it (x[side + 1]) among those of the other parity, and the copy
      // to keep where it is the first or the last column
      const int xp = e ? 1 - a.x_first : a.x_first;
      const int mine = xp ? kOdd + pair : pair, side = xp ? pair : kOdd - 1 + pair;
      const int copy = xp ? (pair == W - 1 ? kOdd - 1 : mine) : (pair == 0 ? W : mine);
#pragma unroll
      for (int it = 0; it < kNodes; ++it) {
        if (at[it] < 0) continue;
        T* own = tile + at[it];
#define X(c, dz, dy, dx) \
  own[((dy) * kPL * 3 + (dz) * 3 + (c)) * NXP + ((dx) == 0 ? mine : ((dx) < 0 ? side : side + 1))]
        const T fx0 = X(0, 0, 0, 1) + X(0, 0, 0, -1), fy0 = X(0, 0, 1, 0) + X(0, 0, -1, 0),
                fz0 = X(0, 1, 0, 0) + X(0, -1, 0, 0);
        const T fx1 = X(1, 0, 0, 1) + X(1, 0, 0, -1), fy1 = X(1, 0, 1, 0) + X(1, 0, -1, 0),
                fz1 = X(1, 1, 0, 0) + X(1, -1, 0, 0);
        const T fx2 = X(2, 0, 0, 1) + X(2, 0, 0, -1), fy2 = X(2, 0, 1, 0) + X(2, 0, -1, 0),
                fz2 = X(2, 1, 0, 0) + X(2, -1, 0, 0);
        // mixed differences f(+,+) - f(+,-) - f(-,+) + f(-,-)
        const T mxy0 = X(0, 0, 1, 1) - X(0, 0, -1, 1) - X(0, 0, 1, -1) + X(0, 0, -1, -1);
        const T mxy1 = X(1, 0, 1, 1) - X(1, 0, -1, 1) - X(1, 0, 1, -1) + X(1, 0, -1, -1);
        const T mxz0 = X(0, 1, 0, 1) - X(0, -1, 0, 1) - X(0, 1, 0, -1) + X(0, -1, 0, -1);
        const T mxz2 = X(2, 1, 0, 1) - X(2, -1, 0, 1) - X(2, 1, 0, -1) + X(2, -1, 0, -1);
        const T myz1 = X(1, 1, 1, 0) - X(1, -1, 1, 0) - X(1, 1, -1, 0) + X(1, -1, -1, 0);
        const T myz2 = X(2, 1, 1, 0) - X(2, -1, 1, 0) - X(2, 1, -1, 0) + X(2, -1, -1, 0);
#undef X
        const T b0 = xp ? bc[it][0].y : bc[it][0].x, b1 = xp ? bc[it][1].y : bc[it][1].x,
                b2 = xp ? bc[it][2].y : bc[it][2].x;
        const T o0 = (cf.h2 * b0 + cf.p * fx0 + cf.q * (fy0 + fz0) + cf.m4 * (mxy1 + mxz2)) * cf.inv_diag;
        const T o1 = (cf.h2 * b1 + cf.p * fy1 + cf.q * (fx1 + fz1) + cf.m4 * (mxy0 + myz2)) * cf.inv_diag;
        const T o2 = (cf.h2 * b2 + cf.p * fz2 + cf.q * (fx2 + fy2) + cf.m4 * (mxz0 + myz1)) * cf.inv_diag;
        own[mine] = o0;
        own[copy] = o0;
        own[NXP + mine] = o1;
        own[NXP + copy] = o1;
        own[2 * NXP + mine] = o2;
        own[2 * NXP + copy] = o2;
      }
      __syncthreads();
    }
  }
  if (!works) return;
  const int rows = min(a.tr, ny - j0);
  for (int m = slot; m < rows * kTP; m += a.slots) {
    const int r = m / kTP, k = k0 + m % kTP;
    if (k >= k1 || (H == 1 && ((r ^ a.row_first) & 1))) continue;
    const T* row = tile + ((j0 - jlo + r) * kPL + k - klo) * 3 * NXP;
    const int o = k * P + (j0 + r) * nx + c0;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      *reinterpret_cast<V*>(dst + c * C + o) = V{row[c * NXP + pair], row[c * NXP + kOdd + pair]};
  }
}

// Row strides (columns plus four) the kernel is built for.
int tile_stride(int nx) {
  for (const int s : {36, 52, 68, 84, 100, 132, 164})
    if (nx + 4 <= s) return s;
  return 0;
}

// Row-planes of the widest phase: the rows of one parity (one more than half
// the tile's where a second half of the rows follows), by half the planes of
// the tile and one (three) more.
int phase_rows(int tr, int H) { return H == 2 ? (tr / 2 + 1) * (kTP / 2 + 3) : tr / 2 * (kTP / 2 + 1); }

size_t tile_lds(int nx, int tr, int H, int bytes) {
  return static_cast<size_t>(tr + (H == 2 ? 3 : 1)) * planes_held(H) * 3 * tile_stride(nx) * bytes;
}

#define QS_STRIDES(X) X(36) X(52) X(68) X(84) X(100) X(132) X(164)

// The kernels there are: whole sweeps up to kFullStride, zero starts in FP32 (the
// corrections of the refinement) alone.
template <typename T>
constexpr bool has_tile(int stride, int H, int Z) {
  return (H == 1 || stride <= kFullStride) && (Z == 0 || sizeof(T) == 4);
}

template <typename T, int NXP>
void launch_stride(const T* src, const T* nbr, T* dst, const T* b, const TileArgs& a,
                   const FineCoef<T>& cf, int H, int Z, int threads, size_t lds, hipStream_t s) {
  const dim3 grid(a.ntr * a.ntp), block(threads);
#define QS_TILE(H_, Z_)                                                                             \
  if constexpr (has_tile<T>(NXP, H_, Z_))                                                           \
    if (H == H_ && Z == Z_)                                                                         \
      hipLaunchKernelGGL((k_sweep_tile<T, NXP, H_, Z_>), grid, block, lds, s, src, nbr, dst, b, a, cf)
  QS_TILE(2, 0);
  QS_TILE(2, 2);
  QS_TILE(1, 0);
  QS_TILE(1, 1);
  QS_TILE(1, 2);
#undef QS_TILE
}

template <typename T, int NXP, int H, int Z>
void tile_limit_one(int bytes) {
  if constexpr (has_tile<T>(NXP, H, Z))
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sweep_tile<T, NXP, H, Z>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <typename T, int NXP>
void tile_limit(int bytes) {
  tile_limit_one<T, NXP, 2, 0>(bytes);
  tile_limit_one<T, NXP, 2, 2>(bytes);
  tile_limit_one<T, NXP, 1, 0>(bytes);
  tile_limit_one<T, NXP, 1, 1>(bytes);
  tile_limit_one<T, NXP, 1, 2>(bytes);
}

// Rounds of resident workgroups of a launch with tr rows per tile.
int tile_rounds(Dims d, int tr, int H, size_t lds_limit, int bytes) {
  const size_t lds = tile_lds(d.nx, tr, H, bytes);
  if (lds > lds_limit || kNodes * (kTileThreads / (d.nx / 2)) < phase_rows(tr, H)) return kNone;
  const int per_cu = std::max<int>(1, std::min<size_t>(lds_limit / lds, 2048 / kTileThreads));
  const long long wgs = 1LL * ((d.ny + tr - 1) / tr) * ((d.nz - 1 + kTP - 1) / kTP);
  return static_cast<int>((wgs + 256 * per_cu - 1) / (256 * per_cu));
}

}  // namespace

void tile_set_lds_limit(size_t bytes) {
#define QS_LIMIT(N)                          \
  tile_limit<double, N>(static_cast<int>(bytes)); \
  tile_limit<float, N>(static_cast<int>(bytes));
  QS_STRIDES(QS_LIMIT)
#undef QS_LIMIT
}

// Which sweep a fine level takes.  The tile re-reads its halo (1.7 to 2.5 times
// the level's x per half sweep against 1.5 of the row sweep) but has no march:
// it wins as long as x, dst and b stay in the 256 MB Infinity Cache, where that
// costs little.  Per V-cycle, tile against row sweep: FP64 128^3 (151 MB) 491
// against 516 us, 96 x 192 x 192 (255 MB) 877 against 885, 160^3 (295 MB) 983
// against 945; FP32 128^3 334 against 375 us, 160^3 (147 MB) 646 against 680,
// 160 x 256 x 256 (377 MB) 1158 against 1154.  One launch for both halves where
// it is one round of resident workgroups (sweep of 64 x 64 x 32, FP32: 8.0 us
// against 10.4 in halves and 17.4 by rows; 96 x 96 x 24, FP64, two rounds: 20.6
// against 15.2 in halves).  Rows per tile: the fewest rounds, then two rows for
// the whole sweep (its fill is shorter) and four for a half (less halo).
int sweep_tile_rows(Dims d, size_t lds_limit, int bytes, int* halves) {
  if (d.nx % 2 || d.ny % 2 || d.nx < 4 || d.ny < 4 || d.nz < 2 || !tile_stride(d.nx)) return 0;
  if (3 * d.elems() * bytes > (256ull << 20)) return 0;
  if (tile_stride(d.nx) <= kFullStride) {
    *halves = 2;
    if (tile_rounds(d, 2, 2, lds_limit, bytes) == 1) return 2;
    if (tile_rounds(d, 4, 2, lds_limit, bytes) == 1) return 4;
  }
  *halves = 1;
  const int two = tile_rounds(d, 2, 1, lds_limit, bytes), four = tile_rounds(d, 4, 1, lds_limit, bytes);
  if (std::min(two, four) == kNone) return 0;
  return two < four ? 2 : 4;
}

template <typename T>
void launch_sweep_tile(const T* src, const T* nbr, T* dst, const T* b, Dims d, int tr,
                       int halves, int row_first, bool reverse, int zero, const FineCoef<T>& cf,
                       hipStream_t s) {
  TileArgs a;
  a.nx = d.nx;
  a.ny = d.ny;
  a.nz = d.nz;
  a.row_first = row_first;
  a.plane_first = a.x_first = reverse ? 1 : 0;
  a.tr = tr;
  a.ntr = (d.ny + tr - 1) / tr;
  a.ntp = (d.nz - 1 + kTP - 1) / kTP;
  const int W = d.nx / 2;
  a.slots = std::min(phase_rows(tr, halves), kTileThreads / W);
  const int threads = (a.slots * W + 63) / 64 * 64;
  const size_t lds = tile_lds(d.nx, tr, halves, sizeof(T));
  switch (tile_stride(d.nx)) {
#define QS_LAUNCH(N)                                                                      \
  case N:                                                                                 \
    launch_stride<T, N>(src, nbr, dst, b, a, cf, halves, zero, threads, lds, s); \
    break;
    QS_STRIDES(QS_LAUNCH)
#undef QS_LAUNCH
  }
}

template void launch_sweep_tile<double>(const double*, const double*, double*, const double*, Dims, int,
                                        int, int, bool, int, const FineCoef<double>&, hipStream_t);
template void launch_sweep_tile<float>(const float*, const float*, float*, const float*, Dims, int, int,
                                       int, bool, int, const FineCoef<float>&, hipStream_t);

}  // namespace qs
