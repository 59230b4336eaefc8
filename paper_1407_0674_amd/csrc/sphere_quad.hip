// Surface integrals over spheres by product quadrature (Sec. 3.5), as an
// alternative to the spectral delta-shell weights of the main evaluation.
//
// For a field f on the grid and a radius R, Sec. 3.5 writes
//   I(r)   = int f(r') delta(|r' - r| - R) dr'
//          = R^2 int_0^{2 pi} int_0^{pi} f(r + R n(theta, phi)) sin(phi) dphi dtheta
// and approximates the double integral by a k-by-k product rule in (theta,
// phi).  The 1D rules and the interpolation between grid points are not
// fixed by the paper; here theta_i = 2 pi i / k with weights 2 pi / k (the
// trapezoidal rule of a periodic integrand), phi_j the k Gauss-Legendre
// points of [0, pi], and f(r + R n) the trilinear interpolant of the grid
// values.  The vector integral R^2 int f(r + R n) n dOmega (the FMT n_2v of
// one species) uses the same nodes.
//
// On a uniform grid every node sits at the same displacement R n_ij / h from
// every output point, so its eight trilinear corners are the same integer
// offsets everywhere: the whole rule collapses into one fixed stencil of
// integer offsets with four weights each (scalar, x, y, z), merged on the
// host in double.  The kernel is then a 3D stencil: a workgroup stages a
// tile of f with a halo of the stencil reach in LDS and every thread sums
// the stencil for TX outputs along x.
//
// It is bound by the vector ALU (three fields at 192^3 move 850 MB, 130 us at
// 6.6 TB/s).  The rule's symmetry in y and z lets a thread fold the four mirror
// columns of a (|dy|, |dz|) into three sums once per tile plane, and all the
// offsets along x of those columns share them; a rule of even order is symmetric in
// x too, so the eight offsets (+-dx, +-dy, +-dz) then take four multiply-adds, four
// to six additions and a share of the folding, against 24 operations and eight LDS
// reads when each offset was paired with its antipode alone.  192^3, order 8, mixed,
// R = 1.4, 2.6 and 3.9 h: 102, 164 and 232 us with pairs, 65, 91 and 123 with columns
// (FP64 120, 237 and 418; 72, 123 and 218).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <vector>

namespace pnp {

constexpr int kQuadTY = 8;       // outputs per workgroup along y
constexpr int kQuadTZ = 32;      // outputs per workgroup along z (the fastest axis)
constexpr int kQuadCols = kQuadTY * kQuadTZ;  // output columns per workgroup
constexpr int kQuadMaxFields = 64;
constexpr size_t kQuadMaxLds = 163840;   // the most LDS one workgroup can hold on gfx950

// A column of the merged stencil: the offsets (dx, +-dy, +-dz) of one (|dy|, |dz|)
// over all dx.  The rule is even in y and in z (theta and 2 pi - theta, phi and
// pi - phi are nodes together), so the four mirror images share their weights up
// to sign: with a, b, c, d the values at (+dy, +dz), (+dy, -dz), (-dy, +dz),
// (-dy, -dz), the scalar and x weights multiply ss = a + b + c + d, the y weight
// ds = a + b - c - d and the z weight sd = a - b + c - d.
struct QuadColumn {
  int32_t near_lds, far_lds;  // tile positions of (dy, dz) and (dy, -dz) relative to the output's
  uint32_t dx;                // bit k: a weight at dx = k (even orders: at +-k); bit 16 + k: at dx = -k (odd ones)
  int32_t w;                  // first weight, in units of four, of the bits set in the order 0, 1, -1, 2, -2, ..
};

// Kinds of columns: bit 0 dy = 0 (two images, ds = 0), bit 1 dz = 0 (sd = 0).
constexpr int kQuadKinds = 4;

struct QuadArgs {
  const double* f;        // [F][N]
  double* out;            // [F][4][N]
  const int32_t* begin;   // [4F + 1]: field f's columns of kind k are [begin[4f+k], begin[4f+k+1]);
                          // then the reach of each field [F]
  const QuadColumn* columns;
  const void* weights;    // four T each: scalar, x, y, z
  int32_t nx, ny, nz;
  int32_t H;              // stencil reach (max |offset| over all fields and axes); selects
                          // the kernel, whose tile extents follow from it
  int32_t tiles_y, tiles_z;
  int32_t aperiodic;
  int32_t even;           // the rule is of even order
};

__device__ __forceinline__ int quad_wrap(int i, int n) {
  int r = i % n;
  return r < 0 ? r + n : r;
}

// Tile height along x for a stencil reach H: 8 or 4 outputs if two workgroups
// then share a compute unit's 160 KB, else the most that fits one workgroup
// (fewer than four outputs a column share its folding too thinly: FP64 reach 5,
// order 8, two groups of two outputs 415 us, one group of eight 282); 0 if
// nothing fits.
constexpr size_t quad_tile_bytes(int tx, int H, size_t elem) {
  return (size_t)(tx + 2 * H) * (kQuadTY + 2 * H) * (kQuadTZ + 2 * H) * elem;
}
constexpr size_t quad_table_bytes(int tx, int H) { return (size_t)(tx + kQuadTY + kQuadTZ + 6 * H) * sizeof(int32_t); }
constexpr int quad_tx(int H, size_t elem) {
  for (int tx = 8; tx >= 4; tx /= 2)
    if (quad_tile_bytes(tx, H, elem) + quad_table_bytes(tx, H) <= kQuadMaxLds / 2) return tx;
  for (int tx = 8; tx >= 1; tx /= 2)
    if (quad_tile_bytes(tx, H, elem) + quad_table_bytes(tx, H) <= kQuadMaxLds) return tx;
  return 0;
}
// A tile that has the compute unit to itself is taken by two threads per
// column of outputs, so that two wavefronts a SIMD cover each other's LDS reads
// (FP32 reach 9: 1206 us with one, 831 with two, 1376 with four).
constexpr int quad_split(int H, size_t elem) {
  const int tx = quad_tx(H, elem);
  if (quad_tile_bytes(tx, H, elem) + quad_table_bytes(tx, H) <= kQuadMaxLds / 2) return 1;
  return tx < 2 ? 1 : 2;
}

// The rounding error of s = a + b (exact where |a| >= |b|, else to the rounding of
// s - a); finite where s is not, so that an infinite value stays one.
__device__ __forceinline__ float sum_error(float a, float b, float s) {
  return __builtin_amdgcn_fmed3f(b - (s - a), -__FLT_MAX__, __FLT_MAX__);
}

// Sum the columns [c0, c1) of one kind into a thread's TX outputs.  A column's
// values are read and folded once per tile plane, at most TX + 2H of them, and
// serve all its dx: level k reads the two planes that dx = +-k adds.
// EVEN: a rule of even order, which is even in x too: +-k share their weights, the
// x weight up to sign and times the difference of the two values.  Rules of odd
// order have no such symmetry: a point that only the mirror offset touches has no
// part in the sum, not even times zero (it may be infinite or NaN).
//
// Rounding: the vector integrals are small differences of large sums.  The odd
// combinations ds and sd are formed from differences of single values, exact for
// like ones, and FP32 keeps the rounding error es of each ss for the x integral.
// Error against the same rule with its antipodal offsets in pairs, whose
// differences are of single values throughout (geometric mean over radii of 0.8 to
// 5 h and orders 4 to 20; scalar, x, y, z): FP32 0.76, 0.83, 0.81, 0.86, FP64 0.90,
// 0.69, 0.81, 0.87.  Without es the FP32 x integral is at 1.14 (192^3, R = 3.9 h
// 123 us with, 114 without), with each x offset times its own weight at 1.31, FP64
// at 1.99 and up to 10.
template <typename T, int H, int TX, int KIND, bool EVEN>
__device__ __forceinline__ void quad_columns(const QuadColumn* columns, int c0, int c1, const T* weights, const T* col,
                                             T (&acc)[TX][4]) {
  constexpr int PLANE = (kQuadTY + 2 * H) * (kQuadTZ + 2 * H);
  constexpr bool Y = !(KIND & 1), Z = !(KIND & 2);
  constexpr bool ERR = EVEN && sizeof(T) == 4 && (Y || Z);
#pragma unroll 1
  for (int e = c0; e < c1; ++e) {
    const QuadColumn q = columns[e];
    const T* w = weights + 4 * (size_t)q.w;
    const uint32_t levels = (q.dx | q.dx >> 16) & 0xffffu;
    T ss[TX + 2 * H], ds[TX + 2 * H], sd[TX + 2 * H], es[TX + 2 * H];
    auto read = [&](int i) {  // plane i - H relative to the first output's
      const T* p = col + (i - H) * PLANE;
      if constexpr (Y && Z) {
        const T va = p[q.near_lds], vb = p[q.far_lds], vc = p[-q.far_lds], vd = p[-q.near_lds];
        // differences before sums: those of like values are exact
        const T ad = va - vd, bc = vb - vc;
        const T p1 = va + vd, p2 = vb + vc;
        ss[i] = p1 + p2;
        if constexpr (ERR) es[i] = sum_error(p1, p2, ss[i]);
        ds[i] = ad + bc;
        sd[i] = ad - bc;
      } else if constexpr (Y) {
        const T va = p[q.near_lds], vd = p[-q.near_lds];
        ss[i] = va + vd;
        if constexpr (ERR) es[i] = sum_error(va, vd, ss[i]);
        ds[i] = va - vd;
      } else if constexpr (Z) {
        const T va = p[q.near_lds], vd = p[-q.near_lds];
        ss[i] = va + vd;
        if constexpr (ERR) es[i] = sum_error(va, vd, ss[i]);
        sd[i] = va - vd;
      } else {
        ss[i] = p[0];
      }
    };
    auto add = [&](int dx, const T* c) {
#pragma unroll
      for (int x = 0; x < TX; ++x) {
        acc[x][0] += c[0] * ss[x + H + dx];
        acc[x][1] += c[1] * ss[x + H + dx];
        if constexpr (Y) acc[x][2] += c[2] * ds[x + H + dx];
        if constexpr (Z) acc[x][3] += c[3] * sd[x + H + dx];
      }
    };
#pragma unroll
    for (int i = H; i < H + TX; ++i) read(i);
    if (q.dx & 1) {
      if constexpr (EVEN) {
#pragma unroll
        for (int x = 0; x < TX; ++x) {
          acc[x][0] += w[0] * ss[x + H];
          if constexpr (Y) acc[x][2] += w[2] * ds[x + H];
          if constexpr (Z) acc[x][3] += w[3] * sd[x + H];
        }
      } else {
        add(0, w);
      }
      w += 4;
    }
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      if ((levels >> k) == 0) break;
      read(H - k);
      read(H + TX - 1 + k);
      if constexpr (EVEN) {
        if (q.dx >> k & 1) {
#pragma unroll
          for (int x = 0; x < TX; ++x) {
            const int u = x + H + k, d = x + H - k;
            acc[x][0] += w[0] * (ss[u] + ss[d]);
            if constexpr (ERR) acc[x][1] += w[1] * ((ss[u] - ss[d]) + (es[u] - es[d]));
            else acc[x][1] += w[1] * (ss[u] - ss[d]);
            if constexpr (Y) acc[x][2] += w[2] * (ds[u] + ds[d]);
            if constexpr (Z) acc[x][3] += w[3] * (sd[u] + sd[d]);
          }
          w += 4;
        }
      } else {
        if (q.dx >> k & 1) {
          add(k, w);
          w += 4;
        }
        if (q.dx >> (16 + k) & 1) {
          add(-k, w);
          w += 4;
        }
      }
    }
  }
}

// H (the stencil reach) is a template parameter so that the tile pitches are
// constants: the TX reads of one stencil offset then share one address and
// differ by immediate offsets.
template <typename T, int H, bool EVEN>
__global__ __launch_bounds__((kQuadCols * quad_split(H, sizeof(T)))) void k_sphere_quad(QuadArgs a) {
  constexpr int HX = quad_tx(H, sizeof(T)), TX = HX / quad_split(H, sizeof(T));  // outputs per tile, per thread
  constexpr int LY = kQuadTY + 2 * H, LZ = kQuadTZ + 2 * H, LX = HX + 2 * H;
  constexpr int kThreads = kQuadCols * quad_split(H, sizeof(T));
  constexpr int PLANE = LY * LZ;
  const int F = (int)gridDim.y;
  __shared__ T tile[LX * PLANE];
  __shared__ int32_t at[LX + LY + LZ];
  static_assert(LX + LY + LZ <= kThreads, "one thread per table entry");
  const int field = blockIdx.y;
  // neighbouring tiles on one XCD (workgroups go round the eight in turn), so
  // that they find each other's halos in its L2
  const int per = (int)gridDim.x / 8, rest = (int)gridDim.x % 8;
  const int xcd = (int)blockIdx.x % 8, nth = (int)blockIdx.x / 8;
  int t = xcd * per + (xcd < rest ? xcd : rest) + nth;
  const int tz = t % a.tiles_z;
  t /= a.tiles_z;
  const int ty = t % a.tiles_y;
  const int tx = t / a.tiles_y;
  const int x0 = tx * HX, y0 = ty * kQuadTY, z0 = tz * kQuadTZ;
  const size_t N = (size_t)a.nx * a.ny * a.nz;
  const double* src = a.f + (size_t)field * N;

  // Tile element (i, j, l) holds f at grid point (x0 - H + i, y0 - H + j,
  // z0 - H + l): its periodic image, or zero outside the grid in the aperiodic
  // mode.  The image is found once per plane, row and column of the tile (three
  // remainders an element were most of the staging), -1 for none; a field of
  // smaller reach than the launch's leaves out what its stencil does not touch.
  const int reach = a.begin[kQuadKinds * F + 1 + field];
  if (threadIdx.x < LX + LY + LZ) {
    const int q = threadIdx.x;
    const int axis = q < LX ? 0 : q < LX + LY ? 1 : 2;
    const int i = axis == 0 ? q : axis == 1 ? q - LX : q - LX - LY;
    const int n = axis == 0 ? a.nx : axis == 1 ? a.ny : a.nz;
    const int g = (axis == 0 ? x0 : axis == 1 ? y0 : z0) - H + i;
    const int len = axis == 0 ? LX : axis == 1 ? LY : LZ;
    const bool used = i >= H - reach && i < len - H + reach;
    int v = a.aperiodic ? (g >= 0 && g < n ? g : -1) : quad_wrap(g, n);
    if (!used) v = -1;
    // grid extents multiply to less than 2^31 points
    at[q] = v < 0 ? -1 : axis == 0 ? v * a.ny * a.nz : axis == 1 ? v * a.nz : v;
  }
  __syncthreads();
#pragma unroll 8
  for (int e = threadIdx.x; e < LX * PLANE; e += kThreads) {
    const int i = e / PLANE;
    const int rem = e - i * PLANE;
    const int j = rem / LZ;
    const int l = rem - j * LZ;
    const int ox = at[i], oy = at[LX + j], oz = at[LX + LY + l];
    const bool in = (ox | oy | oz) >= 0;
    const double v = src[(uint32_t)(in ? ox + oy + oz : 0)];
    tile[e] = in ? (T)v : T(0);
  }
  __syncthreads();

  const int yl = threadIdx.x / kQuadTZ % kQuadTY, zl = threadIdx.x % kQuadTZ;
  const int xl = threadIdx.x / kQuadCols * TX;  // the thread's first output along x
  const T* col = tile + ((H + xl) * LY + (H + yl)) * LZ + (H + zl);
  T acc[TX][4];
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[x][c] = T(0);

  const int32_t* begin = a.begin + kQuadKinds * field;
  const T* w = static_cast<const T*>(a.weights);
  quad_columns<T, H, TX, 0, EVEN>(a.columns, begin[0], begin[1], w, col, acc);
  quad_columns<T, H, TX, 1, EVEN>(a.columns, begin[1], begin[2], w, col, acc);
  quad_columns<T, H, TX, 2, EVEN>(a.columns, begin[2], begin[3], w, col, acc);
  quad_columns<T, H, TX, 3, EVEN>(a.columns, begin[3], begin[4], w, col, acc);

  const int gy = y0 + yl, gz = z0 + zl;
  if (gy >= a.ny || gz >= a.nz) return;
  double* dst = a.out + (size_t)field * 4 * N;
#pragma unroll
  for (int x = 0; x < TX; ++x) {
    const int gx = x0 + xl + x;
    if (gx < a.nx) {
      const size_t idx = ((size_t)gx * a.ny + gy) * a.nz + gz;
#pragma unroll
      for (int c = 0; c < 4; ++c) dst[(size_t)c * N + idx] = (double)acc[x][c];
    }
  }
}

// ---------------------------------------------------------------------------
// Host side: the rule, the merged stencil and the launch.

// Gauss-Legendre points and weights on [-1, 1]: Newton's method on P_k
// (three-term recurrence) from the usual cosine first guesses.
inline void gauss_legendre(int k, std::vector<double>& x, std::vector<double>& w) {
  x.assign(k, 0.0);
  w.assign(k, 0.0);
  // P_k(z) and P_{k-1}(z) by (m + 1) P_{m+1} = (2m + 1) z P_m - m P_{m-1}
  auto legendre = [k](double z, double& pk, double& pkm1) {
    double p0 = 1.0, p1 = z;
    for (int m = 1; m < k; ++m) {
      const double p2 = ((2.0 * m + 1.0) * z * p1 - m * p0) / (m + 1.0);
      p0 = p1;
      p1 = p2;
    }
    pk = p1;
    pkm1 = p0;
  };
  for (int j = 0; j < k; ++j) {
    double z = std::cos(M_PI * (j + 0.75) / (k + 0.5));
    double pk, pkm1;
    for (int it = 0; it < 100; ++it) {
      legendre(z, pk, pkm1);
      const double dp = k * (z * pk - pkm1) / (z * z - 1.0);  // P_k'(z)
      const double dz = pk / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    legendre(z, pk, pkm1);
    const double dp = k * (z * pk - pkm1) / (z * z - 1.0);
    x[j] = z;
    w[j] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

struct QuadStencil {
  struct Column {
    int dy, dz;             // >= 0
    std::vector<double> c;  // [..][4], the order of QuadColumn::w
    uint32_t up = 0, down = 0;  // bit k: a weight at dx = k, at -k (k > 0)
  };
  std::vector<Column> columns[kQuadKinds];
  int reach = 0;          // max |offset|
  int span = 0;           // the same over every cell that a node touches, if only by rounding
};

// Interpolation points along one axis at fraction t of a cell (the node at
// base + t): trilinear, offsets 0 and 1 with 1 - t and t; tricubic, offsets
// -1, 0, 1, 2 with the Lagrange cubics through those points at t.  Returns
// the count; off[] and w[] receive the offsets and weights.
inline int interp_axis(double t, bool cubic, int* off, double* w) {
  if (!cubic) {
    off[0] = 0; w[0] = 1.0 - t;
    off[1] = 1; w[1] = t;
    return 2;
  }
  off[0] = -1; w[0] = -t * (t - 1.0) * (t - 2.0) / 6.0;
  off[1] = 0;  w[1] = (t + 1.0) * (t - 1.0) * (t - 2.0) / 2.0;
  off[2] = 1;  w[2] = -(t + 1.0) * t * (t - 2.0) / 2.0;
  off[3] = 2;  w[3] = (t + 1.0) * t * (t - 1.0) / 6.0;
  return 4;
}

// The k-by-k rule of one sphere of radius r (grid units) and physical radius
// R, merged over the interpolation points of every node (8 trilinear
// corners, or 64 tricubic points) into integer offsets.
inline QuadStencil build_quad_stencil(double r, double R, int k, bool cubic) {
  std::vector<double> gx, gw;
  gauss_legendre(k, gx, gw);
  const bool even = k % 2 == 0;
  const int Hc = (int)std::floor(r) + (cubic ? 2 : 1);
  const int side = 2 * Hc + 1;
  std::vector<double> acc((size_t)side * side * side * 4, 0.0);
  std::vector<char> hit((size_t)side * side * side, 0);
  for (int i = 0; i < k; ++i) {
    const double th = 2.0 * M_PI * i / k, wth = 2.0 * M_PI / k;
    for (int j = 0; j < k; ++j) {
      const double ph = 0.5 * M_PI * (gx[j] + 1.0), wph = 0.5 * M_PI * gw[j];
      const double n[3] = {std::cos(th) * std::sin(ph), std::sin(th) * std::sin(ph), std::cos(ph)};
      const double W = R * R * std::sin(ph) * wth * wph;
      int b[3], off[3][4], cnt[3];
      double wa[3][4];
      for (int a = 0; a < 3; ++a) {
        const double p = r * n[a];
        b[a] = (int)std::floor(p);
        cnt[a] = interp_axis(p - b[a], cubic, off[a], wa[a]);
      }
      for (int cx = 0; cx < cnt[0]; ++cx)
        for (int cy = 0; cy < cnt[1]; ++cy)
          for (int cz = 0; cz < cnt[2]; ++cz) {
            const double tw = wa[0][cx] * wa[1][cy] * wa[2][cz];
            if (tw == 0.0) continue;
            const int ox = b[0] + off[0][cx] + Hc, oy = b[1] + off[1][cy] + Hc, oz = b[2] + off[2][cz] + Hc;
            const size_t cell = ((size_t)ox * side + oy) * side + oz;
            hit[cell] = 1;
            acc[cell * 4 + 0] += W * tw;
            for (int a = 0; a < 3; ++a) acc[cell * 4 + 1 + a] += W * tw * n[a];
          }
    }
  }
  const size_t cells = (size_t)side * side * side;
  double cmax = 0.0;
  for (size_t cell = 0; cell < cells; ++cell)
    if (hit[cell])
      for (int q = 0; q < 4; ++q) cmax = std::max(cmax, std::fabs(acc[cell * 4 + q]));
  const double tol = 1e-14 * cmax;
  // A node on a grid plane up to rounding (every rule has some: cos(pi / 2) is
  // 6e-17) also touches the cell beyond with weights of the rounding's size.
  // Cells with no weight above the same 1e-14 are left out: at order
  // 8 and R = 1.5, 3 and 4 h, 106 -> 100, 218 -> 188 and 248 -> 212 offsets.
  QuadStencil s;
  for (size_t cell = 0; cell < cells; ++cell) {
    if (!hit[cell]) continue;
    const int ox = (int)(cell / ((size_t)side * side)), oy = (int)(cell / side % side), oz = (int)(cell % side);
    s.span = std::max(s.span, std::max(std::abs(ox - Hc), std::max(std::abs(oy - Hc), std::abs(oz - Hc))));
  }
  // The merged weights are even in y and z, and for even orders in x (odd for that
  // axis' vector weight), in exact arithmetic; the node coordinates differ in the
  // last bits, and the mean over the images is taken.
  for (int dy = 0; dy <= Hc; ++dy)
    for (int dz = 0; dz <= Hc; ++dz) {
      QuadStencil::Column col;
      col.dy = dy;
      col.dz = dz;
      int hx = -1;
      // the mean weights at dx; false if none is above tol
      auto weights = [&](int dx, double* m) {
        for (int q = 0; q < 4; ++q) m[q] = 0.0;
        const int nx = even ? 2 : 1;
        const double part = 0.25 / nx;
        for (int ix = 0; ix < nx; ++ix)
          for (int iy = 0; iy < 2; ++iy)
            for (int iz = 0; iz < 2; ++iz) {
              const int ox = Hc + (ix ? -dx : dx), oy = Hc + (iy ? -dy : dy), oz = Hc + (iz ? -dz : dz);
              const double* v = &acc[(((size_t)ox * side + oy) * side + oz) * 4];
              m[0] += part * v[0];
              m[1] += (ix ? -part : part) * v[1];
              m[2] += (iy ? -part : part) * v[2];
              m[3] += (iz ? -part : part) * v[3];
            }
        double big = 0.0;
        for (int q = 0; q < 4; ++q) big = std::max(big, std::fabs(m[q]));
        return big > tol;
      };
      for (int k = 0; k <= Hc; ++k) {
        double m[4];
        if (weights(k, m)) {
          col.c.insert(col.c.end(), m, m + 4);
          col.up |= 1u << k;
          hx = k;
        }
        if (!even && k > 0 && weights(-k, m)) {
          col.c.insert(col.c.end(), m, m + 4);
          col.down |= 1u << k;
          hx = k;
        }
      }
      if (hx < 0) continue;
      s.reach = std::max(s.reach, std::max(hx, std::max(dy, dz)));
      s.columns[(dy == 0 ? 1 : 0) + (dz == 0 ? 2 : 0)].push_back(std::move(col));
    }
  return s;
}

// The packed upload, each part padded to 16 bytes: begin[4F + 1] and the
// reaches [F], the columns of each field by kind, the weights.
struct QuadPack {
  std::vector<unsigned char> bytes;
  size_t columns_at, weights_at;
};

template <typename T>
inline QuadPack pack_quad(const std::vector<QuadStencil>& st, int lz) {
  const int F = (int)st.size();
  size_t columns = 0, weights = 0;
  for (const auto& s : st)
    for (const auto& kind : s.columns)
      for (const auto& q : kind) {
        ++columns;
        weights += q.c.size();
      }
  QuadPack p;
  p.columns_at = ((size_t)(kQuadKinds * F + 1 + F) * sizeof(int32_t) + 15) / 16 * 16;
  p.weights_at = p.columns_at + columns * sizeof(QuadColumn);
  p.bytes.assign(p.weights_at + weights * sizeof(T), 0);
  int32_t* begin = reinterpret_cast<int32_t*>(p.bytes.data());
  QuadColumn* C = reinterpret_cast<QuadColumn*>(p.bytes.data() + p.columns_at);
  T* W = reinterpret_cast<T*>(p.bytes.data() + p.weights_at);
  int32_t e = 0, w = 0;
  for (int f = 0; f < F; ++f) {
    for (int k = 0; k < kQuadKinds; ++k) {
      begin[kQuadKinds * f + k] = e;
      for (const auto& q : st[f].columns[k]) {
        C[e++] = {q.dy * lz + q.dz, q.dy * lz - q.dz, q.up | q.down << 16, w / 4};
        for (double v : q.c) W[w++] = (T)v;
      }
    }
    begin[kQuadKinds * F + 1 + f] = st[f].reach;
  }
  begin[kQuadKinds * F] = e;
  return p;
}

template <typename T, int H>
inline void launch_sphere_quad_h(const QuadArgs& a, int F, hipStream_t s) {
  constexpr int HX = quad_tx(H, sizeof(T));
  static_assert(HX > 0, "tile does not fit the LDS budget");
  const int tiles_x = (a.nx + HX - 1) / HX;
  const dim3 grid((unsigned)(tiles_x * a.tiles_y * a.tiles_z), (unsigned)F);
  const dim3 block(kQuadCols * quad_split(H, sizeof(T)));
  if (a.even) hipLaunchKernelGGL((k_sphere_quad<T, H, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_sphere_quad<T, H, false>), grid, block, 0, s, a);
}

// The largest reach each precision's tile takes.
template <typename T>
constexpr int quad_max_reach() {
  int H = 1;
  while (quad_tx(H + 1, sizeof(T)) > 0) ++H;
  return H;
}

static_assert(quad_max_reach<float>() < 16, "QuadColumn::dx holds two masks of 16 bits");

// Launch for reach a.H, 1 <= a.H <= quad_max_reach<T>() (11 in FP32, 8 in FP64).
template <typename T, int H>
inline hipError_t launch_sphere_quad_upto(const QuadArgs& a, int F, hipStream_t s) {
  if constexpr (H > quad_max_reach<T>()) {
    return hipErrorInvalidValue;
  } else {
    if (a.H == H) {
      launch_sphere_quad_h<T, H>(a, F, s);
      return hipGetLastError();
    }
    return launch_sphere_quad_upto<T, H + 1>(a, F, s);
  }
}

template <typename T>
inline hipError_t launch_sphere_quad(const QuadArgs& a, int F, hipStream_t s) {
  return launch_sphere_quad_upto<T, 1>(a, F, s);
}

}  // namespace pnp
