// Exact coarse-grid solve of the V-cycle (Algorithm 1, "solve" on the
// coarsest level) for the assembled p = 1 operator.
//
// With nodes numbered plane by plane along z, the 27-point operator is block
// tridiagonal in blocks of one or more whole planes: D_k couples the nodes of
// block k among themselves, A_{k,k-1} its first plane to the last plane of the
// block below, A_{k,k+1} its last plane to the first of the block above.  Block
// elimination runs from both ends towards the middle block c = B/2 (a "twisted"
// factorisation), so the solve has two independent chains of half the length:
//   below c:  T_0 = D_0,  H_k = A_{k,k-1} G_{k-1},  T_k = D_k - H_k A_{k-1,k};
//   above c:  T_{B-1} = D_{B-1},  H_k = A_{k,k+1} G_{k+1},  T_k = D_k - H_k A_{k+1,k};
//   at c:     T_c = D_c - Hd_c A_{c-1,c} - Hu_c A_{c+1,c}   (both updates);
//   G_k = T_k^{-1}, and J_k = H_{k+1}^T (below c) or H_{k-1}^T (above c).
// H_k has the rows of one plane only (the first of block k below c, the last
// above), J_k its columns.  Solve: y_k = b_k - H_k y_{k-+1} walking inwards (the
// other planes of y_k are those of b_k), y_c = b_c - Hd_c y_{c-1} - Hu_c y_{c+1},
// x_c = G_c y_c, then outwards x_k = G_k y_k - J_k x_{k+-1}.  One launch advances
// both chains.
// Each T_k is symmetric positive definite (a Schur complement of an SPD
// matrix), so it is inverted in place by blocked Gauss-Jordan elimination
// without pivoting (32x32 blocks: invert the pivot block, scale its block row,
// update the rest, scale its block column).  Dirichlet rows of the stencil are
// identity rows, so they need no special case.  A pivot below 1e-12 of its
// row's diagonal (a numerically singular level, e.g. all-Neumann) is reported
// and the caller keeps the CG.  The diagonal is that of T_k, to which the blocks
// before k have contributed and the planes inside k have not: boxes more than about
// 5e6 times thinner in z than wide, with Neumann z-faces, fail the test in blocks of
// several planes (smallest pivot 2.2e-11 of its diagonal at 1e6, in single planes
// 0.87 at any ratio), so a level that fails is factored once more in single planes.
//
// Storage: per block G [Mp][Mp], H [mp][Mp] and J [Mp][mp] in FP64, Mp = the
// nodes of a block and mp = those of a plane rounded up to 32 (identity / zero
// padding); Hu_c sits in J's slot c.  A solve reads each block once, in about B
// dependent matrix-vector launches with no host interaction, so it can be
// recorded into a graph.  Under an FP32 smoother the sweeps read FP32 copies of
// the factored blocks instead (half the bytes; vectors and sums stay FP64): the
// solve is then exact to about 1e-6, below what the FP32 V-cycle around it
// resolves.
#include <algorithm>
#include <cstdlib>

#include "sem_internal.h"

namespace sem {

constexpr int kGB = 32;  // Gauss-Jordan block

static inline int64_t padded(int64_t m) { return (m + kGB - 1) / kGB * kGB; }

// Planes per block.  With g planes the solve is a chain of K / g launches instead
// of K and reads (g + 2) / 3 times the bytes, and the setup inverts blocks g
// times the size (g^2 times the operations).  g has the smallest sum of: 3.5 us
// per launch (its time before the first byte), the bytes at 4 TB/s (measured, per
// launch), and the inversions at 9 TFLOP/s (measured) spread over 300 solves; the
// blocks stay below 64 M entries (or 1.5 times those of single planes).  5^3
// nodes: one launch instead of 5; 9^3: one instead of 9 (32 us of an FP64 V-cycle's
// 412 at 9x7x8, p = 9: now 391); 17^3: 3 instead of 17; 33^3 keeps single planes
// (pairs: 1.3 % of the 32^3 solve for 30 ms of setup).
// planes > 0: that many instead.
BtShape coarse_direct_shape(int64_t nx, int64_t ny, int64_t nz, bool f32, int planes) {
  BtShape best{};
  double best_us = 0.0;
  const int64_t m = nx * ny, mp = padded(m), one = 3 * nz * mp * mp;
  const int64_t most = std::max<int64_t>((int64_t)64 << 20, one + one / 2);
  // SEM_COARSE_PLANES=g: that many planes per block
  const char *gv = getenv("SEM_COARSE_PLANES");
  if (planes == 0 && gv) planes = std::max(atoi(gv), 1);
  const int64_t forced = std::min<int64_t>(planes, nz);
  for (int64_t g = 1; g <= nz; ++g) {
    const int64_t B = (nz + g - 1) / g, Mp = padded(g * m), c = B / 2;
    const int64_t entries = B * (Mp * Mp + 2 * mp * Mp);
    if (forced ? g != forced : g > 1 && entries > most) continue;
    const int64_t up = std::max<int64_t>(std::max(c - 1, B - 2 - c), 0);
    const int64_t launches = B == 1 ? 1 : up + 2 + std::max(c, B - 1 - c);
    const double us = 3.5 * launches + (double)entries * (f32 ? 4 : 8) / 4e6 +
                      2.0 * B * Mp * Mp * (double)Mp / 9e6 / 300.0;
    if (best.g == 0 || us < best_us) {
      best_us = us;
      best = BtShape{(int)m, (int)nz, (int)g, (int)B, (int)Mp, (int)mp};
    }
  }
  return best;
}

// ---- setup kernels ----------------------------------------------------------

// stencil entry of row t for the node offset (dx, dy, dz)
__device__ inline double st_at(const double *St, int64_t n, int64_t t, int dx, int dy, int dz) {
  return St[(int64_t)((dz + 1) * 9 + (dy + 1) * 3 + (dx + 1)) * n + t];
}

// H[i][l] = sum_a A_{k,k+dz}[i][a] G_{k+dz}[a][l] (a over the plane of the
// neighbouring block next to this one: its rows from ra), dz = -1 or +1; plane =
// the plane of block k that takes it, ml = nodes of the neighbouring block
__global__ void k_bt_H(int nx, int ny, int64_t n, int plane, int ml, int mp, int Mp, int ra,
                       const double *__restrict__ St, const double *__restrict__ Gp,
                       double *__restrict__ H, int dz) {
  const int m = nx * ny;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)mp * Mp) return;
  const int i = (int)(e / Mp), l = (int)(e - (int64_t)i * Mp);
  double h = 0.0;
  if (i < m && l < ml) {
    const int xi = i % nx, yi = i / nx;
    const int64_t row = (int64_t)plane * m + i;
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        const int xa = xi + dx, ya = yi + dy;
        if (xa < 0 || xa >= nx || ya < 0 || ya >= ny) continue;
        h += st_at(St, n, row, dx, dy, dz) * Gp[(int64_t)(ra + ya * nx + xa) * Mp + l];
      }
  }
  H[e] = h;
}

// T[i][j] = D_k[i][j] - sum_l H1[i][l] A_{k,k-1}[j][l] (first plane)
//                     - sum_l H2[i][l] A_{k,k+1}[j][l] (last plane)
// (A_{k+dz,k} = A_{k,k+dz}^T; absent updates are null; padding: identity).  H1's
// columns of the plane below start at c1, H2's of the plane above at 0.  The
// diagonal is also kept in `diag` for the pivot test of the inversion.
__device__ inline double bt_update(int nx, int ny, int64_t n, int64_t rowj, int xj, int yj,
                                   const double *__restrict__ St, const double *__restrict__ Hi,
                                   int dz) {
  double v = 0.0;
  for (int ey = -1; ey <= 1; ++ey)
    for (int ex = -1; ex <= 1; ++ex) {
      const int xl = xj + ex, yl = yj + ey;
      if (xl < 0 || xl >= nx || yl < 0 || yl >= ny) continue;
      v += Hi[yl * nx + xl] * st_at(St, n, rowj, ex, ey, dz);
    }
  return v;
}

__global__ void k_bt_T(int nx, int ny, int64_t n, int plane0, int np, int Mp,
                       const double *__restrict__ St, const double *__restrict__ H1, int c1,
                       const double *__restrict__ H2, double *__restrict__ T,
                       double *__restrict__ diag) {
  const int m = nx * ny, M = np * m;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)Mp * Mp) return;
  const int i = (int)(e / Mp), j = (int)(e - (int64_t)i * Mp);
  if (i >= M || j >= M) {
    T[e] = i == j ? 1.0 : 0.0;
    if (i == j) diag[i] = 1.0;
    return;
  }
  const int pi = i / m, pj = j / m, ii = i - pi * m, jj = j - pj * m;
  const int xi = ii % nx, yi = ii / nx, xj = jj % nx, yj = jj / nx;
  const int dx = xj - xi, dy = yj - yi, dz = pj - pi;
  double v = 0.0;
  if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1)
    v = st_at(St, n, (int64_t)(plane0 + pi) * m + ii, dx, dy, dz);
  const int64_t rowj = (int64_t)(plane0 + pj) * m + jj;
  if (H1 && pi == 0 && pj == 0) v -= bt_update(nx, ny, n, rowj, xj, yj, St, H1 + (int64_t)ii * Mp + c1, -1);
  if (H2 && pi == np - 1 && pj == np - 1)
    v -= bt_update(nx, ny, n, rowj, xj, yj, St, H2 + (int64_t)ii * Mp, 1);
  T[e] = v;
  if (i == j) diag[i] = v;
}

// in-place inverse of the pivot block (Kb, Kb) in LDS.  For an SPD matrix
// every pivot lies in (0, original diagonal]; a pivot below 1e-12 of its row's
// original diagonal marks a (numerically) singular level.
__global__ __launch_bounds__(256) void k_gj_diag(double *A, int Mp, int Kb,
                                                 const double *__restrict__ diag, int *flag) {
  __shared__ double P[kGB][kGB + 1];
  const int tid = threadIdx.x;
  double *blk = A + (int64_t)Kb * kGB * Mp + (int64_t)Kb * kGB;
  for (int e = tid; e < kGB * kGB; e += 256) P[e / kGB][e % kGB] = blk[(int64_t)(e / kGB) * Mp + e % kGB];
  __syncthreads();
  for (int p = 0; p < kGB; ++p) {
    const double piv = P[p][p];
    const double d = 1.0 / piv;
    __syncthreads();
    if (tid < kGB && tid != p) P[p][tid] *= d;
    __syncthreads();
    for (int e = tid; e < kGB * kGB; e += 256) {
      const int i = e / kGB, j = e % kGB;
      if (i != p && j != p) P[i][j] -= P[i][p] * P[p][j];
    }
    __syncthreads();
    if (tid < kGB && tid != p) P[tid][p] = -P[tid][p] * d;
    if (tid == 0) {
      P[p][p] = d;
      if (!(piv > 1e-12 * diag[Kb * kGB + p])) atomicOr(flag, 1);
    }
    __syncthreads();
  }
  for (int e = tid; e < kGB * kGB; e += 256) blk[(int64_t)(e / kGB) * Mp + e % kGB] = P[e / kGB][e % kGB];
}

// block row: A[Kb][J] <- P A[Kb][J] for J != Kb (P = inverted pivot block)
__global__ __launch_bounds__(256) void k_gj_row(double *A, int Mp, int Kb) {
  __shared__ double P[kGB][kGB + 1], B[kGB][kGB + 1];
  const int tid = threadIdx.x;
  const int J = (int)blockIdx.x < Kb ? (int)blockIdx.x : (int)blockIdx.x + 1;
  const double *pb = A + (int64_t)Kb * kGB * Mp + (int64_t)Kb * kGB;
  double *tb = A + (int64_t)Kb * kGB * Mp + (int64_t)J * kGB;
  for (int e = tid; e < kGB * kGB; e += 256) {
    const int i = e / kGB, j = e % kGB;
    P[i][j] = pb[(int64_t)i * Mp + j];
    B[i][j] = tb[(int64_t)i * Mp + j];
  }
  __syncthreads();
  for (int e = tid; e < kGB * kGB; e += 256) {
    const int i = e / kGB, j = e % kGB;
    double s = 0.0;
#pragma unroll 8
    for (int q = 0; q < kGB; ++q) s += P[i][q] * B[q][j];
    tb[(int64_t)i * Mp + j] = s;
  }
}

// rest: A[I][J] -= A[I][Kb] A[Kb][J] for I, J != Kb (block row already scaled)
__global__ __launch_bounds__(256) void k_gj_trail(double *A, int Mp, int Kb, int nbk) {
  __shared__ double L[kGB][kGB + 1], R[kGB][kGB + 1];
  const int tid = threadIdx.x;
  const int ti = (int)blockIdx.x / (nbk - 1), tj = (int)blockIdx.x % (nbk - 1);
  const int I = ti < Kb ? ti : ti + 1, J = tj < Kb ? tj : tj + 1;
  const double *lb = A + (int64_t)I * kGB * Mp + (int64_t)Kb * kGB;
  const double *rb = A + (int64_t)Kb * kGB * Mp + (int64_t)J * kGB;
  double *ob = A + (int64_t)I * kGB * Mp + (int64_t)J * kGB;
  for (int e = tid; e < kGB * kGB; e += 256) {
    const int i = e / kGB, j = e % kGB;
    L[i][j] = lb[(int64_t)i * Mp + j];
    R[i][j] = rb[(int64_t)i * Mp + j];
  }
  __syncthreads();
  for (int e = tid; e < kGB * kGB; e += 256) {
    const int i = e / kGB, j = e % kGB;
    double s = 0.0;
#pragma unroll 8
    for (int q = 0; q < kGB; ++q) s += L[i][q] * R[q][j];
    ob[(int64_t)i * Mp + j] -= s;
  }
}

// block column: A[I][Kb] <- -A[I][Kb] P for I != Kb
__global__ __launch_bounds__(256) void k_gj_col(double *A, int Mp, int Kb) {
  __shared__ double P[kGB][kGB + 1], B[kGB][kGB + 1];
  const int tid = threadIdx.x;
  const int I = (int)blockIdx.x < Kb ? (int)blockIdx.x : (int)blockIdx.x + 1;
  const double *pb = A + (int64_t)Kb * kGB * Mp + (int64_t)Kb * kGB;
  double *tb = A + (int64_t)I * kGB * Mp + (int64_t)Kb * kGB;
  for (int e = tid; e < kGB * kGB; e += 256) {
    const int i = e / kGB, j = e % kGB;
    P[i][j] = pb[(int64_t)i * Mp + j];
    B[i][j] = tb[(int64_t)i * Mp + j];
  }
  __syncthreads();
  for (int e = tid; e < kGB * kGB; e += 256) {
    const int i = e / kGB, j = e % kGB;
    double s = 0.0;
#pragma unroll 8
    for (int q = 0; q < kGB; ++q) s += B[i][q] * P[q][j];
    tb[(int64_t)i * Mp + j] = -s;
  }
}

// J[i][a] = H[a][i], H [mp][Mp], J [Mp][mp]
__global__ void k_bt_transpose(int mp, int Mp, const double *__restrict__ H,
                               double *__restrict__ J) {
  __shared__ double t[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;  // 256 threads: 8 rows per pass
  for (int r = ty; r < 32; r += 8) t[r][tx] = H[(int64_t)(by + r) * Mp + bx + tx];
  __syncthreads();
  for (int r = ty; r < 32; r += 8) J[(int64_t)(bx + r) * mp + by + tx] = t[tx][r];
}

// ---- solve kernel -------------------------------------------------------------

// One product of a sweep over the rows of a block: out = c + s1 * (M1 v1) - (M2
// v2); a term holds for the rows r0 .. r0 + rows - 1 (row r0 is the matrix's row
// 0; rows = 0: absent), over n columns with row stride ld (zeros from n to ld).
// MT is the type of the stored blocks.
template <typename MT>
struct BtTerm {
  const MT *M;
  const double *v;
  int r0, rows, n, ld;
};
template <typename MT>
struct BtOp {
  BtTerm<MT> t1, t2;
  const double *c;
  double *out;
  double s1;
  int rows;  // of the block
};

__global__ void k_bt_narrow(int64_t n, const double *__restrict__ a, float *__restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

// Up to two independent products (the two chains of the sweep) for NV right
// sides (vectors vs apart in v1, v2, c and out); one wavefront per row, the
// matrix rows are read once for all right sides.  Each right side is summed in
// the same order for any NV (four strided partial sums per lane, then the wave
// reduction).
template <int NV, typename MT>
__global__ __launch_bounds__(256) void k_bt_mv(BtOp<MT> o0, BtOp<MT> o1, int rb, int64_t vs) {
  constexpr int W = 16 / (int)sizeof(MT);  // entries per 16-byte load
  struct alignas(16) Chunk {
    MT e[W];
  };
  const int which = (int)blockIdx.x >= rb;
  const BtOp<MT> &o = which ? o1 : o0;
  const int row = ((int)blockIdx.x - which * rb) * 4 + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= o.rows) return;  // whole wave
  double a1[NV], a2[NV];
  // The matrix row (16-byte aligned: ld is a multiple of 32) streams as 16-byte
  // loads of W entries, four per lane per step (256 W entries a wave), into four
  // partial sums per right side; x (L2 resident, any alignment) is read per
  // entry.  The last step's loads are issued together too, each if it starts
  // before ld; the row is zero from n on, where x is read at its last entry.
  auto rowdot = [&](const BtTerm<MT> &t_, double *acc) {
    const MT *__restrict__ r = t_.M + (int64_t)(row - t_.r0) * t_.ld;
    const double *__restrict__ x = t_.v;
    const int m = t_.n;
    double t[NV][4];
#pragma unroll
    for (int v = 0; v < NV; ++v) t[v][0] = t[v][1] = t[v][2] = t[v][3] = 0.0;
    const Chunk *__restrict__ rc = reinterpret_cast<const Chunk *>(r);
    int j0 = 0;
    for (; j0 + 256 * W <= m; j0 += 256 * W) {
      Chunk q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = rc[j0 / W + 64 * u + lane];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + 64 * W * u + W * lane;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double *xv = x + v * vs;
#pragma unroll
          for (int w = 0; w < W; ++w) t[v][u] += (double)q[u].e[w] * xv[j + w];
        }
      }
    }
    if (j0 < m) {
      Chunk q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + 64 * W * u + W * lane;
        if (j < t_.ld) {
          q[u] = rc[j / W];
        } else {
#pragma unroll
          for (int w = 0; w < W; ++w) q[u].e[w] = MT(0);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j0 + 64 * W * u >= m) break;
        const int j = j0 + 64 * W * u + W * lane;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double *xv = x + v * vs;
#pragma unroll
          for (int w = 0; w < W; ++w)
            t[v][u] += (double)q[u].e[w] * xv[j + w < m ? j + w : m - 1];
        }
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = (t[v][0] + t[v][1]) + (t[v][2] + t[v][3]);
  };
  const bool in1 = row >= o.t1.r0 && row < o.t1.r0 + o.t1.rows;
  const bool in2 = row >= o.t2.r0 && row < o.t2.r0 + o.t2.rows;
#pragma unroll
  for (int v = 0; v < NV; ++v) a1[v] = a2[v] = 0.0;
  if (in1) rowdot(o.t1, a1);
  if (in2) rowdot(o.t2, a2);
  if (in1 || in2) {
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        a1[v] += __shfl_xor(a1[v], sh, 64);
        a2[v] += __shfl_xor(a2[v], sh, 64);
      }
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      o.out[v * vs + row] = (o.c ? o.c[v * vs + row] : 0.0) + o.s1 * a1[v] - a2[v];
  }
}

// ---- host side -------------------------------------------------------------------

static inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

static void bt_invert(double *Gk, int Mp, int nbk, const double *diag, int *flag, hipStream_t s) {
  for (int b = 0; b < nbk; ++b) {
    hipLaunchKernelGGL(k_gj_diag, dim3(1), dim3(256), 0, s, Gk, Mp, b, diag, flag);
    SEM_LAUNCH("k_gj_diag");
    if (nbk == 1) continue;
    hipLaunchKernelGGL(k_gj_row, dim3(nbk - 1), dim3(256), 0, s, Gk, Mp, b);
    SEM_LAUNCH("k_gj_row");
    hipLaunchKernelGGL(k_gj_trail, dim3((nbk - 1) * (nbk - 1)), dim3(256), 0, s, Gk, Mp, b, nbk);
    SEM_LAUNCH("k_gj_trail");
    hipLaunchKernelGGL(k_gj_col, dim3(nbk - 1), dim3(256), 0, s, Gk, Mp, b);
    SEM_LAUNCH("k_gj_col");
  }
}

// the blocks of one factored operator
template <typename MT>
struct BtBlocks {
  MT *g, *h, *j;
  BtShape q;
  MT *G(int k) const { return g + (int64_t)k * q.Mp * q.Mp; }
  MT *H(int k) const { return h + (int64_t)k * q.mp * q.Mp; }
  MT *J(int k) const { return j + (int64_t)k * q.mp * q.Mp; }
  int plane0(int k) const { return k * q.g; }
  int planes(int k) const { return std::min(q.g, q.K - k * q.g); }
  int rows(int k) const { return planes(k) * q.m; }
};

// factors the level in the blocks S.shape; S.direct: no pivot failed its test
static void bt_factor(CoarseSolver &S, int64_t nx, int64_t ny, int64_t nz, hipStream_t s) {
  const BtBlocks<double> D{S.dG, S.dH, S.dJ, S.shape};
  const BtShape &q = S.shape;
  const int B = q.B, c = B / 2, Mp = q.Mp, mp = q.mp, nbk = Mp / kGB;
  const unsigned gT = nblk((int64_t)Mp * Mp), gH = nblk((int64_t)mp * Mp);
  if (q.m != nx * ny || q.K != nz) fail(SEM_EINVAL, "coarse solve: blocks of another grid");
  SEM_HIP(hipMemsetAsync(S.dflag, 0, sizeof(int), s));
  // H of block k towards k + dz, into `out`
  auto make_h = [&](int k, int dz, double *out) {
    const int nb = k + dz, plane = dz < 0 ? D.plane0(k) : D.plane0(k) + D.planes(k) - 1;
    hipLaunchKernelGGL(k_bt_H, dim3(gH), dim3(256), 0, s, (int)nx, (int)ny, S.n, plane, D.rows(nb),
                       mp, Mp, dz < 0 ? D.rows(nb) - q.m : 0, S.St, (const double *)D.G(nb), out, dz);
    SEM_LAUNCH("k_bt_H");
  };
  // T_k from the updates from below (hd) and above (hu), inverted in place
  auto make_g = [&](int k, const double *hd, const double *hu) {
    hipLaunchKernelGGL(k_bt_T, dim3(gT), dim3(256), 0, s, (int)nx, (int)ny, S.n, D.plane0(k),
                       D.planes(k), Mp, S.St, hd, hd ? D.rows(k - 1) - q.m : 0, hu, D.G(k), S.dy);
    SEM_LAUNCH("k_bt_T");
    bt_invert(D.G(k), Mp, nbk, S.dy, S.dflag, s);
  };
  for (int k = 0; k < c; ++k) {  // chain from block 0 up to c - 1
    if (k > 0) make_h(k, -1, D.H(k));
    make_g(k, k > 0 ? D.H(k) : nullptr, nullptr);
  }
  for (int k = B - 1; k > c; --k) {  // chain from block B - 1 down to c + 1
    if (k < B - 1) make_h(k, 1, D.H(k));
    make_g(k, nullptr, k < B - 1 ? D.H(k) : nullptr);
  }
  // block c takes both updates: from below in H's slot, from above in J's slot
  if (c > 0) make_h(c, -1, D.H(c));
  if (c < B - 1) make_h(c, 1, D.J(c));
  make_g(c, c > 0 ? D.H(c) : nullptr, c < B - 1 ? D.J(c) : nullptr);
  // back-substitution blocks: J_k = H_{k+1}^T below c, H_{k-1}^T above c (Hu_c for c + 1)
  for (int k = 0; k < B; ++k) {
    if (k == c) continue;
    const double *src = k < c ? D.H(k + 1) : (k - 1 == c ? D.J(c) : D.H(k - 1));
    hipLaunchKernelGGL(k_bt_transpose, dim3(Mp / 32, mp / 32), dim3(256), 0, s, mp, Mp, src, D.J(k));
    SEM_LAUNCH("k_bt_transpose");
  }
  if (S.fG) {
    const int64_t ng = (int64_t)B * Mp * Mp, nh = (int64_t)B * mp * Mp;
    hipLaunchKernelGGL(k_bt_narrow, dim3(nblk(ng)), dim3(256), 0, s, ng, (const double *)S.dG,
                       S.fG);
    hipLaunchKernelGGL(k_bt_narrow, dim3(nblk(nh)), dim3(256), 0, s, nh, (const double *)S.dH,
                       S.fH);
    hipLaunchKernelGGL(k_bt_narrow, dim3(nblk(nh)), dim3(256), 0, s, nh, (const double *)S.dJ,
                       S.fJ);
    SEM_LAUNCH("k_bt_narrow");
  }
  int flag = 0;
  SEM_HIP(hipMemcpyAsync(&flag, S.dflag, sizeof(int), hipMemcpyDeviceToHost, s));
  SEM_HIP(hipStreamSynchronize(s));
  S.direct = flag == 0;
}

void coarse_direct_setup(CoarseSolver &S, int64_t nx, int64_t ny, int64_t nz, hipStream_t s) {
  bt_factor(S, nx, ny, nz, s);
  if (S.direct || S.shape.g == 1) return;
  S.shape = coarse_direct_shape(nx, ny, nz, S.fG != nullptr, 1);
  bt_factor(S, nx, ny, nz, s);
}

template <int NV, typename MT>
static void bt_sweeps(const BtBlocks<MT> &D, int64_t vs, const double *b, double *x, double *y,
                      hipStream_t s) {
  using BtOp = sem::BtOp<MT>;
  using BtTerm = sem::BtTerm<MT>;
  const BtShape &q = D.q;
  const int B = q.B, c = B / 2, m = q.m;
  const BtTerm none{nullptr, nullptr, 0, 0, 0, 1};
  auto at = [&](const double *v, int k) { return v + (int64_t)D.plane0(k) * m; };
  auto to = [&](double *v, int k) { return v + (int64_t)D.plane0(k) * m; };
  // y_k of the sweep; y_0 and y_{B-1} are b itself (unless they are block c)
  auto Y = [&](int k) { return (k == 0 || k == B - 1) && k != c ? at(b, k) : at(y, k); };
  auto launch = [&](const BtOp &o0, const BtOp *o1) {
    const BtOp empty{};
    const int rows = std::max(o0.rows, o1 ? o1->rows : 0), rb = (rows + 3) / 4;
    hipLaunchKernelGGL((k_bt_mv<NV, MT>), dim3(o1 ? 2 * rb : rb), dim3(256), 0, s, o0,
                       o1 ? *o1 : empty, rb, vs);
    SEM_LAUNCH("k_bt_mv");
  };
  // the terms H_k v (v of the block below, dz = -1, or above), G_k v, J_k v (v
  // of the plane of the neighbouring block next to k)
  auto h_term = [&](const MT *H, int k, int dz) {
    return BtTerm{H, Y(k + dz), dz < 0 ? 0 : D.rows(k) - m, m, D.rows(k + dz), q.Mp};
  };
  auto g_term = [&](int k, const double *v) { return BtTerm{D.G(k), v, 0, D.rows(k), D.rows(k), q.Mp}; };
  auto j_term = [&](int k, int dz) {
    const double *v = dz > 0 ? at(x, k + 1) : at(x, k - 1) + (D.rows(k - 1) - m);
    return BtTerm{D.J(k), v, 0, D.rows(k), m, q.mp};
  };
  if (B == 1) {  // one block: x = G b
    launch(BtOp{g_term(0, b), none, nullptr, x, 1.0, D.rows(0)}, nullptr);
    return;
  }
  // inwards: y_k = b_k - H_k y_{k-1} (k < c), y_k = b_k - H_k y_{k+1} (k > c)
  for (int t = 1;; ++t) {
    const int kd = t, ku = B - 1 - t;
    const bool dn = kd < c, up = ku > c;
    if (!dn && !up) break;
    BtOp od{}, ou{};
    if (dn) od = BtOp{h_term(D.H(kd), kd, -1), none, at(b, kd), to(y, kd), -1.0, D.rows(kd)};
    if (up) ou = BtOp{h_term(D.H(ku), ku, 1), none, at(b, ku), to(y, ku), -1.0, D.rows(ku)};
    if (dn && up) launch(od, &ou);
    else launch(dn ? od : ou, nullptr);
  }
  // block c: y_c = b_c - Hd_c y_{c-1} - Hu_c y_{c+1}; x_c = G_c y_c
  launch(BtOp{c > 0 ? h_term(D.H(c), c, -1) : none, c < B - 1 ? h_term(D.J(c), c, 1) : none, at(b, c),
              to(y, c), -1.0, D.rows(c)},
         nullptr);
  launch(BtOp{g_term(c, at(y, c)), none, nullptr, to(x, c), 1.0, D.rows(c)}, nullptr);
  // outwards: x_k = G_k y_k - J_k x_{k+1} (k < c), x_k = G_k y_k - J_k x_{k-1} (k > c)
  for (int t = 1;; ++t) {
    const int kd = c - t, ku = c + t;
    const bool dn = kd >= 0, up = ku < B;
    if (!dn && !up) break;
    BtOp od{}, ou{};
    if (dn) od = BtOp{g_term(kd, Y(kd)), j_term(kd, 1), nullptr, to(x, kd), 1.0, D.rows(kd)};
    if (up) ou = BtOp{g_term(ku, Y(ku)), j_term(ku, -1), nullptr, to(x, ku), 1.0, D.rows(ku)};
    if (dn && up) launch(od, &ou);
    else launch(dn ? od : ou, nullptr);
  }
}

template <typename MT>
static void bt_apply(const CoarseSolver &S, const BtBlocks<MT> &D, const double *b, double *x,
                     hipStream_t s, int nv) {
  for (int v0 = 0; v0 < nv; v0 += 4) {  // up to four right sides per sweep
    const int64_t o = (int64_t)v0 * S.n;
    switch (std::min(4, nv - v0)) {
      case 1: bt_sweeps<1, MT>(D, S.n, b + o, x + o, S.dy + o, s); break;
      case 2: bt_sweeps<2, MT>(D, S.n, b + o, x + o, S.dy + o, s); break;
      case 3: bt_sweeps<3, MT>(D, S.n, b + o, x + o, S.dy + o, s); break;
      default: bt_sweeps<4, MT>(D, S.n, b + o, x + o, S.dy + o, s); break;
    }
  }
}

void coarse_direct_apply(const CoarseSolver &S, const double *b, double *x, hipStream_t s, int nv) {
  if (S.fG)
    bt_apply<float>(S, BtBlocks<float>{S.fG, S.fH, S.fJ, S.shape}, b, x, s, nv);
  else
    bt_apply<double>(S, BtBlocks<double>{S.dG, S.dH, S.dJ, S.shape}, b, x, s, nv);
}

}  // namespace sem
