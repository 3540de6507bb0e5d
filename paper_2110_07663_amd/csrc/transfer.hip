// p-multigrid transfers (Sec. 2.2.2, Algorithm 1, "coarsen" and "prolongate").
//
// P interpolates the coarse cardinal basis to the fine GLL nodes element by
// element, P = J (x) J (x) J with J[i][j] = h^c_j(xi^f_i); a continuous coarse
// field stays continuous, so the fine E-vector comes out consistent.
// P^T (on global vectors) = assemble_c o (J^T (x) J^T (x) J^T) o (1/mult_f):
// the consistent fine residual is split among its copies, contracted, then
// summed over shared coarse nodes (QQ^T) and masked by the caller.
#include "sem_internal.h"

namespace sem {

constexpr int kTN = 11;  // largest N handled (p <= 10)

// any sizes, from the arguments; one element per workgroup
template <typename T>
__global__ __launch_bounds__(256) void k_prolong(int Nf, int Nc, const T *__restrict__ J,
                                                 const T *__restrict__ xc, T *__restrict__ xf) {
  __shared__ T sJ[kTN * kTN];
  __shared__ T a[kTN * kTN * kTN];
  __shared__ T b[kTN * kTN * kTN];
  const int64_t e = blockIdx.x;
  const int tid = threadIdx.x, bs = (int)blockDim.x;
  const int Nc3 = Nc * Nc * Nc, Nf3 = Nf * Nf * Nf;
  xc += blockIdx.y * (int64_t)gridDim.x * Nc3;  // right side blockIdx.y
  xf += blockIdx.y * (int64_t)gridDim.x * Nf3;
  for (int t = tid; t < Nf * Nc; t += bs) sJ[t] = J[t];
  for (int t = tid; t < Nc3; t += bs) a[t] = xc[e * Nc3 + t];
  __syncthreads();
  // b[c][bb][i] = sum_a J[i][a] x[c][bb][a]
  for (int t = tid; t < Nc * Nc * Nf; t += bs) {
    int i = t % Nf, cb = t / Nf;
    T s = 0;
    for (int q = 0; q < Nc; ++q) s += sJ[i * Nc + q] * a[cb * Nc + q];
    b[t] = s;
  }
  __syncthreads();
  // a[c][j][i] = sum_bb J[j][bb] b[c][bb][i]
  for (int t = tid; t < Nc * Nf * Nf; t += bs) {
    int i = t % Nf, j = (t / Nf) % Nf, c = t / (Nf * Nf);
    T s = 0;
    for (int q = 0; q < Nc; ++q) s += sJ[j * Nc + q] * b[(c * Nc + q) * Nf + i];
    a[t] = s;
  }
  __syncthreads();
  // xf[k][j][i] += sum_c J[k][c] a[c][j][i]
  for (int t = tid; t < Nf3; t += bs) {
    int ji = t % (Nf * Nf), k = t / (Nf * Nf);
    T s = 0;
    for (int q = 0; q < Nc; ++q) s += sJ[k * Nc + q] * a[q * Nf * Nf + ji];
    xf[e * Nf3 + t] += s;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_restrict(int Nf, int Nc, const T *__restrict__ J,
                                                  const T *__restrict__ w, const T *__restrict__ rf,
                                                  const T *__restrict__ bf, T *__restrict__ rc) {
  __shared__ T sJ[kTN * kTN];
  __shared__ T a[kTN * kTN * kTN];
  __shared__ T b[kTN * kTN * kTN];
  const int64_t e = blockIdx.x;
  const int tid = threadIdx.x, bs = (int)blockDim.x;
  const int Nc3 = Nc * Nc * Nc, Nf3 = Nf * Nf * Nf;
  rf += blockIdx.y * (int64_t)gridDim.x * Nf3;  // right side blockIdx.y
  rc += blockIdx.y * (int64_t)gridDim.x * Nc3;
  for (int t = tid; t < Nf * Nc; t += bs) sJ[t] = J[t];
  if (bf) {  // residual b - A x formed on the way in
    bf += blockIdx.y * (int64_t)gridDim.x * Nf3;
    for (int t = tid; t < Nf3; t += bs) a[t] = w[e * Nf3 + t] * (bf[e * Nf3 + t] - rf[e * Nf3 + t]);
  } else {
    for (int t = tid; t < Nf3; t += bs) a[t] = w[e * Nf3 + t] * rf[e * Nf3 + t];
  }
  __syncthreads();
  // b[k][j][aa] = sum_i J[i][aa] r[k][j][i]
  for (int t = tid; t < Nf * Nf * Nc; t += bs) {
    int aa = t % Nc, kj = t / Nc;
    T s = 0;
    for (int q = 0; q < Nf; ++q) s += sJ[q * Nc + aa] * a[kj * Nf + q];
    b[t] = s;
  }
  __syncthreads();
  // a[k][bb][aa] = sum_j J[j][bb] b[k][j][aa]
  for (int t = tid; t < Nf * Nc * Nc; t += bs) {
    int aa = t % Nc, bb = (t / Nc) % Nc, k = t / (Nc * Nc);
    T s = 0;
    for (int q = 0; q < Nf; ++q) s += sJ[q * Nc + bb] * b[(k * Nf + q) * Nc + aa];
    a[t] = s;
  }
  __syncthreads();
  // rc[c][bb][aa] = sum_k J[k][c] a[k][bb][aa]
  for (int t = tid; t < Nc3; t += bs) {
    int ba = t % (Nc * Nc), c = t / (Nc * Nc);
    T s = 0;
    for (int q = 0; q < Nf; ++q) s += sJ[q * Nc + c] * a[q * Nc * Nc + ba];
    rc[e * Nc3 + t] = s;
  }
}

// Sizes fixed at compile time: NF^2 threads per element, EPB elements per
// workgroup.  A thread owns a line of the direction being contracted, holds it in
// registers and forms all its outputs with the entries of J as scalar operands
// (the same for every element).  k goes last (prolongation) or first
// (restriction): its lines are the element's (i, j) columns, so global memory is
// read and written plane by plane, contiguously, and all NF loads of a thread are
// in flight at once, before the other contractions (prolongation) or all at the
// start (restriction).  Bound by memory: restriction reads the fine vector (its
// weight mask / multiplicity is formed from the grid position, exact), the
// prolongation reads and writes it.  At 20^3 elements, p = 9 -> 5, FP32 (39 and 71
// MB) 11.8 and 14.2 us (3.3 and 5.0 TB/s; 22.5 and 20.6 before: the stored weights
// read as a third vector, one output per thread and step with one
// LDS read per multiply-add, 256 threads for any element).
template <int NF>
struct TrShape {
  static constexpr int NF2 = NF * NF;
  static constexpr int EPB = NF2 >= 128 ? 1 : 256 / NF2;
  static constexpr int BS = (EPB * NF2 + 63) / 64 * 64;
};
template <typename T, int NF, int NC>
__global__ __launch_bounds__(TrShape<NF>::BS) void k_prolong_l(int64_t E, const T *__restrict__ J,
                                                               const T *__restrict__ xc,
                                                               T *__restrict__ xf, int stream) {
  using S = TrShape<NF>;
  constexpr int NF2 = S::NF2, EPB = S::EPB, Nc2 = NC * NC, Nc3 = Nc2 * NC, Nf3 = NF2 * NF;
  __shared__ T sa[EPB][Nc2 * NF];   // [c][b][i]
  __shared__ T sb[EPB][NC * NF2];   // [c][j][i]
  const int le = threadIdx.x / NF2, l = threadIdx.x - le * NF2;
  const int64_t e = (int64_t)blockIdx.x * EPB + le;
  const bool act = le < EPB && e < E;
  xc += (blockIdx.y * E + e) * Nc3;  // right side blockIdx.y
  xf += (blockIdx.y * E + e) * Nf3 + l;
  T old[NF];
  if (act) {
#pragma unroll
    for (int k = 0; k < NF; ++k)
      old[k] = stream ? __builtin_nontemporal_load(xf + k * NF2) : xf[k * NF2];
    // sa[c][b][i] = sum_a J[i][a] xc[c][b][a]: line (c, b)
    if (l < Nc2) {
      T v[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) v[q] = xc[l * NC + q];
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        T s = 0;
#pragma unroll
        for (int q = 0; q < NC; ++q) s += J[i * NC + q] * v[q];
        sa[le][l * NF + i] = s;
      }
    }
  }
  __syncthreads();
  if (act && l < NC * NF) {  // sb[c][j][i] = sum_b J[j][b] sa[c][b][i]: line (c, i)
    const int c = l / NF, i = l - c * NF;
    T v[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) v[q] = sa[le][(c * NC + q) * NF + i];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      T s = 0;
#pragma unroll
      for (int q = 0; q < NC; ++q) s += J[j * NC + q] * v[q];
      sb[le][(c * NF + j) * NF + i] = s;
    }
  }
  __syncthreads();
  if (!act) return;
  T v[NC];  // xf[k][j][i] += sum_c J[k][c] sb[c][j][i]: line (j, i)
#pragma unroll
  for (int q = 0; q < NC; ++q) v[q] = sb[le][q * NF2 + l];
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    T s = 0;
#pragma unroll
    for (int q = 0; q < NC; ++q) s += J[k * NC + q] * v[q];
    old[k] += s;
    if (stream)
      __builtin_nontemporal_store(old[k], xf + k * NF2);
    else
      xf[k * NF2] = old[k];
  }
}

template <typename T, int NF, int NC>
__global__ __launch_bounds__(TrShape<NF>::BS) void k_restrict_l(int64_t E, int nex, int ney, int nez,
                                                                int bcm, const T *__restrict__ J,
                                                                const T *__restrict__ rf,
                                                                const T *__restrict__ bf,
                                                                T *__restrict__ rc) {
  using S = TrShape<NF>;
  constexpr int NF2 = S::NF2, EPB = S::EPB, Nc2 = NC * NC, Nc3 = Nc2 * NC, Nf3 = NF2 * NF;
  __shared__ T sa[EPB][NC * NF2];   // [c][j][i]
  __shared__ T sb[EPB][Nc2 * NF];   // [c][b][i]
  const int le = threadIdx.x / NF2, l = threadIdx.x - le * NF2;
  const int64_t e = (int64_t)blockIdx.x * EPB + le;
  const bool act = le < EPB && e < E;
  const int64_t at = (blockIdx.y * E + e) * Nf3 + l;  // right side blockIdx.y
  if (act) {  // sa[c][j][i] = sum_k J[k][c] w r[k][j][i]: line (j, i)
    T v[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) v[k] = rf[at + k * NF2];
    if (bf) {  // b - A x on the way in
#pragma unroll
      for (int k = 0; k < NF; ++k) v[k] = bf[at + k * NF2] - v[k];
    }
    int64_t ex, ey, ez;
    elem_coords(e, nex, ney, ex, ey, ez);
    const int j = l / NF, i = l - j * NF;
    const T wij = node_w1(i, NF, ex, nex, bcm, 0) * node_w1(j, NF, ey, ney, bcm, 2);
    const T wlo = node_w1(0, NF, ez, nez, bcm, 4), whi = node_w1(NF - 1, NF, ez, nez, bcm, 4);
#pragma unroll
    for (int k = 0; k < NF; ++k) v[k] *= k == 0 ? wij * wlo : (k == NF - 1 ? wij * whi : wij);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      T s = 0;
#pragma unroll
      for (int k = 0; k < NF; ++k) s += J[k * NC + c] * v[k];
      sa[le][c * NF2 + l] = s;
    }
  }
  __syncthreads();
  if (act && l < NC * NF) {  // sb[c][b][i] = sum_j J[j][b] sa[c][j][i]: line (c, i)
    const int c = l / NF, i = l - c * NF;
    T v[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) v[j] = sa[le][(c * NF + j) * NF + i];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      T s = 0;
#pragma unroll
      for (int j = 0; j < NF; ++j) s += J[j * NC + q] * v[j];
      sb[le][(c * NC + q) * NF + i] = s;
    }
  }
  __syncthreads();
  if (act && l < Nc2) {  // rc[c][b][a] = sum_i J[i][a] sb[c][b][i]: line (c, b)
    T v[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) v[i] = sb[le][l * NF + i];
    T *out = rc + (blockIdx.y * E + e) * Nc3 + l * NC;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      T s = 0;
#pragma unroll
      for (int i = 0; i < NF; ++i) s += J[i * NC + q] * v[i];
      out[q] = s;
    }
  }
}

static int transfer_threads(int Nf) {
  int n = Nf * Nf * Nf;
  int t = ((n + 63) / 64) * 64;
  return t > 256 ? 256 : t;
}

// compile-time sizes for the pairs (fine N, coarse N) of the usual schedules, the
// generic kernels otherwise
#define SEM_TRANSFER_PAIRS(X)                                                             \
  X(3, 2) X(4, 2) X(4, 3) X(5, 2) X(5, 3) X(6, 2) X(6, 4) X(7, 4) X(8, 2) X(8, 4) X(8, 6) \
  X(9, 5) X(10, 4) X(10, 6) X(10, 8) X(11, 6)

template <typename T>
void launch_prolong(const Level &F, const Level &C, const T *xc, T *xf, hipStream_t s, int nv) {
  const T *J = sizeof(T) == 8 ? (const T *)F.J64 : (const T *)F.J32;
  // (the fine vector past the caches where it would displace what they hold)
  const int stream = F.nloc * nv * (int64_t)sizeof(T) > (int64_t)48 << 20;
#define SEM_PROLONG_CASE(NF, NC)                                                             \
  if (F.N == NF && C.N == NC) {                                                              \
    constexpr int EPB = TrShape<NF>::EPB;                                                    \
    hipLaunchKernelGGL((k_prolong_l<T, NF, NC>), dim3((unsigned)((F.E + EPB - 1) / EPB), (unsigned)nv), \
                       dim3(TrShape<NF>::BS), 0, s, F.E, J, xc, xf, stream);                 \
    SEM_LAUNCH("k_prolong");                                                                 \
    return;                                                                                  \
  }
  SEM_TRANSFER_PAIRS(SEM_PROLONG_CASE)
#undef SEM_PROLONG_CASE
  hipLaunchKernelGGL(k_prolong<T>, dim3((unsigned)F.E, (unsigned)nv), dim3(transfer_threads(F.N)), 0, s,
                     F.N, C.N, J, xc, xf);
  SEM_LAUNCH("k_prolong");
}

template <typename T>
void launch_restrict(const Level &F, const Level &C, const T *rf, T *rc, hipStream_t s, int nv,
                     const T *bf) {
  const T *J = sizeof(T) == 8 ? (const T *)F.J64 : (const T *)F.J32;
  const T *w = sizeof(T) == 8 ? (const T *)F.w64 : (const T *)F.w32;
  int bcm = 0;
  for (int f = 0; f < 6; ++f) bcm |= (F.bc[f] ? 1 : 0) << f;
#define SEM_RESTRICT_CASE(NF, NC)                                                             \
  if (F.N == NF && C.N == NC) {                                                               \
    constexpr int EPB = TrShape<NF>::EPB;                                                     \
    hipLaunchKernelGGL((k_restrict_l<T, NF, NC>), dim3((unsigned)((F.E + EPB - 1) / EPB), (unsigned)nv), \
                       dim3(TrShape<NF>::BS), 0, s, F.E, F.nex, F.ney, F.nez, bcm, J, rf, bf, rc); \
    SEM_LAUNCH("k_restrict");                                                                 \
    return;                                                                                   \
  }
  SEM_TRANSFER_PAIRS(SEM_RESTRICT_CASE)
#undef SEM_RESTRICT_CASE
  hipLaunchKernelGGL(k_restrict<T>, dim3((unsigned)F.E, (unsigned)nv), dim3(transfer_threads(F.N)), 0, s,
                     F.N, C.N, J, w, rf, bf, rc);
  SEM_LAUNCH("k_restrict");
}
#undef SEM_TRANSFER_PAIRS

template void launch_prolong<double>(const Level &, const Level &, const double *, double *,
                                     hipStream_t, int);
template void launch_prolong<float>(const Level &, const Level &, const float *, float *,
                                    hipStream_t, int);
template void launch_restrict<double>(const Level &, const Level &, const double *, double *,
                                      hipStream_t, int, const double *);
template void launch_restrict<float>(const Level &, const Level &, const float *, float *,
                                     hipStream_t, int, const float *);

}  // namespace sem
