// FP64 Schwarz local solves by the fast diagonalisation method (Sec. 2.2.2,
// eqs. 8-9) on the matrix cores, RAS and ASM.
//
// Each of the six 1D contractions of the (p+3)^3 box is out[m][line] =
// sum_k S[k][m] in[k][line].  v_mfma_f64_4x4x4 (four blocks) takes four k and
// four m for 16 lines at a time: lane 16k + line holds in[k][line] (B), lane
// 16k + 4b + i holds S[k][i] (A, the same in the four blocks b), and lane
// 16m + line receives out[m][line].  The result of a contraction therefore has
// the layout of an operand whose k is the old m, and the forward x pass, the
// division by the eigenvalue sums and the backward x pass follow each other in
// registers; the other passes exchange lines through LDS.
//
// Why the matrix cores: FP64 runs at the same rate there and on the vector
// pipe (66 and 60 TFLOP/s measured with independent products), but the vector
// form needs every entry of the three factors as a scalar operand, and the
// scalar loads of 2.4 KB of factors per element (p = 7; all elements of a CU
// together exceed the scalar cache) stalled it for three quarters of its time:
// 63 us for 8000 elements against 38.7 us here (RAS; its HBM
// traffic alone would take 16 us).  What bounds it now: the matrix pipe is busy
// 48 % of the cycles (68 % of that on real entries, the rest pads 10 modes and
// nodes to 12 and 100 lines to 112) and the vector pipe most of the others
// (addresses, the 1000 reciprocals of the eigenvalue sums).
//
// The passes run z, y, x forward and x, y, z backward, so that the first
// reads and the last writes address consecutive nodes of the E-vector across
// the 16 lines.  One wavefront per element, four per workgroup, no workgroup
// barriers; on small meshes four per element (WPE below).
#include "sem_internal.h"

namespace sem {

namespace {

template <int P, bool ASM, int WPE = 1>  // WPE: wavefronts per element
struct Md {
  static constexpr int PB = P + 3, N = P + 1, N3 = N * N * N;
  static constexpr int K4 = (PB + 3) / 4;        // groups of four k or modes
  static constexpr int NK = ASM ? PB : N;        // nodes kept per direction
  static constexpr int K0 = ASM ? 0 : 1;         // the first of them
  static constexpr int KG = (NK + 3) / 4;        // groups of four kept nodes
  static constexpr int L3 = PB * PB, S3 = (L3 + 15) / 16;  // lines and slots of 16
  static constexpr int L2 = NK * PB, S2 = (L2 + 15) / 16;  // backward y: (i, c')
  static constexpr int L1 = NK * NK, S1 = (L1 + 15) / 16;  // backward z: (i, j)
  // LDS addresses (doubles) of the exchanges, each written by one pass (16
  // lines across lanes, digit d0 fastest) and read by the next along another
  // direction.  One side of each is linear in the line number, the other
  // needs the line's second digit alone:
  //   1: Y a + X b + c'    written over (a, b), read over (c', a): line + X b
  //   2: c' + Y a + X b'   written over (c', a): line + X b', read over (c', b')
  //   3: c' + Y b' + X i   written over (c', b'): line + X i, read over (c', i)
  //   4: c' + Y i + X j    written over (c', i): line + X j, read over (i, j)
  // (a line of the digits d0, d1 has the number d0 + Y d1 there).
  static constexpr int Y = PB | 1, X = PB * Y;
  // Lanes past the last line read (and never write): their second digit is
  // held at the last one, and BOX covers every address they then form.
  // (slots in multiples of the element's waves)
  static constexpr int Q3 = (S3 + WPE - 1) / WPE * WPE * 16, Q1 = (S1 + WPE - 1) / WPE * WPE * 16;
  static constexpr int D3 = Q3 - 1 - (PB - 1) * PB, D1 = Q1 - 1 - (NK - 1) * NK;
  static constexpr int R1 = Q3 - 1 + (PB - 1) * (X + Y - PB), R2 = D3 + (PB - 1) * (X + Y);
  static constexpr int R3 = D1 * Y + (NK - 1) * X + PB - 1, R12 = R1 > R2 ? R1 : R2;
  static constexpr int BOX = (R12 > R3 ? R12 : R3) + 1;
  static constexpr int LAM = D3 < PB ? 3 * PB : 2 * PB + D3 + 1;  // eigenvalues, and what those lanes read
  static constexpr int BUF = BOX + LAM;
  static constexpr int WAVES = 4;
};

// Raw-buffer view of an FP64 array: a load at a byte offset past the window
// returns zero, as nodes outside the domain and the padding of the factors do.
constexpr uint32_t kOut64 = 0x80000000u;
constexpr uint32_t kWin64 = 0x7FFFFF00u;
struct BufF64 {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ BufF64(const double *p, uint32_t nbytes)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), (short)0, (int)nbytes,
                                               0x00020000)) {}
  __device__ double ld(uint32_t off, int imm = 0) const {  // imm < 4096
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off + imm, 0, 0));
  }
};

// 1 / d by two Newton steps from the hardware estimate (within an ulp).
// Decoupled nodes carry kHuge instead of +inf: their quotients are some 1e-300
// of the others, and only nodes whose weight is zero, or that nobody reads, see
// them.  A zero sum (a box floating on Neumann faces in all directions) stays
// with the vector kernel, which drops that mode.
constexpr double kHuge = 1e300;
__device__ inline double md_inv(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
  return __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
}

// orders the LDS traffic of the element's wavefronts between passes
template <int WPE>
__device__ inline void md_sync() {
  if constexpr (WPE > 1) {
    __syncthreads();
  } else {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only
    __builtin_amdgcn_wave_barrier();
  }
}

// A operands of direction d: forward (k group, m group) -> lane (k, m) holds
// S[4kg + k][4g + m]; backward (m group, node group) -> S[K0 + 4g + i][4mg + m];
// zero past the factor
template <int P, bool ASM>
__device__ __attribute__((always_inline)) inline void md_forward_op(const BufF64 &Se, int d,
                                                                    int lane, double *A) {
  using F = Md<P, ASM>;
  const int k = lane >> 4, m = lane & 3;
  const uint32_t in = (uint32_t)(k * F::PB + m) * 8;
  const bool kl = 4 * (F::K4 - 1) + k < F::PB, ml = 4 * (F::K4 - 1) + m < F::PB;
  const uint32_t at[2][2] = {{in, ml ? in : kOut64}, {kl ? in : kOut64, kl && ml ? in : kOut64}};
#pragma unroll
  for (int kg = 0; kg < F::K4; ++kg)
#pragma unroll
    for (int g = 0; g < F::K4; ++g)
      A[kg * F::K4 + g] = Se.ld(at[kg == F::K4 - 1][g == F::K4 - 1],
                                ((d * F::PB + 4 * kg) * F::PB + 4 * g) * 8);
}
template <int P, bool ASM>
__device__ __attribute__((always_inline)) inline void md_backward_op(const BufF64 &Se, int d,
                                                                     int lane, double *A) {
  using F = Md<P, ASM>;
  const int m = lane >> 4, i = lane & 3;
  const uint32_t in = (uint32_t)(i * F::PB + m) * 8;
  const bool ml = 4 * (F::K4 - 1) + m < F::PB, il = 4 * (F::KG - 1) + i < F::NK;
  const uint32_t at[2][2] = {{in, il ? in : kOut64}, {ml ? in : kOut64, ml && il ? in : kOut64}};
#pragma unroll
  for (int mg = 0; mg < F::K4; ++mg)
#pragma unroll
    for (int g = 0; g < F::KG; ++g)
      A[mg * F::KG + g] = Se.ld(at[mg == F::K4 - 1][g == F::KG - 1],
                                ((d * F::PB + F::K0 + 4 * g) * F::PB + 4 * mg) * 8);
}

// acc[s][g] = sum over the k groups, the operand of slot s and group kg from
// in(s, kg)
template <int S, int K, int G, typename In>
__device__ __attribute__((always_inline)) inline void md_contract(const double *A, In in,
                                                                  double (&acc)[S][G]) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    double b[K];
#pragma unroll
    for (int kg = 0; kg < K; ++kg) b[kg] = in(s, kg);
#pragma unroll
    for (int g = 0; g < G; ++g) acc[s][g] = 0.0;
#pragma unroll
    for (int kg = 0; kg < K; ++kg)
#pragma unroll
      for (int g = 0; g < G; ++g)
        acc[s][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[kg * G + g], b[kg], acc[s][g], 0, 0, 0);
  }
}

struct RasGrid {
  int bcm;  // bit f set when domain face f (x-, x+, y-, y+, z-, z+) is Dirichlet
};

// RAS: z = the element's own nodes times the RAS weight (mask / multiplicity,
// formed from the grid position: exact, equal to the assembled weight);
// ASM: z = the whole boxes [E][PB^3].
// RS: the local solves act on r - rs (a residual formed as it is read).
// WPE: wavefronts per element.  One (four elements per workgroup) fills the device
// from a few thousand elements on; below, a launch lasts as long as one element's
// chain of passes, and WPE = 4 (one element per workgroup, its line slots dealt
// out to the waves, workgroup barriers between the passes) shortens that.
template <int P, bool ASM, bool RS, int WPE>
__global__ __launch_bounds__(256) void k_fdm_mf64(int64_t E, int nex, int ney, int nez,
                                                  const double *__restrict__ r,
                                                  const double *__restrict__ rs,
                                                  const double *__restrict__ Sg,
                                                  const double *__restrict__ lamg, RasGrid W,
                                                  double *__restrict__ z, int nv) {
  using F = Md<P, ASM, WPE>;
  constexpr int PB = F::PB, N = F::N, N3 = F::N3, K4 = F::K4, KG = F::KG, NK = F::NK;
  constexpr int EPB = F::WAVES / WPE;
  __shared__ double lds[EPB * F::BUF];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave % WPE;  // the wave takes the slots sub, sub + WPE, ...
  constexpr int S3 = (F::S3 + WPE - 1) / WPE, S2 = (F::S2 + WPE - 1) / WPE, S1 = (F::S1 + WPE - 1) / WPE;
  const int lane = threadIdx.x & 63, hi = lane >> 4, lo = lane & 15;
  int vec;
  const int64_t e = (int64_t)split_rhs(xcd_block(), nv, vec) * EPB + wave / WPE;
  if (e >= E) return;  // whole wave (WPE = 1: no workgroup barriers below), else whole workgroup
  r += (int64_t)vec * E * N3;
  if (RS) rs += (int64_t)vec * E * N3;
  z += (int64_t)vec * E * (ASM ? PB * PB * PB : N3);
  double *buf = lds + wave / WPE * F::BUF, *lam = buf + F::BOX;
  // the wave's reads start at most a plane, a line and an element below e
  const int64_t back = (int64_t)nex * ney + nex + 1, eb = e > back ? e - back : 0;
  const int64_t wb = (E - eb) * N3 * 8;
  const uint32_t wn = wb < (int64_t)kWin64 ? (uint32_t)wb : kWin64;
  const BufF64 rb(r + eb * N3, wn), rsb(RS ? rs + eb * N3 : r + eb * N3, wn);
  const BufF64 Se(Sg + e * 3 * PB * PB, 3 * PB * PB * 8);

  double Af[K4 * K4], Ab[K4 * KG];
  md_forward_op<P, ASM>(Se, 2, lane, Af);
  if (sub == 0 && lane < 3 * PB) lam[lane] = fmin(lamg[e * 3 * PB + lane], kHuge);

  int64_t ex64, ey64, ez64;
  elem_coords(e, nex, ney, ex64, ey64, ez64);
  const int ex = (int)ex64, ey = (int)ey64, ez = (int)ez64;
  // first line of the wave's slot s, and a bound on its last over the waves
  auto at0 = [&](int s) { return 16 * (WPE * s + sub); };
  auto last = [](int s) constexpr { return 16 * (WPE * s + WPE - 1) + 15; };
  // the second digits of the lane's lines
  int hi3[S3];
#pragma unroll
  for (int s = 0; s < S3; ++s) {
    const int d = (at0(s) + lo) / PB;
    hi3[s] = last(s) < F::L3 ? d : (d < PB ? d : PB - 1);
  }
  // z forward on the box lines (a, b): node c = 4kg + hi of the lane's line.
  // Byte offsets from element eb; a neighbour outside the domain sets bit 31,
  // which puts the offset past the window.
  constexpr uint32_t kO = kOut64;
  const uint32_t plane = (uint32_t)(nex * ney) * (N3 * 8), line = (uint32_t)nex * (N3 * 8);
  uint32_t zoff[K4], zbit[K4];
#pragma unroll
  for (int kg = 0; kg < K4; ++kg) {
    const int c = 4 * kg + hi;
    zoff[kg] = (uint32_t)(c - 1) * (N * N * 8);
    zbit[kg] = 0;
    if (kg == 0) {
      zoff[kg] = c == 0 ? (P - 1) * N * N * 8 - plane : zoff[kg];
      zbit[kg] = c == 0 && ez == 0 ? kO : 0;
    }
    if (4 * kg + 3 >= PB - 1) {
      zoff[kg] = c == PB - 1 ? N * N * 8 + plane : zoff[kg];
      zbit[kg] |= c >= PB || (c == PB - 1 && ez == nez - 1) ? kO : 0;
    }
  }
  const uint32_t base = (uint32_t)(e - eb) * (N3 * 8);
  const uint32_t xl = ex == 0 ? kO : 0, xr = ex == nex - 1 ? kO : 0;
  const uint32_t yl = ey == 0 ? kO : 0, yr = ey == ney - 1 ? kO : 0;
  double f3[S3][K4];
  {
    double in[S3][K4];
#pragma unroll
    for (int s = 0; s < S3; ++s) {
      const int b = hi3[s], a = at0(s) + lo - b * PB;
      uint32_t at = (uint32_t)((b - 1) * N + a - 1) * 8, bit = 0;
      at = a == 0 ? at + (P - N3) * 8 : (a == PB - 1 ? at + (N3 - P) * 8 : at);
      bit = a == 0 ? xl : (a == PB - 1 ? xr : 0);
      at = b == 0 ? at + P * N * 8 - line : (b == PB - 1 ? at - P * N * 8 + line : at);
      bit |= b == 0 ? yl : (b == PB - 1 ? yr : 0);
      if (last(s) >= F::L3) bit = at0(s) + lo >= F::L3 ? kO : bit;
      at += base;
#pragma unroll
      for (int kg = 0; kg < K4; ++kg) {
        const uint32_t off = (at + zoff[kg]) | bit | zbit[kg];
        in[s][kg] = rb.ld(off);
        if constexpr (RS) in[s][kg] -= rsb.ld(off);
      }
    }
    md_contract<S3, K4, K4>(Af, [&](int s, int kg) { return in[s][kg]; }, f3);
  }
  md_forward_op<P, ASM>(Se, 1, lane, Af);
#pragma unroll
  for (int s = 0; s < S3; ++s) {
    const int l = at0(s) + lo, b = hi3[s], at = (l - b * PB) * F::Y + b * F::X + hi;
#pragma unroll
    for (int g = 0; g < K4; ++g)
      if (l < F::L3 && 4 * g + hi < PB) buf[at + 4 * g] = f3[s][g];
  }
  md_sync<WPE>();
  // the lane's k in each group, 0 past the box (its factor entries are zero)
  int kc[K4];
#pragma unroll
  for (int kg = 0; kg < K4; ++kg) kc[kg] = 4 * kg + hi < PB ? 4 * kg + hi : 0;
  int at3[S3];  // d0 + Y d1 of the lane's lines
#pragma unroll
  for (int s = 0; s < S3; ++s) at3[s] = at0(s) + lo + hi3[s] * (F::Y - PB);
  // y forward on the lines (c', a)
  md_contract<S3, K4, K4>(
      Af, [&](int s, int kg) { return buf[at3[s] + kc[kg] * F::X]; }, f3);
  md_forward_op<P, ASM>(Se, 0, lane, Af);
  md_sync<WPE>();
#pragma unroll
  for (int s = 0; s < S3; ++s)
#pragma unroll
    for (int g = 0; g < K4; ++g)
      if (at0(s) + lo < F::L3 && 4 * g + hi < PB) buf[at3[s] + (4 * g + hi) * F::X] = f3[s][g];
  md_sync<WPE>();
  // x forward on the lines (c', b'), division, x backward in registers
  md_backward_op<P, ASM>(Se, 0, lane, Ab);
  md_contract<S3, K4, K4>(
      Af,
      [&](int s, int kg) {
        return buf[at0(s) + lo - hi3[s] * PB + hi3[s] * F::X + kc[kg] * F::Y];
      },
      f3);
  double b3[S3][KG], lx[K4];
#pragma unroll
  for (int g = 0; g < K4; ++g) lx[g] = lam[kc[g]];
#pragma unroll
  for (int s = 0; s < S3; ++s) {
    const double lyz = lam[PB + hi3[s]] + lam[2 * PB + at0(s) + lo - hi3[s] * PB];
#pragma unroll
    for (int g = 0; g < K4; ++g) f3[s][g] *= md_inv(lyz + lx[g]);
  }
  md_contract<S3, K4, KG>(Ab, [&](int s, int kg) { return f3[s][kg]; }, b3);
  md_backward_op<P, ASM>(Se, 1, lane, Ab);
  md_sync<WPE>();
#pragma unroll
  for (int s = 0; s < S3; ++s)
#pragma unroll
    for (int g = 0; g < KG; ++g)
      if (at0(s) + lo < F::L3 && 4 * g + hi < NK) buf[at3[s] + (4 * g + hi) * F::X] = b3[s][g];
  md_sync<WPE>();
  // y backward on the lines (c', i)
  double b2[S2][KG];
  md_contract<S2, K4, KG>(
      Ab,
      [&](int s, int kg) {
        return buf[at0(s) + lo - hi3[s] * PB + hi3[s] * F::X + kc[kg] * F::Y];
      },
      b2);
  md_backward_op<P, ASM>(Se, 2, lane, Ab);
  md_sync<WPE>();
#pragma unroll
  for (int s = 0; s < S2; ++s)
#pragma unroll
    for (int g = 0; g < KG; ++g)
      if (at0(s) + lo < F::L2 && 4 * g + hi < NK) buf[at3[s] + (4 * g + hi) * F::X] = b2[s][g];
  md_sync<WPE>();
  // z backward on the lines (i, j): the kept nodes of the element
  double b1[S1][KG];
  md_contract<S1, K4, KG>(
      Ab,
      [&](int s, int kg) {
        const int l = at0(s) + lo, d = l / NK;
        const int j = last(s) < F::L1 ? d : (d < NK ? d : NK - 1);
        return buf[(l - j * NK) * F::Y + j * F::X + kc[kg]];
      },
      b1);
  if constexpr (ASM) {
    double *zb = z + e * PB * PB * PB;
#pragma unroll
    for (int s = 0; s < S1; ++s) {
      const int l = at0(s) + lo;
#pragma unroll
      for (int g = 0; g < KG; ++g)
        if (l < F::L1 && 4 * g + hi < PB) zb[(4 * g + hi) * PB * PB + l] = b1[s][g];
    }
  } else {
    double *ze = z + e * N3;
    double wk[KG];
#pragma unroll
    for (int g = 0; g < KG; ++g) wk[g] = node_w1(4 * g + hi, N, ez, nez, W.bcm, 4);
#pragma unroll
    for (int s = 0; s < S1; ++s) {
      const int l = at0(s) + lo, i = l % N, j = l / N;
      const double wij =
          node_w1(i, N, ex, nex, W.bcm, 0) * node_w1(j, N, ey, ney, W.bcm, 2);
#pragma unroll
      for (int g = 0; g < KG; ++g)
        if (l < F::L1 && 4 * g + hi < N) ze[(4 * g + hi) * N * N + l] = wij * wk[g] * b1[s][g];
    }
  }
}

// Four waves per element up to 640 elements (2.5 waves per SIMD) and from p = 7,
// where an element has enough slots of lines to deal out.  With the assembly, one against
// four: 512 elements p = 7 14.9 / 13.3 us, p = 9 17.3 / 15.4, p = 10 22.6 / 18.7, p =
// 5 9.8 / 10.4; 768 elements p = 7 16.6 / 16.5; 1728 elements p = 9 32.4 / 34.4.
constexpr int kWideP = 7;
constexpr int64_t kWideElements = 640;

template <int P, bool ASM>
void mf64_launch(const Ctx &c, const Level &L, const double *r, const double *rs, double *z,
                 hipStream_t s, int nv) {
  using F = Md<P, ASM>;
  RasGrid W{0};
  for (int f = 0; f < 6; ++f) W.bcm |= (L.bc[f] ? 1 : 0) << f;
  const bool wide = P >= kWideP && (c.fdm_mf64_waves ? c.fdm_mf64_waves == 4 : L.E * nv <= kWideElements);
  const int epb = wide ? F::WAVES / 4 : F::WAVES;
  const dim3 grid((unsigned)((L.E + epb - 1) / epb * nv)), block(64 * F::WAVES);
  constexpr int WPE = P >= kWideP ? 4 : 1;
#define SEM_MF64_LAUNCH(RS, WPE)                                                                   \
  hipLaunchKernelGGL((k_fdm_mf64<P, ASM, RS, WPE>), grid, block, 0, s, L.E, c.nex, c.ney, c.nez, r, \
                     RS ? rs : r, L.S64, L.lam64, W, z, nv)
  if (rs && wide) SEM_MF64_LAUNCH(true, WPE);
  else if (rs) SEM_MF64_LAUNCH(true, 1);
  else if (wide) SEM_MF64_LAUNCH(false, WPE);
  else SEM_MF64_LAUNCH(false, 1);
#undef SEM_MF64_LAUNCH
  SEM_LAUNCH("k_fdm_mf64");
}

}  // namespace

// A wave's reads span two planes, two lines and two elements around its own:
// their bytes must fit one buffer window.  A box floats only when every
// direction has one element and Neumann faces at both ends.  Below p = 4 (RAS:
// p = 3) the box leaves the groups of 16 lines and 4 modes mostly padding, and
// the vector kernel is as fast or faster
// (2e6 nodes with the assembly: RAS at p = 2 90 us there and 103 us here, at
// p = 3 67 and 60; ASM at p = 3 66 and 70, at p = 4 106 and 98).
bool fdm_mf64_supported(const Ctx &c, int p, bool asm_mode) {
  const bool floating = c.nex == 1 && c.ney == 1 && c.nez == 1 && !c.bc[0] && !c.bc[1] &&
                        !c.bc[2] && !c.bc[3] && !c.bc[4] && !c.bc[5];
  const int64_t span = 2 * ((int64_t)c.nex * c.ney + c.nex + 1) + 4;
  return c.fdm_mf64 && p >= (asm_mode ? 4 : 3) && p <= kMaxP && !floating &&
         span * (p + 1) * (p + 1) * (p + 1) * 8 < (int64_t)kWin64;
}

void launch_fdm_mf64(const Ctx &c, const Level &L, const double *r, double *z, bool asm_mode,
                     hipStream_t s, int nv, const double *rs) {
  if (!L.S64 || !L.lam64) fail(SEM_EINVAL, "FDM data of this precision were not built");
#define SEM_MF64_CASE(P)                                              \
  case P:                                                             \
    if (!asm_mode) return mf64_launch<P, false>(c, L, r, rs, z, s, nv); \
    if constexpr (P >= 4) return mf64_launch<P, true>(c, L, r, rs, z, s, nv); \
    break;
  switch (L.p) {
    SEM_MF64_CASE(3)
    SEM_MF64_CASE(4)
    SEM_MF64_CASE(5)
    SEM_MF64_CASE(6)
    SEM_MF64_CASE(7)
    SEM_MF64_CASE(8)
    SEM_MF64_CASE(9)
    SEM_MF64_CASE(10)
    default: break;
  }
#undef SEM_MF64_CASE
  fail(SEM_EUNSUPPORTED, "matrix-core FDM: unsupported degree");
}

}  // namespace sem
