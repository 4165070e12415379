// Bloch sums and Hermitian eigensolves on the fine grid (gfx950).
//
// Electrons: H(k) = sum_R w_R e^{ik.R} H(R) and dH/dk_a = sum_R w_R i R_a
// e^{ik.R} H(R) (Sec. II.B, Wannier interpolation of H); eigenpairs
// H V = V diag(eps); velocities v_n = Re(V^+ dH V)_nn / hbar (Hellmann-Feynman
// form of the velocities of the preprocessing step, Sec. III.A).
// Phonons: D(q) = sum_R w_R Phi(R)/sqrt(M M') e^{iq.R}, (hbar w)^2 = C lambda,
// u_{mu nu} = e_{mu nu} sqrt(C/(2 M_mu hbar w_nu)) (Sec. II.B).
//
// Layout on the chip: a matrix takes NP lanes (its size n rounded up to a power
// of two), one column of A and of V per lane in registers, so a wave holds
// 64 / NP matrices.  The eigensolve is a parallel cyclic Jacobi with
// round-robin pairing: every round applies n/2 disjoint complex rotations at
// once.  A lane rotates its column with its partner's, whose elements come
// over the cross-lane network, and then the rows of its column, which are all
// its own.  Everything stays in FP64.
//
// What bounds it: vector instructions, some 250 FP64 operations and 100
// cross-lane moves to a round of eight 8 x 8 matrices, 7 rounds to a sweep.
// Both tables of a grid, 130^3 with 8 bands and 6 modes: 25 ms; 100^3 with 4
// and 3: 1.3 ms.  With one element per lane, read from LDS with the rows and
// columns it mixes, each lane formed the rotation of its row and column anew
// and the wave waited three times a round: 89 and 4.2 ms.
#include <algorithm>
#include <utility>

#include "dev_util.h"
#include "internal.h"

namespace eph {
namespace {

constexpr int kMaxSweeps = 40;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }

// Partner of index x in round r of the round-robin (circle) schedule of NP
// indices; NP-1 rounds cover every pair once.
template <int NP>
__host__ __device__ constexpr int rr_partner(int x, int r) {
  if (NP == 1) return x;
  constexpr int M = NP > 1 ? NP - 1 : 1;
  const int pos = (x == 0) ? 0 : ((x - 1 - r + 2 * M) % M) + 1;
  const int ppos = NP - 1 - pos;
  return (ppos == 0) ? 0 : ((ppos - 1 + r) % M) + 1;
}

constexpr int pow2_up(int n) { return n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : 8; }

// the value of x in the lane at byte address at (4 times its number)
__device__ __forceinline__ double lane_get(double x, int at) {
  const int lo = __builtin_amdgcn_ds_bpermute(at, __double2loint(x));
  const int hi = __builtin_amdgcn_ds_bpermute(at, __double2hiint(x));
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ double quad_get(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// the value of x in the matrix's lane I
template <int NP, int I>
__device__ __forceinline__ double lane_of(double x, int base4) {
  if constexpr (NP == 4) return quad_get<I * 0x55>(x);
  else return lane_get(x, base4 + 4 * I);
}
// the value of x in the lane of the partner column in round R (at: its address)
template <int NP, int R>
__device__ __forceinline__ double partner_get(double x, int at) {
  if constexpr (NP == 4)
    return quad_get<rr_partner<4>(0, R) | rr_partner<4>(1, R) << 2 | rr_partner<4>(2, R) << 4 | rr_partner<4>(3, R) << 6>(x);
  else
    return lane_get(x, at);
}

// A matrix's lanes: column j, base4 = 4 * (lane of column 0).
struct Cols {
  int j, base4;
};

// the rotation of rows I and rr_partner(I), if I is the smaller
template <int NE, int NP, int R, int I>
__device__ __forceinline__ void rotate_rows(double2 (&A)[NE], const Cols &m, double c, double2 se) {
  constexpr int Q = rr_partner<NP>(I, R);
  if constexpr (I < Q && Q < NE) {
    const double cr = lane_of<NP, I>(c, m.base4);
    const double2 s = make_double2(lane_of<NP, I>(se.x, m.base4), lane_of<NP, I>(se.y, m.base4));
    const double2 bp = A[I], bq = A[Q];
    // rows of J^H: (c, -s e) and (conj(s e), c)
    A[I] = cadd(make_double2(cr * bp.x, cr * bp.y), cmul(make_double2(-s.x, -s.y), bq));
    A[Q] = cadd(make_double2(cr * bq.x, cr * bq.y), cmul(make_double2(s.x, -s.y), bp));
    if (m.j == I) A[Q] = make_double2(0.0, 0.0);  // the annihilated pair
    if (m.j == Q) A[I] = make_double2(0.0, 0.0);
  }
}

template <int NE, int NP, bool VEC, int R, int... I>
__device__ __forceinline__ void jacobi_round(double2 (&A)[NE], double2 (&V)[NE], const Cols &m,
                                             std::integer_sequence<int, I...>) {
  const int j = m.j;
  int pj = j;
  double2 apq = make_double2(0.0, 0.0);
  double dg = 0.0;
#pragma unroll
  for (int x = 0; x < NE; x++) {
    const int px = rr_partner<NP>(x, R);
    if (j == x) {
      dg = A[x].x;
      if (px < NE) {
        pj = px;
        apq = A[px];
      }
    }
  }
  const int at = m.base4 + 4 * pj, up = m.base4 + 4 * max(j, pj);
  const double dgo = lane_get(dg, at);
  apq = make_double2(lane_get(apq.x, up), lane_get(apq.y, up));  // A_pq, p < q, from column q
  double c = 1.0;
  double2 se = make_double2(0.0, 0.0);  // s e^{i phi}: J_pp = J_qq = c, J_pq = se, J_qp = -conj(se)
  const double g = sqrt(apq.x * apq.x + apq.y * apq.y);
  if (pj != j && g != 0.0) {
    const double app = j < pj ? dg : dgo, aqq = j < pj ? dgo : dg;
    const double theta = (aqq - app) / (2.0 * g);
    const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
    c = 1.0 / sqrt(t * t + 1.0);
    const double s = t * c;
    se = make_double2(s * apq.x / g, s * apq.y / g);
  }
  const double2 jp = make_double2(j > pj ? se.x : -se.x, se.y);  // the partner column's factor
#pragma unroll
  for (int i = 0; i < NE; i++) {
    const double2 o = make_double2(partner_get<NP, R>(A[i].x, at), partner_get<NP, R>(A[i].y, at));
    A[i] = cadd(make_double2(A[i].x * c, A[i].y * c), cmul(o, jp));
    if constexpr (VEC) {
      const double2 v = make_double2(partner_get<NP, R>(V[i].x, at), partner_get<NP, R>(V[i].y, at));
      V[i] = cadd(make_double2(V[i].x * c, V[i].y * c), cmul(v, jp));
    }
  }
  (rotate_rows<NE, NP, R, I>(A, m, c, se), ...);
#pragma unroll
  for (int i = 0; i < NE; i++)
    if (j == i) A[i].y = 0.0;
}

template <int NE, int NP, bool VEC, int... R>
__device__ __forceinline__ void jacobi_sweep(double2 (&A)[NE], double2 (&V)[NE], const Cols &m,
                                             std::integer_sequence<int, R...>) {
  (jacobi_round<NE, NP, VEC, R>(A, V, m, std::make_integer_sequence<int, NE>()), ...);
}

// Parallel cyclic Jacobi on the matrices of one wave; lanes of columns past
// NE hold zeros.  On return the diagonal holds the eigenvalues and, with VEC,
// V the eigenvectors.
template <int NE, bool VEC>
__device__ __forceinline__ void jacobi(double2 (&A)[NE], double2 (&V)[NE], const Cols &m, bool live) {
  constexpr int NP = pow2_up(NE);
  if constexpr (VEC)
#pragma unroll
    for (int i = 0; i < NE; i++) V[i] = make_double2(i == m.j ? 1.0 : 0.0, 0.0);
  for (int sweep = 0; sweep < kMaxSweeps; sweep++) {
    double off = 0.0, tot = 0.0;
#pragma unroll
    for (int i = 0; i < NE; i++) {
      const double a2 = A[i].x * A[i].x + A[i].y * A[i].y;
      off += (i != m.j) ? a2 : 0.0;
      tot += a2;
    }
#pragma unroll
    for (int d = 1; d < NP; d <<= 1) {
      off += __shfl_xor(off, d, 64);
      tot += __shfl_xor(tot, d, 64);
    }
    const bool done = (off == 0.0) || (off <= 1e-33 * tot) || !live;
    // matrices settle in runs of 64 / NP^2, so that a point's rotations do not
    // depend on how many matrices share a wave
    constexpr int G = 64 / NP;
    const unsigned long long open = __ballot(!done);
    if (open == 0) break;
    const unsigned long long mine = (G == 64 ? ~0ull : (1ull << G % 64) - 1) << ((threadIdx.x & 63) / G * G % 64);
    if (open & mine) jacobi_sweep<NE, NP, VEC>(A, V, m, std::make_integer_sequence<int, NP - 1>());
  }
}

// Outputs of the eigensolve, shared by both Bloch-sum forms.
struct EigOut {
  int64_t n2;  // points per plane
  const double *mode_mass;
  double cph, omega_cut, vel_unit;
  double *eval;
  double2 *evec;
  double *vel;
  unsigned long long *n_excluded;
};

// kElectrons: energies, eigenvectors, velocities; kPhonons: frequencies and
// mode amplitudes; kEnergies: the electrons' energies alone.
enum { kElectrons = 0, kPhonons = 1, kEnergies = 2 };

// One row block of a derivative matrix per wave, staged for its velocities;
// matrices start 16 bytes apart in the banks.
constexpr int stage_rows(int ne) { return ne < 4 ? ne : 4; }
constexpr int stage_stride(int ne) { return stage_rows(ne) * ne + 1; }
constexpr size_t stage_bytes(int ne) { return sizeof(double2) * (size_t)(64 / pow2_up(ne)) * stage_stride(ne); }

// Eigenvalues sorted ascending, eigenvectors (or mode amplitudes) and
// velocities of grid point kl from the column A of its matrix.  deriv(b, d)
// gives the column of the matrix's derivative along b, lat(b, a) Cartesian
// component a of that direction; stage is the wave's own.
template <int NE, int MODE, class Deriv, class Lat>
__device__ __forceinline__ void eig_store(const EigOut &o, bool live, int64_t kl, double2 (&A)[NE], const Cols &m,
                                          double2 *stage, Deriv deriv, Lat lat) {
  constexpr int NP = pow2_up(NE);
  const int j = m.j;
  double2 V[NE];
  jacobi<NE, MODE != kEnergies>(A, V, m, live);
  double wj = 0.0;
#pragma unroll
  for (int i = 0; i < NE; i++) wj = (i == j) ? A[i].x : wj;
  int rank = 0;
#pragma unroll
  for (int i = 0; i < NE; i++) {
    const double wo = lane_get(wj, m.base4 + 4 * i);
    rank += (wo < wj) || (wo == wj && i < j);
  }
  const bool on = live && j < NE;
  if constexpr (MODE == kPhonons) {
    const double hw = sqrt(o.cph * fmax(wj, 0.0));
    if (on) {
      o.eval[plane_at(kl, rank, NE, o.n2)] = hw;
      if (hw < o.omega_cut) atomicAdd(o.n_excluded, 1ull);
#pragma unroll
      for (int i = 0; i < NE; i++) {
        double2 u = make_double2(0.0, 0.0);
        if (hw >= o.omega_cut) {
          const double f = sqrt(o.cph / (2.0 * o.mode_mass[i] * hw));
          u = make_double2(V[i].x * f, V[i].y * f);
        }
        o.evec[plane_at(kl, rank * NE + i, NE * NE, o.n2)] = u;  // u_{mu nu} at nu n + mu
      }
    }
  } else {
    if (on) {
      o.eval[plane_at(kl, rank, NE, o.n2)] = wj;
      if constexpr (MODE == kElectrons)
#pragma unroll
        for (int i = 0; i < NE; i++) o.evec[plane_at(kl, rank * NE + i, NE * NE, o.n2)] = V[i];
    }
  }
  if constexpr (MODE == kElectrons) {
    // velocities: Re sum_ij conj(V_i) dH_ij V_j of the lane's own column V,
    // dH by blocks of rows through LDS
    constexpr int RB = stage_rows(NE);
    double v0 = 0.0, v1 = 0.0, v2 = 0.0;
    double2 *sm = stage + (m.base4 / 4 / NP) * stage_stride(NE);
#pragma unroll 1
    for (int b = 0; b < 3; b++) {
      double2 d[NE];
      deriv(b, d);
      double u = 0.0;
#pragma unroll
      for (int r = 0; r < NE; r += RB) {
        if (j < NE)
#pragma unroll
          for (int i = 0; i < RB; i++) sm[i * NE + j] = d[r + i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < RB; i++) {
          double yr = 0.0, yi = 0.0;
#pragma unroll
          for (int c = 0; c < NE; c++) {
            const double2 h = sm[i * NE + c];
            cmac<double>(yr, yi, h.x, h.y, V[c].x, V[c].y);
          }
          u = fma(V[r + i].x, yr, u);
          u = fma(V[r + i].y, yi, u);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      v0 = fma(lat(b, 0), u, v0);
      v1 = fma(lat(b, 1), u, v1);
      v2 = fma(lat(b, 2), u, v2);
    }
    if (on) {
      double *vo = o.vel + (kl * NE + rank) * 3;
      vo[0] = v0 * o.vel_unit;
      vo[1] = v1 * o.vel_unit;
      vo[2] = v2 * o.vel_unit;
    }
  }
}

// Direct sum over the R list, a wave per 64 / NP points.  With 3 columns and
// more to a matrix its lanes share the phases (weights in them): they are formed
// together for a run of R vectors, each by one lane, and wait in LDS, while the
// next matrix column loads; with 1 or 2 each lane forms its own, four at a time.
// What bounds it on a small grid is the chain of a pass over the list (four
// passes: H and its derivatives), on a large one the phases and the Jacobi.
// Tables, 87 R vectors each: 4 bands and 3 modes, 16^3: 0.125 ms (0.219 with a
// phase per lane and pass, its remainder of 64-bit integers), 100^3: 4.0 (5.2);
// 8 and 6, 80^3: 9.0 (12.8); 1 and 3, 100^3: 1.5 (1.9), 2.0 with shared phases.
template <int NE, int MODE>
__global__ __launch_bounds__(64) void bloch_eig_kernel(EigOut o, int N, int64_t nk, int nr,
                                                       const int *__restrict__ R, const double *__restrict__ w,
                                                       const double *__restrict__ Rcart,
                                                       const double2 *__restrict__ M,
                                                       const double2 *__restrict__ tab) {
  constexpr int NP = pow2_up(NE), MPW = 64 / NP;
  constexpr bool kShare = NE > 2;
  constexpr int RC = 512 / MPW;  // R vectors to a run
  __shared__ double2 stage[MODE == kElectrons ? stage_bytes(NE) / sizeof(double2) : 1];
  __shared__ double2 sPh[kShare ? RC * MPW : 1];  // [R][point]
  const int lane = threadIdx.x;
  const Cols m{lane % NP, 4 * (lane / NP * NP)};
  const int jc = min(m.j, NE - 1);
  const float inv_n = 1.0f / (float)N;

  const int64_t ngroups = (nk + MPW - 1) / MPW;
  for (int64_t gidx = blockIdx.x; gidx < ngroups; gidx += gridDim.x) {
    const int64_t kl = gidx * MPW + lane / NP;
    const bool live = kl < nk;
    const int64_t kp = min(gidx * MPW + (kShare ? lane % MPW : lane / NP), nk - 1);  // whose phases the lane forms
    const int k1 = (int)(kp % N), k2 = (int)((kp / N) % N), k3 = (int)(kp / ((int64_t)N * N));
    auto phase = [&](int r) __attribute__((always_inline)) {
      // k . R mod N: below 3 N^2 < 2^20, so the float quotient is off by one at most
      const int a = k1 * imod(R[3 * r], N) + k2 * imod(R[3 * r + 1], N) + k3 * imod(R[3 * r + 2], N);
      int s = a - (int)((float)a * inv_n) * N;
      s += (s < 0) ? N : 0;
      s -= (s >= N) ? N : 0;
      const double2 ph = tab[s];
      const double wr = w[r];
      return make_double2(ph.x * wr, ph.y * wr);
    };
    // use(r, phase, the lane's column of the matrix) for every R vector in order
    auto over_list = [&](auto use) __attribute__((always_inline)) {
      double2 col[NE];
      auto load = [&](int r, double2 (&c)[NE]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NE; i++) c[i] = M[(size_t)min(r, nr - 1) * NE * NE + i * NE + jc];
      };
      if constexpr (!kShare) {
#pragma unroll 4
        for (int r = 0; r < nr; r++) {
          load(r, col);
          use(r, phase(r), col);
        }
      } else {
        double2 next[NE];
        load(0, next);
        for (int r0 = 0; r0 < nr; r0 += RC) {
          const int n = min(RC, nr - r0);
          __syncthreads();  // the last run's phases are read
          for (int r = lane / MPW; r < n; r += NP) sPh[r * MPW + lane % MPW] = phase(r0 + r);
          __syncthreads();
          for (int r = 0; r < n; r++) {
#pragma unroll
            for (int i = 0; i < NE; i++) col[i] = next[i];
            load(r0 + r + 1, next);
            use(r0 + r, sPh[r * MPW + lane / NP], col);
          }
        }
      }
    };
    // ---- Bloch sum ----
    double2 A[NE];
#pragma unroll
    for (int i = 0; i < NE; i++) A[i] = make_double2(0.0, 0.0);
    over_list([&](int, double2 ph, const double2 (&col)[NE]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NE; i++) A[i] = cadd(A[i], cmul(ph, col[i]));
    });
    if (m.j >= NE)
#pragma unroll
      for (int i = 0; i < NE; i++) A[i] = make_double2(0.0, 0.0);
    // i R_a times the terms of the sum
    auto deriv = [&](int a, double2 (&d)[NE]) {
#pragma unroll
      for (int i = 0; i < NE; i++) d[i] = make_double2(0.0, 0.0);
      over_list([&](int r, double2 ph, const double2 (&col)[NE]) __attribute__((always_inline)) {
        const double ra = Rcart[3 * r + a];
#pragma unroll
        for (int i = 0; i < NE; i++) {
          const double2 t = cmul(ph, col[i]);
          d[i].x -= ra * t.y;
          d[i].y += ra * t.x;
        }
      });
    };
    eig_store<NE, MODE>(o, live, kl, A, m, stage, deriv, [](int b, int a) { return b == a ? 1.0 : 0.0; });
  }
}

// Separable form of the same Bloch sum for R lists that fill a box
// [lo, lo + nb) (missing vectors are zero in the dense copy Mb, weights
// folded in).  One workgroup per k-line (k2, k3): its threads first sum the
// elements over the (R2, R3) planes for each R1,
//   T0(R1) = sum_{R2,R3} e^{i2pi(k2 R2 + k3 R3)/N} M(R),  T2, T3 the same
//   weighted by R2, R3 (electrons),
// into LDS, then per k1 on the line
//   M(k) = sum_R1 e^{i2pi k1 R1/N} T0(R1),  S1 = sum_R1 R1 e^{..} T0(R1),
//   S2, S3 = sum_R1 e^{..} T2,3(R1),  dM/dk_a = i sum_b L_ba S_b
// (L the lattice vectors as rows), which is the direct sum associated
// differently.
struct BoxArgs {
  int lo[3], nb[3];
  double lat[9];
};

constexpr int kLineWaves = 4;  // most waves per workgroup

template <int NE, int MODE>
__global__ __launch_bounds__(64 * kLineWaves) void bloch_line_kernel(EigOut o, int N, BoxArgs bx,
                                                                     const double2 *__restrict__ Mb,
                                                                     const double2 *__restrict__ tab) {
  constexpr int NP = pow2_up(NE), MPW = 64 / NP, NN = NE * NE;
  extern __shared__ __align__(16) double2 sm[];
  const int n1 = bx.nb[0], n2 = bx.nb[1], n3 = bx.nb[2];
  double2 *sT = sm;                                          // [T0, T2, T3][n1][NN]
  double2 *stage = sm + (MODE == kElectrons ? 3 : 1) * n1 * NN + threadIdx.x / 64 * (int)(stage_bytes(NE) / sizeof(double2));
  const int k2 = (int)(blockIdx.x % N), k3 = (int)(blockIdx.x / N);
  for (int x = threadIdx.x; x < n1 * NN; x += blockDim.x) {
    const double2 *mx = Mb + (size_t)(x / NN) * n2 * n3 * NN + x % NN;
    double2 t0 = make_double2(0.0, 0.0), t2 = t0, t3 = t0;
    int i2 = imod(k2 * bx.lo[1], N);
    const int i3s = imod(k3 * bx.lo[2], N);
    for (int b2 = 0; b2 < n2; b2++) {
      const double r2 = (double)(bx.lo[1] + b2);
      int i23 = i2 + i3s;
      i23 -= (i23 >= N) ? N : 0;
      for (int b3 = 0; b3 < n3; b3++) {
        const double2 t = cmul(tab[i23], mx[((size_t)b2 * n3 + b3) * NN]);
        t0 = cadd(t0, t);
        if constexpr (MODE == kElectrons) {
          const double r3 = (double)(bx.lo[2] + b3);
          t2.x = fma(r2, t.x, t2.x);
          t2.y = fma(r2, t.y, t2.y);
          t3.x = fma(r3, t.x, t3.x);
          t3.y = fma(r3, t.y, t3.y);
        }
        i23 += k3;
        i23 -= (i23 >= N) ? N : 0;
      }
      i2 += k2;
      i2 -= (i2 >= N) ? N : 0;
    }
    sT[x] = t0;
    if constexpr (MODE == kElectrons) {
      sT[n1 * NN + x] = t2;
      sT[2 * n1 * NN + x] = t3;
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const Cols m{lane % NP, 4 * (lane / NP * NP)};
  const int jc = min(m.j, NE - 1);
  // waves take MPW points at a time
  for (int kb = threadIdx.x / 64 * MPW; kb < N; kb += (int)blockDim.x / 64 * MPW) {
    const int k1r = kb + lane / NP;
    const bool live = k1r < N;
    const int k1 = live ? k1r : 0;
    const int i1s = imod(k1 * bx.lo[0], N);
    double2 A[NE];
#pragma unroll
    for (int i = 0; i < NE; i++) A[i] = make_double2(0.0, 0.0);
    int i1 = i1s;
    for (int b1 = 0; b1 < n1; b1++) {
      const double2 ph = tab[i1];
#pragma unroll
      for (int i = 0; i < NE; i++) A[i] = cadd(A[i], cmul(ph, sT[b1 * NN + i * NE + jc]));
      i1 += k1;
      i1 -= (i1 >= N) ? N : 0;
    }
    if (m.j >= NE)
#pragma unroll
      for (int i = 0; i < NE; i++) A[i] = make_double2(0.0, 0.0);
    auto deriv = [&](int b, double2(&d)[NE]) {  // i S_b
#pragma unroll
      for (int i = 0; i < NE; i++) d[i] = make_double2(0.0, 0.0);
      int i1 = i1s;
      for (int b1 = 0; b1 < n1; b1++) {
        double2 ph = tab[i1];
        if (b == 0) {
          const double r1 = (double)(bx.lo[0] + b1);
          ph = make_double2(r1 * ph.x, r1 * ph.y);
        }
#pragma unroll
        for (int i = 0; i < NE; i++) {
          const double2 t = cmul(ph, sT[((b == 0 ? 0 : b) * n1 + b1) * NN + i * NE + jc]);
          d[i].x -= t.y;
          d[i].y += t.x;
        }
        i1 += k1;
        i1 -= (i1 >= N) ? N : 0;
      }
    };
    eig_store<NE, MODE>(o, live, (int64_t)k1 + (int64_t)N * blockIdx.x, A, m, stage, deriv,
                        [&](int b, int a) { return bx.lat[3 * b + a]; });
  }
}

__global__ void phase_table_kernel(int N, double2 *tab) {
  int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < N) {
    double s, c;
    sincospi(2.0 * (double)m / (double)N, &s, &c);
    tab[m] = make_double2(c, s);
  }
}

}  // namespace

hipError_t launch_phase_table(int N, double2 *tab, hipStream_t st) {
  hipLaunchKernelGGL(phase_table_kernel, dim3((N + 255) / 256), dim3(256), 0, st, N, tab);
  return hipGetLastError();
}

#define EPH_BLOCH_DISPATCH(GO) \
  switch (mode) {              \
    case kElectrons:           \
      switch (n) {             \
        GO(1, kElectrons)      \
        GO(2, kElectrons)      \
        GO(4, kElectrons)      \
        GO(8, kElectrons)      \
      }                        \
      break;                   \
    case kPhonons:             \
      switch (n) {             \
        GO(3, kPhonons)        \
        GO(6, kPhonons)        \
      }                        \
      break;                   \
    case kEnergies:            \
      switch (n) {             \
        GO(1, kEnergies)       \
        GO(2, kEnergies)       \
        GO(4, kEnergies)       \
        GO(8, kEnergies)       \
      }                        \
  }

hipError_t launch_bloch_eig(int mode, int n, int N, int64_t n2, int64_t nk, int nr, const int *R,
                            const double *w, const double *Rcart, const double2 *M, const double2 *tab, const double *mode_mass,
                            double cph, double omega_cut, double vel_unit, double *eval, double2 *evec, double *vel,
                            unsigned long long *n_excluded, hipStream_t st) {
  if (nk <= 0) return hipSuccess;
  const EigOut o{n2, mode_mass, cph, omega_cut, vel_unit, eval, evec, vel, n_excluded};
  const int64_t ngroups = (nk * pow2_up(n) + 63) / 64;
  const int grid = (int)(ngroups < 262144 ? ngroups : 262144);
#define EPH_GO(NE, MODE)                                                                                             \
  case NE:                                                                                                           \
    hipLaunchKernelGGL((bloch_eig_kernel<NE, MODE>), dim3(grid), dim3(64), 0, st, o, N, nk, nr, R, w, Rcart, M, tab); \
    return hipGetLastError();
  EPH_BLOCH_DISPATCH(EPH_GO)
#undef EPH_GO
  return hipErrorInvalidValue;
}

hipError_t launch_bloch_lines(int mode, int n, int N, int64_t n2, const int *lo, const int *nb, const double *lattice,
                              const double2 *Mb, const double2 *tab, const double *mode_mass, double cph,
                              double omega_cut, double vel_unit, double *eval, double2 *evec, double *vel,
                              unsigned long long *n_excluded, hipStream_t st) {
  const EigOut o{n2, mode_mass, cph, omega_cut, vel_unit, eval, evec, vel, n_excluded};
  if (nb[0] > kBoxMaxR1) return hipErrorInvalidValue;
  BoxArgs bx;
  for (int a = 0; a < 3; a++) {
    bx.lo[a] = lo[a];
    bx.nb[a] = nb[a];
  }
  for (int a = 0; a < 9; a++) bx.lat[a] = lattice[a];
  const int waves = std::min(kLineWaves, (N * pow2_up(n) + 63) / 64);
  const size_t sh = sizeof(double2) * (mode == kElectrons ? 3 : 1) * nb[0] * n * n +
                    (mode == kElectrons ? waves * stage_bytes(n) : 0);
#define EPH_GO(NE, MODE)                                                                                            \
  case NE: {                                                                                                        \
    auto kern = bloch_line_kernel<NE, MODE>;                                                                        \
    const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh); \
    if (e != hipSuccess) return e;                                                                                  \
    hipLaunchKernelGGL(kern, dim3((unsigned)(N * N)), dim3(64 * waves), sh, st, o, N, bx, Mb, tab);                 \
    return hipGetLastError();                                                                                       \
  }
  EPH_BLOCH_DISPATCH(EPH_GO)
#undef EPH_GO
  return hipErrorInvalidValue;
}
#undef EPH_BLOCH_DISPATCH

}  // namespace eph
