// Internal declarations of the gfx950 EPWI library: context layout, device
// buffers and the host-side launchers of every kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "eph.h"

namespace eph {

// Exact SI 2019 constants (amu: CODATA 2022).
constexpr double kPlanck = 6.62607015e-34;
constexpr double kCharge = 1.602176634e-19;
constexpr double kBoltz = 1.380649e-23;
constexpr double kAmu = 1.66053906892e-27;
constexpr double kPi = 3.14159265358979323846;
constexpr int kMaxLine = EPH_MAX_LINE;

struct Units {
  double hbar_evs;   // hbar in eV s
  double kb_evk;     // k_B in eV/K
  double cph_ev;     // hbar^2/(amu A^2) in eV: (hbar w)^2 = cph * lambda
  double vel_unit;   // (1 eV A)/hbar in m/s
  double rate_pref;  // 2 pi / hbar in 1/(eV s)
};
Units units();

// Makes a device current for the lifetime of the guard and restores the
// caller's current device afterwards.
struct DeviceGuard {
  int prev = -1;
  bool ok = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    ok = hipSetDevice(dev) == hipSuccess;
  }
  ~DeviceGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

// Grow-only device buffer.
struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
  ~DevBuf();
  hipError_t ensure(size_t n);
  template <class T>
  T *as() const { return static_cast<T *>(p); }
};

// Grid tables with several components per point (bands, eigenvector elements,
// modes, mode-matrix elements) are kept by i3 plane, each component of a
// plane contiguous over its N^2 points, so that neighbouring points are read
// together: element (k, c) of nc components is at plane_at(k, c, nc, N^2).
// That is for the wave kernel, whose lanes are neighbours in p and q; the
// workgroup form, whose lanes lie scattered along a line, and the k-batch order
// gather whole points and have them contiguous, k nc + c: one point to a plane
// (Al-like 40^3, Rp box 3^3, FP32: 138.7 ms, 145.3 by plane; k-batch order,
// Si-like 8^3: 394 and 405 ms).
__host__ __device__ inline int64_t plane_at(int64_t k, int c, int nc, int64_t n2) {
  return ((k / n2) * nc + c) * n2 + k % n2;
}

// A launch has less than 2^32 threads along x (HIP refuses some larger sizes and
// wraps others): launchers whose work may pass that go in pieces of this many.
constexpr int64_t kLaunchThreads = (int64_t)1 << 31;

struct RpBox {
  int lo[3];
  int n[3];
  int count() const { return n[0] * n[1] * n[2]; }
};

}  // namespace eph

struct eph_ctx {
  int device = 0;
  std::string err;
  // model
  int nw = 0, na = 0, nm = 0;
  double lattice[9];
  double volume = 0;  // A^3
  std::vector<double> mode_mass;  // [nm]
  int nrh = 0, nrd = 0, nre = 0, nrp = 0;
  eph::RpBox box;
  // device copies of the model
  eph::DevBuf rh, rh_w, rh_cart, ham;   // ham: [nrh][nw*nw] double2
  eph::DevBuf rd, rd_w, dyn;            // dyn: Phi/sqrt(MM') as double2 [nrd][nm*nm]
  // dense boxes of the weighted H(R) and D(R) for the separable Bloch sum
  // (empty when the R list does not fill its box well enough)
  eph::DevBuf hbox, dbox;
  int hbox_lo[3] = {0, 0, 0}, hbox_n[3] = {0, 0, 0}, dbox_lo[3] = {0, 0, 0}, dbox_n[3] = {0, 0, 0};
  eph::DevBuf re;                       // [nre][3] int
  eph::DevBuf wt64;                     // [nre*nw][box*nm*nw] double2 (K-major)
  eph::DevBuf wt32;                     // same in float2 (lazy)
  eph::DevBuf wtbf;                     // bf16 hi/lo split (lazy)
  eph::DevBuf mode_mass_d;              // [nm]
  // per-call workspaces (grow-only)
  eph::DevBuf tab;                      // e^{2 pi i m/N}, [N] double2
  eph::DevBuf eps, evec, vel, om, uu;   // grid tables
  eph::DevBuf evec32, uu32;             // FP32 copies for reduced forms
  eph::DevBuf part;                     // sums of each slab of a launch of several
  eph::DevBuf cnt, offs, scan_tmp, subset;
  eph::DevBuf grp_start, grp_tmp;
  eph::DevBuf line_e, line_key;         // energy-sorted p-lines
  eph::DevBuf xbuf;                     // X_s = Re transform + j rotation
  eph::DevBuf abf;                      // bf16 hi/lo state operand of the BF16x3 Re transform
  eph::DevBuf counters;                 // int64 counters
  eph::DevBuf sig_part;                 // sigma partial sums
  double *scratch = nullptr;            // device address of the static workspace (eph_conductivity_noalloc)
  eph::DevBuf state_cnt;                // per-state int64 counts
  eph::DevBuf stidx;                    // [N^3][nw] state index table (transition rates)
  eph::DevBuf gcur;                     // per-state transition-rate counts / cursors
  eph::DevBuf gslot;                    // the same per slab of a launch
  eph::DevBuf gstage_col, gstage_val;   // staging of spilled transition rates
  eph::DevBuf bte_f;                    // F0, F, F' of the iteration
  eph::DevBuf kb_g;                     // G_q of a q batch (k-batch order)
  eph::DevBuf occ;                      // Fermi and Bose factor tables
  eph::DevBuf rec;                      // FP32 records of the wave kernel
  eph::DevBuf ranges;                   // band energy ranges of its chunks
  // stage timing
  bool profiling = false;
  std::vector<hipEvent_t> ev;  // created on demand, reused across calls
  int64_t launches[2] = {0, 0};
  double stage_ms[5] = {0, 0, 0, 0, 0};
  ~eph_ctx() {
    for (auto &e : ev)
      if (e) (void)hipEventDestroy(e);
  }
};

// Transition rates of the iterative BTE, row by row (CSR): row s holds the
// entries of state s, each a final-state index (into the same state list)
// and one value per temperature.  Kept in device memory, or in pinned host
// memory when it does not fit the device budget (streamed back in batches
// of rows for every iteration).
struct eph_gamma {
  eph_ctx *ctx = nullptr;
  int64_t ns = 0, nnz = 0;
  int nt = 0;
  double temps[EPH_MAX_TEMPS] = {0, 0, 0, 0};
  double mu = 0;
  bool on_host = false;
  std::vector<int64_t> h_row;   // [ns+1] row starts (host copy)
  eph::DevBuf row;              // [ns+1] row starts (device)
  eph::DevBuf col, val;         // device entries: col [nnz] int32, val [nt][nnz] (resident)
  int32_t *h_col = nullptr;     // pinned host entries (spilled)
  double *h_val = nullptr;      // [nt][nnz]
  int64_t stage_nnz = 0;        // entries per staging batch (spilled)
  ~eph_gamma();
};

namespace eph {

// ---- launchers (each returns the launch error) ----
// Bloch sum + Hermitian eigensolve on grid points [0, nk); n2 points per plane
// of the tables (plane_at).
//  mode 0 (electrons): eval (k, n), evec (k, m n + i) = V_im, vel[k][n][3] (m/s)
//  mode 1 (phonons):   eval (k, nu) = hbar w (eV), evec (k, nu n + mu) = u_{mu nu}
//                      (A), zero for hbar w < omega_cut; counts excluded modes
//  mode 2:             mode 0's eval alone
hipError_t launch_bloch_eig(int mode, int n, int N, int64_t n2, int64_t nk, int nr, const int *R,
                            const double *w, const double *Rcart, const double2 *M, const double2 *tab,
                            const double *mode_mass, double cph, double omega_cut, double vel_unit,
                            double *eval, double2 *evec, double *vel, unsigned long long *n_excluded,
                            hipStream_t st);
hipError_t launch_phase_table(int N, double2 *tab, hipStream_t st);
// The same tables for all N^3 grid points from the separable form of the
// Bloch sum: Mb is the dense copy [nb0][nb1][nb2][n][n] of the weighted
// matrices on the box [lo, lo + nb) of R vectors (zero where the list has
// no vector), nb[0] <= kBoxMaxR1; lattice as rows a1, a2, a3 (Angstrom).
constexpr int kBoxMaxR1 = 12;
hipError_t launch_bloch_lines(int mode, int n, int N, int64_t n2, const int *lo, const int *nb, const double *lattice,
                              const double2 *Mb, const double2 *tab, const double *mode_mass, double cph,
                              double omega_cut, double vel_unit, double *eval, double2 *evec, double *vel,
                              unsigned long long *n_excluded, hipStream_t st);

// State selection.  cnt/offs sized nklist+1.
hipError_t launch_count_states(int64_t nklist, const int64_t *klist, int64_t n2, int nw, const double *eps, int blo,
                               int bhi, double wlo, double whi, int64_t *cnt, hipStream_t st);
hipError_t launch_scan(int64_t n, const int64_t *in, int64_t *out_excl, int64_t *tmp, hipStream_t st);
size_t scan_tmp_elems(int64_t n);
hipError_t launch_write_states(int64_t nklist, const int64_t *klist, int64_t n2, int nw, const double *eps,
                               const double *vel, int blo, int bhi, double wlo, double whi,
                               const int64_t *offs, int32_t *sk, int32_t *sn, double *se, double *sv,
                               hipStream_t st);
// Group heads: states of one k-line (same i2,i3), chunks of at most gmax.
hipError_t launch_group_heads(int64_t ns, const int32_t *sk, int N, int gmax, int64_t *flag,
                              hipStream_t st);
hipError_t launch_group_starts(int64_t ns, const int64_t *flag, const int64_t *pos, int64_t *gstart,
                               hipStream_t st);
// Energy-sorted p-lines: for each line (i2,i3), entries key = i1*nw + m sorted by eps.
hipError_t launch_line_sort(int N, int nw, const double *eps, double *line_e, uint16_t *line_key,
                            hipStream_t st);

// Re transform fused with the j->n rotation:
//   X[s][rp][mu][i] = sum_{Re,j} Wt[(Re,j)][(rp,mu,i)] e^{i k_s.Re} V_{j n_s}(k_s)
hipError_t launch_xform64(int64_t ns, const int32_t *sk, const int32_t *sn, int N, int64_t n2, int nw, int nre,
                          const int *re, int ncol, const double2 *wt, const double2 *evec,
                          const double2 *tab, double2 *X, hipStream_t st);
hipError_t launch_xform32(int64_t ns, const int32_t *sk, const int32_t *sn, int N, int64_t n2, int nw, int nre,
                          const int *re, int ncol, const float2 *wt, const double2 *evec,
                          const double2 *tab, float2 *X, hipStream_t st);
hipError_t launch_to_f32(int64_t n, const double2 *in, float2 *out, hipStream_t st);
// bf16 hi/lo split of the g operand in real form (2 * bf16_w_elems bf16 values)
size_t bf16_w_elems(int nre, int nw, int ncol);
// bf16 values per state of one half (hi or lo) of the state-side operand
size_t bf16_a_elems(int nre, int nw);
hipError_t launch_split_bf16(int nre, int nw, int ncol, const double2 *wt, void *out, hipStream_t st);
// abf: workspace of 2 * ns * bf16_a_elems bf16 values (the state operand, hi and lo)
hipError_t launch_xform_bf16x3(int64_t ns, const int32_t *sk, const int32_t *sn, int N, int64_t n2, int nw, int nre,
                               const int *re, int ncol, const void *wbf, void *abf, const double2 *evec,
                               const double2 *tab, float2 *X, hipStream_t st);

// Most final-state lines (p2 of one p3 plane) per batch of the wave kernel:
// the columns of one matrix product.
constexpr int kWaveLines = 16;
// FP32 tables of the wave kernel, one record per gather: of a final state
// (p, m) the eigenvector row, energy and Fermi factors, of a q the mode
// matrix [nu][mu], energies and Bose factors [nu][t]; stored by 16-byte
// chunks (RatesArgs::rec_p, rec_q).
template <int NW, int NT>
struct alignas(16) PRec {
  float2 v[NW];
  double e;
  float f[NT];
};
template <int NM, int NT>
struct alignas(16) QRec {
  float2 u[NM * NM];
  double w[NM];
  float n[NM * NT];
};

struct RatesArgs {
  int N, nw, nm, nt;
  RpBox box;
  double mu, eta, sw, wcut, wmax;
  double temps_kt[EPH_MAX_TEMPS];  // k_B T in eV
  double pref;                     // 2 pi / hbar / N^3
  int64_t ng;                      // groups in this launch
  const int64_t *gstart;           // [ng+1] absolute state indices
  int64_t s_base;                  // state index of X row 0
  const int32_t *sk, *sn;
  // grid tables by plane_at (wave kernel; by point otherwise): energies (k, m), (q, nu) (inf below omega_cut for
  // the wave kernel), eigenvectors (k, m nw + i),
  // mode matrices (q, nu nm + mu)
  const double *eps, *om;
  const double2 *evec, *uu;
  const float2 *evec32, *uu32;
  const double *line_e;
  const uint16_t *line_key;
  const double2 *tab;
  const void *X;                   // [ns][box][nm*nw] double2 or float2
  double *inv_tau;                 // [nt][ns_total]
  int64_t ns_total;
  int64_t *st_counts;              // [ns_total][2]: n_q_valid, n_terms
  unsigned long long *n_kq;
  unsigned long long *n_vertex;
  // wave kernel
  int64_t *kv_counts;              // [ns_total][2]: (k,q) pairs, vertices
  int64_t s_lo, ns_launch;         // states s_lo .. s_lo + ns_launch - 1 of this launch
  const double *occ_f;             // Fermi factors (k, m) and Bose factors (q, nu), 0 below omega_cut: by plane_at
  const double *occ_n;             // for one temperature, else two components of two temperatures each
  const float4 *rec_p, *rec_q;     // FP32 records in place of evec .. occ_n: 16-byte chunk c of PRec (k, m) at
                                   // component m chunks + c, of QRec (q) at component c
  const float2 *band_range;        // [N][plane_groups][nw] lowest and highest energy of each group of 16 p
  int batch_lines, plane_groups;   // p-lines per batch; groups of a p3 plane, a batch's from its first p on
  int slab_planes;                 // q3 planes per workgroup (a slab)
  int slab_lo, slab_hi;            // slabs of this launch, one row of workgroups each
  double *part_tau;                // [slabs][nt][ns_total] sums of each slab of a launch of several, or
                                   // nullptr: one slab, added to inv_tau
  int64_t *part_cnt;               // [slabs][ns_total][4], with part_tau
  // transition rates of the iterative BTE (wave kernel, FP64, count and emit modes)
  const int32_t *stidx;            // [N^3][nw] index of state (k, m) in the list, -1 if none
  int64_t *g_cursor;               // [ns_total] next position of each state (emit)
  int64_t *g_slot;                 // [slabs][ns_total] counts (count mode); offsets of the slabs of a launch
                                   // from g_cursor (emit); nullptr for one slab, which advances g_cursor
  int32_t *g_col;                  // emitted final-state indices, position - g_base
  double *g_val;                   // emitted values [t][g_stride], 1/s
  int64_t g_stride;                // temperature stride of g_val
  int64_t g_base;                  // position of g_col[0] / g_val[0]
};
// rate-kernel modes (wave kernel)
constexpr int kRates = 0, kCount = 1, kEmit = 2;
hipError_t launch_rates(int precision, const RatesArgs &a, hipStream_t st);
// Temperatures per element of the wave kernel's occupation tables: one, or
// two pairs for two to four.
__host__ __device__ inline int occ_stride(int nt) { return nt == 1 ? 1 : EPH_MAX_TEMPS; }
// Wave rate kernel; rates_wave_group gives the states per group that the
// state batches and the transition-rate staging count with (0 when the shape
// is not served and launch_rates must be used).
int rates_wave_group(int nw, int nm, RpBox box, int N, int precision);
hipError_t launch_rates_wave(int precision, const RatesArgs &a, hipStream_t st, int mode = kRates);
// Adds the slabs of a launch (a.part_tau, a.part_cnt) to a.inv_tau and
// a.st_counts in order, and with a.g_slot moves a.g_cursor past them.
hipError_t launch_add_slabs(const RatesArgs &a, hipStream_t st);
// Counts of a counting launch (a.g_slot): total 1 adds them to a.g_cursor,
// 0 turns them into offsets and leaves the sums in the row after the slabs.
hipError_t launch_slab_counts(const RatesArgs &a, int total, hipStream_t st);
// k-batch order of the vertex (k_kbatch.hip): step 1 forms G_q for a batch
// of q, step 2 runs one wave per state over that batch.
struct KBatchArgs {
  int N, nw, nm, nt, nre, nb;
  int64_t q0, ns;
  double eta, sw, wcut, pref;
  const int32_t *sk, *sn;
  const int *re;
  const double *eps, *om;
  const double2 *evec, *tab, *Gq;
  const double *occ_f, *occ_n;
  double *inv_tau;
  int64_t *st_counts;
};
hipError_t launch_kbatch_step1(int64_t q0, int nb, int N, RpBox box, int nre, int nm, int nw, int ncol,
                               const double2 *wt, const double2 *uu, const double2 *tab, double2 *Gq, hipStream_t st);
hipError_t launch_kbatch_step2(const KBatchArgs &a, hipStream_t st);
// Occupation tables, for every element of eps and om (zeros past nt):
// f = 1/(exp((eps-mu)/kT_t)+1), N = 1/expm1(hbar w/kT_t) (0 when hbar w < wcut).
// rows true: EPH_MAX_TEMPS values per element (k-batch kernels); else as the
// wave kernel reads them.
hipError_t launch_occupations(int N, int nw, int nm, const double *eps, const double *om, double mu, int nt,
                              const double *kts_host, double wcut, bool rows, double *occ_f, double *occ_n,
                              hipStream_t st);

// sigma partial sums per block, then out[T*9 + ab] = pref * sum of partials
// (partials: [nblk][EPH_MAX_TEMPS*9], out: [EPH_MAX_TEMPS*9], kts: device [nt]).
// moments 0 .. n_orders - 1 (1 or 3) weight each state by (eps - mu)^n (n = 0:
// sigma), into out[n_orders][EPH_MAX_TEMPS * 9] (partials [n_orders][nblk] of
// the same).  F (optional, [nt][ns][3], one moment) replaces v_b tau by the
// mean free path F_b.
hipError_t launch_sigma(int64_t ns, const double *e, const double *v, const double *inv_tau, double mu,
                        int nt, const double *kts_host, double pref, double *partials, int nblk, double *out,
                        hipStream_t st, int n_orders, const double *F = nullptr);
// iterative BTE (k_bte.hip)
hipError_t launch_state_index(int64_t nq, int nw, int64_t ns, const int32_t *sk, const int32_t *sn, int32_t *stidx,
                              hipStream_t st);
hipError_t launch_f0(int64_t ns, int nt, const double *vel, const double *inv_tau, double *F0, hipStream_t st);
hipError_t launch_bte_step(int64_t r0, int64_t r1, const int64_t *row_start, int64_t base, const int32_t *col,
                           const double *val, const double *inv_tau, const double *F0, const double *Fin, double *Fout,
                           hipStream_t st);
hipError_t launch_check_rows(int64_t ns, const int64_t *cursor, const int64_t *row_start, unsigned long long *bad,
                             hipStream_t st);
// out[t] = pref * sum_{k, blo <= n <= bhi} f(eps_nk) (partials: [nblk][EPH_MAX_TEMPS])
hipError_t launch_density(int N, int nw, const double *eps, int blo, int bhi, double mu, int nt,
                          const double *kts, double pref, double *partials, int nblk, double *out, hipStream_t st);
// Wave kernel tables: the energy range of every band in every group of 16 p
// (rounded outwards), and the FP32 records (factors as launch_occupations).
int wave_batch_lines(int N);
int wave_plane_groups(int N);
int wave_slab_planes(int N, int64_t ns, bool fp64);  // q3 planes per workgroup
hipError_t launch_band_ranges(int N, int nw, const double *eps, float2 *out, hipStream_t st);
size_t wave_rec_bytes(int nw, int nm, int nt, int64_t nq, size_t *q_offset);
hipError_t launch_wave_records(int N, int nw, int nm, const double *eps, const double *om, const double2 *evec,
                               const double2 *uu, double mu, int nt, const double *kts_host, double wcut, void *out,
                               hipStream_t st);
int rates_group_max(int nw, int nm);
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st);
// also sets the elements below cut to +inf
hipError_t launch_max_nonneg(int64_t n, double *x, double cut, unsigned long long *out, hipStream_t st);
// out[1..3] += sum n_q_valid, sum n_terms, #(inv_tau0 == 0); with kv_counts
// also out[0] += (k,q) pairs and out[4] += vertices
hipError_t launch_summarize(int64_t ns, const int64_t *st_counts, const int64_t *kv_counts, const double *inv_tau0,
                            unsigned long long *out, hipStream_t st);
size_t rates_smem_bytes(int precision, int N, int nw, int nm, RpBox box);

}  // namespace eph
