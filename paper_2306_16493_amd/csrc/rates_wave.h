#pragma once
// SERTA scattering rates (gfx950): the kernel template.  Instantiated per
// (precision, phonon modes, mode) in k_rates_wave_<p><nm>.hip and dispatched
// by k_rates_wave.hip.
//
// Same arithmetic as the general form (separable Rp box: Y per q3, Z per
// q-line, G per q; vertex contracted onto the final band m first, then onto
// the modes; sieve, occupations, Gaussian delta; Sec. II.B/II.C/III.A/III.C).
// One workgroup takes one initial state s = (n, k) and one q3 plane
// (several on small grids), and goes through the final states p = k + q of a
// plane in batches of p-lines:
//   * Y_s(p1,p2; q3) is formed once per plane, straight into the registers of
//     a matrix-core operand, its (p1, channel) rows spread over the waves;
//   * Z_s(p1; q2,q3) of a batch of lines is one matrix product per 16 lines
//     (16x16x4 MFMA, rows (p1, channel), inner index (p2, re/im), columns the
//     lines) into LDS, where all waves read it;
//   * a table of the lowest and highest energy of every band in each group of
//     16 p says which (group, band) can reach the state's energy (about one in
//     ten for a metal with well separated bands); those are listed and sieved
//     exactly in FP64, four to a pass; the compares go into wave masks, which
//     the scalar unit joins and counts, and the (p, m) with a kept term go to
//     the wave's queue;
//   * the queues of the waves are then evaluated as one list, one vertex per
//     lane, whole passes dealt out to the waves, while the waves with fewer
//     passes take more of the next batch's sieve.
// Fermi and Bose factors come from per-call grid tables, so a vertex pays one
// exp per kept term (the delta) and no other transcendental.  The phase of
// the box corner, e^{i q.lo}, is common to all terms of a vertex and leaves
// |g|^2 alone, so the three sums run over p = 0 .. NB-1, the last one by
// Horner's rule.  The lists, their order and the sums over lanes, waves and
// planes are fixed, so results are bit-reproducible.
//
// What bounds it.  Al-like model (4 bands, 3 modes, box 6^3), 71^3, 3
// temperatures, FP32: 328 ms for 1.2e10 vertices, about 172 ms of it the
// vertices (535 vector instructions to a pass of 64), 85 the sieve, 27 Z, 18
// the reading of X; vector instructions issue in nine cycles of ten.  One wave per
// state and line, each with its own Z by vector operations, took 648 ms; 128
// threads per workgroup leave fewer waves waiting at a barrier than 256.  The
// tables are stored by plane and component so that the lanes' reads,
// neighbours in p or q, run along lines: an array of records, one per gather,
// made the L1 the bound (160^3, FP32, 1 temperature: 173 ms against 101).
// FP64, 100^3, 4 % of the states: 164 ms, 102 of it the
// vertices, whose gathers, 370 bytes each, come from the L2s at 11 TB/s.
#include <cstddef>
#include <type_traits>

#include "dev_util.h"
#include "internal.h"

namespace eph {
namespace wave {

// One 16 x 16 x 4 matrix product.  Lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; it holds column l % 16 of D and, counting the rows of A
// by row_of(l % 16), rows 4 (l / 16) .. 4 (l / 16) + 3.
template <class T>
struct Mfma;
template <>
struct Mfma<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int row_of(int i) { return i; }
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  // the FP64 product leaves row l / 16 + 4 r in register r
  static __device__ __forceinline__ int row_of(int i) { return 4 * (i & 3) + (i >> 2); }
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// Load at a 32-bit byte offset from a wave-uniform base (one plane of a table
// is below 4 GB), which needs no 64-bit address arithmetic per lane.
template <class U>
__device__ __forceinline__ U at_offset(const U *base, uint32_t bytes) {
  return *reinterpret_cast<const U *>(reinterpret_cast<const char *>(base) + bytes);
}
// x + d brought into [0, N) for x + d in [-N, 2 N): the unsigned wrap of the
// other candidate is the larger one
__device__ __forceinline__ uint32_t wrap_up(uint32_t x, uint32_t N) { return min(x, x + N); }    // x in [-N, N)
__device__ __forceinline__ uint32_t wrap_down(uint32_t x, uint32_t N) { return min(x, x - N); }  // x in [0, 2 N)
__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// (a mod N) for 0 <= a < 2^14, N <= 512, inv_n the float nearest 1/N: the
// quotient of a + 1/2 is at least 1/(2 N) from a whole number, the float
// product within 2^-9 / N of it, so the truncation is exact
__device__ __forceinline__ uint32_t mod_small(uint32_t a, uint32_t N, float inv_n) {
  return a - __umul24((uint32_t)(((float)a + 0.5f) * inv_n), N);
}
// the value of x in one lane, as a wave-uniform value
__device__ __forceinline__ double lane_value(double x, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane), hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
  return __hiloint2double(hi, lo);
}

template <class T, int NW, int NM, int NB>
struct WaveLayout {
  using C2 = typename V2<T>::t;
  static constexpr int C = NW * NM;
  static constexpr int ROWS = NB * C;               // (p1, channel) rows of Y and Z
  static constexpr int MT = (ROWS + 15) / 16;       // 16-row tiles
  static constexpr int KS = (2 * NB + 3) / 4;       // 4-deep steps over (p2, re/im)
  // Waves per workgroup.  48 channels: each wave's share of Y has to fit its
  // registers beside a vertex (Si-like 130^3, FP64: 95.8 ms with 8, 158 with 4;
  // FP32: 42.5 with 4, 74.5 with 2, 64.8 with 8).  24 channels: 4 are from 4 %
  // faster to 10 % slower than 2 (8 bands with 3 modes and 4 with 6, box 4^3,
  // 30^3 and 60^3, both precisions).
  static constexpr int WPB = (C >= 48 && sizeof(T) == 8) ? 8 : C >= 48 ? 4 : 2;
  static constexpr int TPW = (MT + WPB - 1) / WPB;  // tiles per wave
  // most lines per batch: the matrix product's columns (32 lines with 4 waves
  // to a workgroup took 443 ms for 421 at Al-like 71^3, FP32)
  static constexpr int NL = kWaveLines;
  // one line's Z, padded by 16 bytes so that neighbouring lines start in
  // different LDS banks
  static constexpr int ZB = ROWS + (int)(16 / sizeof(C2));
  // sieve passes (four entries each) whose table entries are loaded together:
  // as many as the registers hold (Al-like 71^3, FP32, half of the states: 157
  // ms with 3, 160 with 2 or 4)
  static constexpr int SG = NM == 3 ? 3 : 2;
  // Planes of Y formed from one reading of X, where the LDS for the waiting
  // ones costs no workgroup per CU.  The rows of X in flight (20 KB each in
  // FP32) do not fit the L2s, and reading one for every plane took 85 of 387
  // ms (Al-like 71^3): 332 with two planes, 388 with three.  FP64: 2.33 ms
  // with one, 3.12 with two at 24^3; with 48 channels 27.3 and 25.9 ms
  // (Si-like 48^3); FP32 with 48 channels 11.5 and 15.8.
  static constexpr int YP = (sizeof(T) == 4 ? NM == 3 : C >= 48) ? 2 : 1;
  // queue entries per wave and round (a sieve pass adds 64 at most): smaller
  // ones cut rounds short, larger ones cost workgroups (Al-like 71^3, FP32:
  // 359 ms with 384, 332 with 512, 345 with 640)
  static constexpr int QC = 512;
  __host__ __device__ static size_t tab_bytes(int N) { return sizeof(C2) * 2 * (size_t)((N + 1) & ~1); }
  static constexpr size_t z_bytes = sizeof(C2) * (size_t)NL * ZB;
  static constexpr size_t q_bytes = 2 * 2 * (size_t)WPB * QC;                      // two rounds of 16-bit entries
  static constexpr size_t rank_bytes = q_bytes;                                     // emit mode
  static constexpr int LC = 128;                    // (group, band) list entries per wave
  static constexpr size_t misc_bytes = 8 * (size_t)WPB * 8 + 2 * 4 * (size_t)WPB * 4 + 2 * (size_t)WPB * LC;
  static constexpr size_t y_bytes = sizeof(T) * (size_t)(YP - 1) * TPW * KS * 64 * WPB;
  __host__ __device__ static size_t total(int N, int mode, int slab_planes) {
    return misc_bytes + (mode == kCount ? 0 : q_bytes + tab_bytes(N) + z_bytes + (slab_planes > 1 ? y_bytes : 0)) +
           (mode == kEmit ? rank_bytes : 0);
  }
};

// Waves per SIMD the register allocation targets, as timed: FP64 with 3 modes
// 244 ms with 3, 269 with 2 (Al-like, 100^3); FP32 with 6 modes 63 ms with 3, 94
// with 4, 77 with 2 (Si-like, 130^3).  Some instances spill at that: FP32 with 6
// modes 20 to 248 bytes a lane (8 bands, box 6^3, one temperature: 116), with 8
// bands and 3 modes up to 92 in FP32 and 88 in FP64, with 4 and 3 at several
// temperatures 16 in FP32.
template <class T, int NW, int NM>
__host__ __device__ constexpr int waves_per_eu() {
  return sizeof(T) == 4 ? (NM == 6 ? 3 : 4) : (NW * NM >= 48 ? 2 : 3);
}

// MODE: kRates computes 1/tau; kCount only counts, per state, the transition
// rates to final states in the state list (no transforms, no vertices);
// kEmit computes 1/tau and also writes those transition rates (the summed
// terms of each (state, q, m) vertex) from the state's cursor on.
// NT: temperatures per row of the occupation tables (1, or 4 for 2..4).
template <class T, int NW, int NM, int NB, int NT, int MODE>
__global__ __launch_bounds__((WaveLayout<T, NW, NM, NB>::WPB * 64))
__attribute__((amdgpu_waves_per_eu(waves_per_eu<T, NW, NM>())))
void rates_wave_kernel(RatesArgs a) {
  using LY = WaveLayout<T, NW, NM, NB>;
  using C2 = typename V2<T>::t;
  using MM = Mfma<T>;
  using Acc = typename MM::acc;
  // modes of a vertex in flight: all, but for 6 in FP64, whose mode matrices
  // would not fit the registers beside the band row
  constexpr int MU = (sizeof(T) == 8 && NM == 6) ? 2 : NM;
  using PR = PRec<NW, NT>;
  using QR = QRec<NM, NT>;
  constexpr int kPC = sizeof(PR) / 16, kQC = sizeof(QR) / 16;          // chunks of the FP32 records
  constexpr int kPE = offsetof(PR, e) / 4, kPF = offsetof(PR, f) / 4;  // floats before their members
  constexpr int kQW = offsetof(QR, w) / 4, kQN = offsetof(QR, n) / 4;
  constexpr int C = LY::C, WPB = LY::WPB, TPW = LY::TPW, KS = LY::KS, QC = LY::QC, YP = LY::YP;
  extern __shared__ __align__(16) unsigned char smem[];
  const int N = a.N;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // XCD-aware order: consecutive block indices go round-robin to the 8 XCDs,
  // so give each XCD a contiguous range of states (neighbours in k share
  // their final-state plane).
  const int64_t per_xcd = (a.ns_launch + 7) / 8;
  const int64_t blk = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (blk >= a.ns_launch) return;  // workgroup-uniform
  const int64_t s = a.s_lo + blk;
  const int slot = blockIdx.y, slab = a.slab_lo + slot;  // planes slab_planes * slab ..

  double *sRed = reinterpret_cast<double *>(smem);                // [WPB][8] reductions
  int *sCnt = reinterpret_cast<int *>(smem + 8 * WPB * 8);        // [2][WPB][4]: queue length, listed entries, more to come
  uint16_t *sL = reinterpret_cast<uint16_t *>(smem + 8 * WPB * 8 + 2 * 4 * WPB * 4) + wave * LY::LC;  // the wave's list
  unsigned char *rest = smem + LY::misc_bytes;
  uint16_t *sQ = reinterpret_cast<uint16_t *>(rest);              // [2][WPB][QC] vertices: NW (p in the batch) + m
  C2 *sTab = reinterpret_cast<C2 *>(rest + LY::q_bytes);          // [2][N]: f = e^{2 pi i m/N}, then i f
  C2 *sZ = reinterpret_cast<C2 *>(rest + LY::q_bytes + LY::tab_bytes(N));  // [NL][ZB]: [p1][mu][i] + pad
  uint16_t *sRank = reinterpret_cast<uint16_t *>(rest + LY::q_bytes + LY::tab_bytes(N) + LY::z_bytes);  // as sQ
  // [YP - 1][tile][step][thread] (slabs of more than one plane)
  [[maybe_unused]] T *sY = reinterpret_cast<T *>(rest + LY::q_bytes + LY::tab_bytes(N) + LY::z_bytes +
                                                 (MODE == kEmit ? LY::rank_bytes : 0));

  if constexpr (MODE != kCount) {
    for (int t = threadIdx.x; t < N; t += WPB * 64) {
      const T c = (T)a.tab[t].x, sn = (T)a.tab[t].y;
      sTab[t] = mk<T>(c, sn);
      sTab[N + t] = mk<T>(-sn, c);
    }
    __syncthreads();
  }

  const int k = a.sk[s], n = a.sn[s];
  const int k1 = k % N, k2 = (k / N) % N, k3 = k / (N * N);
  const int64_t n2 = (int64_t)N * N;
  const double e_k = a.eps[plane_at(k, lane % NW, NW, n2)];  // band energies at k
  const double es = lane_value(e_k, n);
  // the first state of a k point also looks for the other states' terms, so
  // that every (k, q) pair is counted once; the states of a k point are
  // consecutive bands
  const bool count_kq = s == 0 || a.sk[s - 1] != k;
  int nsh = 0;
  if (MODE != kCount && count_kq)
    while (nsh < NW - 1 && s + 1 + nsh < a.ns_total && a.sk[s + 1 + nsh] == k) nsh++;
  const double cut = a.sw * a.eta;
  // a band beyond the reach of these states' energies keeps no term (the
  // margin covers the rounding here and of the exact test)
  const double reach = (a.wmax + cut) * (1.0 + 1e-12);
  const double e_top = lane_value(e_k, n + nsh);
  const float win_lo = __double2float_rd(es - reach - 1e-12 * fabs(es)),
              win_hi = __double2float_ru(e_top + reach + 1e-12 * fabs(e_top));
  const double inv_eta = 1.0 / a.eta;
  const float ex2 = (float)(1.2011224087864498 * inv_eta);  // sqrt(log2 e) / eta: exp(-(x/eta)^2) = 2^-(ex2 x)^2
  const double pref = a.pref / (1.7724538509055160273 * a.eta);
  const float inv_n = 1.0f / (float)N;

  double acc[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) acc[t] = 0.0;
  int n_dup = 0, n_kq = 0, n_v = 0;  // wave-uniform counts; n_dup: vertices at a q already counted
  int64_t n_t = 0;
  int64_t gpos = 0;                // next transition rate of the state
  if constexpr (MODE == kEmit) gpos = a.g_cursor[s] + (a.g_slot ? a.g_slot[slot * a.ns_total + s] : 0) - a.g_base;

  const int nlb = a.batch_lines, nbatch = (N + nlb - 1) / nlb;
  const int gb_full = (nlb * N + 15) >> 4;  // groups of 16 p of a full batch
  constexpr int CG = 64 / NW;               // groups per look at the band ranges
  const int li = lane & 15, lg = lane >> 4;
  const int q3_end = min(N, (slab + 1) * a.slab_planes);
  // modes below the frequency cut have w = inf in om, which keeps no term
#pragma unroll 1
  for (int q3 = slab * a.slab_planes; q3 < q3_end; q3++) {
  const int p3 = (k3 + q3 >= N) ? k3 + q3 - N : k3 + q3;
  // the planes of the tables that this workgroup reads
  const double *eps_p = a.eps + (int64_t)p3 * NW * n2, *om_q = a.om + (int64_t)q3 * NM * n2;
  const float2 *mm_p = a.band_range + (int64_t)a.plane_groups * NW * p3;

  // ---- the sieve: this wave's groups of 16 p, sv_c .. sv_end - 1 of a batch ----
  int sv_p0 = 0, sv_ne = 0;                // first p and number of p of the batch
  int sv_mm = 0, sv_c = 0, sv_end = 0;     // its first group in the band-range table; the wave's next and last group
  float2 range = make_float2(0.f, 0.f);    // band ranges of the groups from sv_c on, loaded ahead
  int l_pos = 0, l_cnt = 0;                // the list's first entry and length
  uint32_t hit_s = 0, hit_k = 0;           // kept p of the last entry's group, of the state and of its k point
  auto load_ranges = [&]() __attribute__((always_inline)) {
    if (sv_c < sv_end) range = mm_p[(sv_mm + min(sv_c + lane / NW, sv_end - 1)) * NW + lane % NW];
  };
  auto start_batch = [&](int b, int c0, int c1) __attribute__((always_inline)) {
    sv_p0 = b * nlb;
    sv_ne = min(nlb, N - sv_p0) * N;
    sv_mm = b * gb_full;
    sv_c = c0;
    sv_end = c1;
    l_cnt = 0;
    load_ranges();
  };
  // sieve until the queue of round parity `par` may be full or the range is done
  auto sieve = [&](int par) __attribute__((always_inline)) {
    constexpr int SG = LY::SG;
    int cnt = 0, listed = 0, more = 0;
    uint16_t *q = sQ + (par * WPB + wave) * QC;
    const double *eps_b = eps_p + sv_p0 * N;
    for (;;) {
      // list the (group, band) pairs within reach: group << 3 | band, and a
      // mark on those whose predecessor is the same group
      while (l_cnt < 4 * SG && sv_c < sv_end) {
        const bool on = (range.x <= win_hi) & (range.y >= win_lo) & (sv_c + lane / NW < sv_end);
        const unsigned long long mask = __ballot(on);
        const uint32_t lower = (uint32_t)(mask >> (lane & ~(NW - 1))) & ((1u << (lane % NW)) - 1u);
        if (on)
          sL[(l_pos + l_cnt + lanes_below(mask)) & (LY::LC - 1)] =
              (uint16_t)((sv_c + lane / NW) << 3 | lane % NW | (lower ? 0x8000 : 0));
        l_cnt += __popcll(mask);
        sv_c += CG;
        load_ranges();
      }
      if (l_cnt == 0) break;
      if (cnt > QC - 64 * SG) {
        more = 1;
        break;
      }
      __builtin_amdgcn_wave_barrier();
      // the next passes of four entries, 16 lanes each, their table entries
      // in one go; lanes of no entry or past the end read in bounds and are
      // masked
      uint32_t ee[SG], mm[SG];
      unsigned long long valid[SG], again[SG];
      double ep[SG], om[SG][NM];
#pragma unroll
      for (int j = 0; j < SG; j++) {
        const uint32_t i = 4 * j + lg;
        const uint32_t code = i < (uint32_t)l_cnt ? sL[(l_pos + i) & (LY::LC - 1)] : 0x7fffu;
        const uint32_t e = (code >> 3 & 0xfffu) * 16u + li;
        mm[j] = code & (NW - 1);
        valid[j] = __ballot(e < (uint32_t)sv_ne);
        again[j] = __ballot(code >> 15);
        ee[j] = min(e, (uint32_t)(sv_ne - 1));
        const uint32_t l = (uint32_t)(((float)ee[j] + 0.5f) * inv_n);
        const uint32_t p1 = ee[j] - __umul24(l, N);
        const uint32_t q1 = wrap_up(p1 - k1, N), q2 = wrap_up(sv_p0 + l - k2, N);
        const uint32_t qoff = (__umul24(q2, N) + q1) * 8u;
        ep[j] = at_offset(eps_b, (__umul24(mm[j], (uint32_t)n2) + ee[j]) * 8u);
#pragma unroll
        for (int nu = 0; nu < NM; nu++) om[j][nu] = at_offset(om_q + nu * n2, qoff);
      }
#pragma unroll
      for (int j = 0; j < SG; j++) {
        if (4 * j >= l_cnt) break;  // wave-uniform
        // a term (nu, +-) is kept when |d +- w| <= cut with d = es - ep: the
        // nearer of the two has |  |d| - w  |
        const double d = fabs(es - ep[j]);
        unsigned long long any = 0;
#pragma unroll
        for (int nu = 0; nu < NM; nu++) any |= __ballot(fabs(d - om[j][nu]) <= cut);
        any &= valid[j];
        unsigned long long any_k = any;
        if (nsh > 0) {  // the other states at this k point
          for (int i = 0; i < nsh; i++) {
            const double d2 = fabs(lane_value(e_k, n + 1 + i) - ep[j]);
#pragma unroll
            for (int nu = 0; nu < NM; nu++) any_k |= __ballot(fabs(d2 - om[j][nu]) <= cut) & valid[j];
          }
          n_kq += __popcll(any_k);
        }
        // a p kept for several bands is one q
        if (again[j]) {
#pragma unroll
          for (int g = 0; g < 4; g++) {
            const uint32_t h = (uint32_t)(any >> 16 * g) & 0xffffu, hk = (uint32_t)(any_k >> 16 * g) & 0xffffu;
            const bool same = (again[j] >> 16 * g) & 1ull;
            n_dup += same ? __popc(h & hit_s) : 0;
            if (nsh > 0) n_kq -= same ? __popc(hk & hit_k) : 0;
            hit_s = h | (same ? hit_s : 0u);
            hit_k = hk | (same ? hit_k : 0u);
          }
        } else {
          hit_s = (uint32_t)(any >> 48);
          hit_k = (uint32_t)(any_k >> 48);
        }
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(any);
        const uint32_t at = cnt + lanes_below(any);
        if constexpr (MODE == kRates) {
          if (mine) q[at] = (uint16_t)(ee[j] * NW + mm[j]);
        } else {
          const bool in_list = mine && at_offset(a.stidx + (p3 * n2 + sv_p0 * N) * NW, (ee[j] * NW + mm[j]) * 4u) >= 0;
          const unsigned long long lm = __ballot(in_list);
          if constexpr (MODE == kEmit) {
            if (mine) {
              q[at] = (uint16_t)(ee[j] * NW + mm[j]);
              // rank among the wave's listed entries of the round, or none
              sRank[(par * WPB + wave) * QC + at] = in_list ? (uint16_t)(listed + lanes_below(lm)) : (uint16_t)0xffff;
            }
          }
          listed += __popcll(lm);
        }
        if constexpr (MODE != kCount) cnt += __popcll(any);
      }
      const int done = min(l_cnt, 4 * SG);
      l_pos += done;
      l_cnt -= done;
    }
    if constexpr (MODE == kCount) {
      n_v += listed;
    } else {
      n_v += cnt;
      if (lane == 0) {
        int *o = sCnt + (par * WPB + wave) * 4;
        o[0] = cnt;
        o[1] = listed;
        o[2] = more;
      }
    }
  };

  if constexpr (MODE == kCount) {
    for (int b = 0; b < nbatch; b++) {
      const int nc = (min(nlb, N - b * nlb) * N + 15) >> 4;
      start_batch(b, nc * wave / WPB, nc * (wave + 1) / WPB);
      sieve(0);
    }
  } else {
    int b = 0, rot = (int)(s & (WPB - 1));
    const int nc0 = (min(nlb, N) * N + 15) >> 4;
    start_batch(0, nc0 * wave / WPB, nc0 * (wave + 1) / WPB);
    // ---- Y_s(p1, p2; q3) as the A operand: lane (i, g) of tile t and step ks
    //      holds row 16 t + row_of(i) = (p1, channel), inner index 4 ks + g =
    //      (p2, re/im).  Rows past the last repeat it (their products are not
    //      kept), so that a tile's loads go out together.  One reading of X
    //      serves YP planes; the later ones wait in the lane's own LDS words. ----
    static_assert(NB % 2 == 0, "whole steps over (p2, re/im)");
    T ya[TPW][KS];
    const int yj = YP == 1 || a.slab_planes == 1 ? 0 : (q3 - slab * a.slab_planes) % YP;
    if (yj == 0) {
      int64_t x0 = (s - a.s_base) * (int64_t)(NB * NB * NB * C);
      asm volatile("" : "+s"(x0));  // read again, not kept over the loop: the row would fill the registers
      const C2 *X = reinterpret_cast<const C2 *>(a.X) + x0;
      C2 ph3[YP][NB];  // Re(f x) = (f.x, -f.y) . x, Im(f x) = (f.y, f.x) . x
#pragma unroll
      for (int j = 0; j < YP; j++) {
        const int qj = min(q3 + j, N - 1);
        int i3 = 0;
#pragma unroll
        for (int p = 0; p < NB; p++) {
          const C2 f = sTab[((lg & 1) ? N : 0) + i3];
          ph3[j][p] = (lg & 1) ? mk<T>(-f.x, f.y) : mk<T>(f.x, -f.y);
          i3 += qj;
          i3 -= (i3 >= N) ? N : 0;
        }
      }
#pragma unroll
      for (int i = 0; i < TPW; i++) {
        int lo = lane;
        asm volatile("" : "+v"(lo));  // the offsets are not kept over the planes
        const int row = min(16 * (wave + WPB * i) + MM::row_of(lo & 15), LY::ROWS - 1);
        const int p1 = row / C, c = row - p1 * C;
        const uint32_t off0 = (uint32_t)(((p1 * NB + (lo >> 5)) * NB) * C + c) * (uint32_t)sizeof(C2);
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
          const uint32_t off = off0 + ks * (uint32_t)(2 * NB * C * sizeof(C2));
          T y[YP];
#pragma unroll
          for (int j = 0; j < YP; j++) y[j] = 0;
#pragma unroll
          for (int p = 0; p < NB; p++) {
            const C2 v = at_offset(X + p * C, off);
#pragma unroll
            for (int j = 0; j < YP; j++) {
              y[j] = fma(ph3[j][p].x, v.x, y[j]);
              y[j] = fma(ph3[j][p].y, v.y, y[j]);
            }
          }
          if constexpr (sizeof(T) == 8) asm volatile("" : "+v"(y[0]));
          ya[i][ks] = y[0];
          if (YP > 1 && a.slab_planes > 1)
#pragma unroll
            for (int j = 1; j < YP; j++) sY[(((j - 1) * TPW + i) * KS + ks) * (64 * WPB) + threadIdx.x] = y[j];
        }
        // the loads in flight fit the registers: one tile's, in FP64 one step's
        if constexpr (sizeof(T) == 4) asm volatile("" : "+v"(ya[i][0]), "+v"(ya[i][KS - 1]));
      }
    } else {
#pragma unroll
      for (int i = 0; i < TPW; i++)
#pragma unroll
        for (int ks = 0; ks < KS; ks++) ya[i][ks] = sY[(((yj - 1) * TPW + i) * KS + ks) * (64 * WPB) + threadIdx.x];
    }
    sieve(0);
    bool new_z = true;
    for (int par = 0;; par ^= 1) {  // rounds: one queue each, of one batch
      __syncthreads();
      const int p0 = b * nlb, nl = min(nlb, N - p0);
      int pre[WPB + 1], lpre[WPB + 1];
      pre[0] = lpre[0] = 0;
      int more = 0;
#pragma unroll
      for (int w = 0; w < WPB; w++) {
        const int *o = sCnt + (par * WPB + w) * 4;
        pre[w + 1] = pre[w] + __builtin_amdgcn_readfirstlane(o[0]);
        if constexpr (MODE == kEmit) lpre[w + 1] = lpre[w] + __builtin_amdgcn_readfirstlane(o[1]);
        more |= __builtin_amdgcn_readfirstlane(o[2]);
      }
      const int total = pre[WPB];
      if (new_z) {
        // ---- Z_s(p1; q2, q3) of the batch -> LDS ----
        const C2 *tab = sTab + ((lg & 1) ? N : 0);
        for (int lt = 0; lt < nl; lt += 16) {
          const uint32_t q2 = wrap_up(p0 + lt + li - k2, N);
          C2 f[KS];
#pragma unroll
          for (int ks = 0; ks < KS; ks++) f[ks] = tab[mod_small(__umul24(q2, (4 * ks + lg) >> 1), N, inv_n)];
#pragma unroll
          for (int i = 0; i < TPW; i++) {
            const int tile = wave + WPB * i;
            if (tile < LY::MT) {  // wave-uniform
              Acc zr = Acc{0, 0, 0, 0}, zi = Acc{0, 0, 0, 0};
#pragma unroll
              for (int ks = 0; ks < KS; ks++) {
                zr = MM::mul(ya[i][ks], f[ks].x, zr);
                zi = MM::mul(ya[i][ks], f[ks].y, zi);
              }
              const int row = 16 * tile + 4 * lg;
              C2 *z = sZ + __umul24(lt + li, LY::ZB) + row;
              if constexpr (LY::ROWS % 4 == 0) {
                if (LY::ROWS % 16 == 0 || row < LY::ROWS)
#pragma unroll
                  for (int r = 0; r < 4; r++) z[r] = mk<T>(zr[r], zi[r]);
              } else {
#pragma unroll
                for (int r = 0; r < 4; r++)
                  if (row + r < LY::ROWS) z[r] = mk<T>(zr[r], zi[r]);
              }
            }
          }
        }
        __syncthreads();
      }
      // ---- the next batch's share of the sieve: waves with a pass of
      //      vertices more take fewer chunks; its band ranges load meanwhile ----
      const int turn = (wave - rot) & (WPB - 1);  // this wave's turn in the round
      if (!more && b + 1 < nbatch) {
        // groups of sieve that cost a pass; with 6 modes it hardly matters (Si-like
        // 48^3, FP64: 20.16 ms with 256, 20.21 with 32, 20.15 with 1024; 130^3,
        // FP32: 42.5, 41.3, 42.5)
        constexpr int kPassChunks = NM == 3 ? 32 : 256;
        const int nc = (min(nlb, N - (b + 1) * nlb) * N + 15) >> 4;
        const int heavy = ((total + 63) >> 6) % WPB, light = WPB - heavy;
        const int x = heavy ? max(0, nc - light * kPassChunks) / WPB : 0, rest_c = nc - heavy * x;
        const int j = turn - heavy;
        const float r = __builtin_amdgcn_rcpf((float)light);  // (rest_c j + 1/2) / light: exact at j = light
        const int c0 = j < 0 ? turn * x : heavy * x + (int)(((float)(rest_c * j) + 0.5f) * r);
        const int c1 = j < 0 ? c0 + x : heavy * x + (int)(((float)(rest_c * (j + 1)) + 0.5f) * r);
        start_batch(b + 1, __builtin_amdgcn_readfirstlane(c0), __builtin_amdgcn_readfirstlane(c1));
      }
      // ---- vertices of all queues, one per lane ----
      // bases of the batch's first p and of the plane's first q
      [[maybe_unused]] const double2 *evec_b = a.evec + (int64_t)p3 * (NW * NW) * n2 + p0 * N;
      [[maybe_unused]] const double2 *uu_q = a.uu + (int64_t)q3 * (NM * NM) * n2;
      [[maybe_unused]] const double *occ_b =
          a.occ_f + (NT == 1 ? (int64_t)p3 * NW * n2 + p0 * N : 2 * ((int64_t)p3 * NW * 2 * n2 + p0 * N));
      [[maybe_unused]] const float4 *rec_b = a.rec_p + (int64_t)p3 * NW * kPC * n2 + p0 * N;
      [[maybe_unused]] const float4 *rec_qp = a.rec_q + (int64_t)q3 * kQC * n2;
      for (int v0 = 64 * turn; v0 < total; v0 += 64 * WPB) {
        const bool live = v0 + lane < total;
        const int i = min(v0 + lane, total - 1);  // lanes past the end repeat the last vertex and drop it
        int at = i, lbase = 0;
#pragma unroll
        for (int w = 1; w < WPB; w++) {
          at = (i >= pre[w]) ? i - pre[w] + w * QC : at;
          if constexpr (MODE == kEmit) lbase = (i >= pre[w]) ? lpre[w] : lbase;
        }
        at += par * WPB * QC;
        const uint32_t pm = sQ[at], e = pm / NW, m = pm % NW;  // p from the batch's first on, band
        const uint32_t vl = (uint32_t)(((float)e + 0.5f) * inv_n), vp1 = e - __umul24(vl, N);
        const uint32_t q1 = wrap_up(vp1 - k1, N), q2 = wrap_up(p0 + vl - k2, N);
        const uint32_t qoff = __umul24(q2, N) + q1;  // q in its plane
        double d;
        C2 vrow[NW];
        // FP32: the records' chunks, all loads of the vertex issued here, ahead of
        // the sum below, which hides them
        [[maybe_unused]] float4 pc[kPC], qc[kQC];
        [[maybe_unused]] auto p_float = [&](int f) __attribute__((always_inline)) {
          const float4 c = pc[f / 4];
          return f % 4 == 0 ? c.x : f % 4 == 1 ? c.y : f % 4 == 2 ? c.z : c.w;
        };
        [[maybe_unused]] auto q_float = [&](int f) __attribute__((always_inline)) {
          const float4 c = qc[f / 4];
          return f % 4 == 0 ? c.x : f % 4 == 1 ? c.y : f % 4 == 2 ? c.z : c.w;
        };
        [[maybe_unused]] double wq[NM];
        [[maybe_unused]] double2 uq[NM][NM];
        if constexpr (sizeof(T) == 8) {
          d = es - at_offset(eps_p + p0 * N, (m * (uint32_t)n2 + e) * 8u);
#pragma unroll
          for (int j = 0; j < NW; j++) vrow[j] = at_offset(evec_b + j * n2, (m * (uint32_t)(NW * n2) + e) * 16u);
          if constexpr (NM == 3) {  // the modes too, ahead of the sum (6 would not fit the registers)
#pragma unroll
            for (int nu = 0; nu < NM; nu++) {
              wq[nu] = at_offset(om_q + nu * n2, qoff * 8u);
#pragma unroll
              for (int mu = 0; mu < NM; mu++) uq[nu][mu] = at_offset(uu_q + (nu * NM + mu) * n2, qoff * 16u);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int c = 0; c < kPC; c++) pc[c] = at_offset(rec_b + c * n2, (m * (uint32_t)(kPC * n2) + e) * 16u);
#pragma unroll
          for (int c = 0; c < kQC; c++) qc[c] = at_offset(rec_qp + c * n2, qoff * 16u);
          __builtin_amdgcn_sched_barrier(0);
          d = es - __hiloint2double(__float_as_int(p_float(kPE + 1)), __float_as_int(p_float(kPE)));
#pragma unroll
          for (int j = 0; j < NW; j++) vrow[j] = mk<T>(p_float(2 * j), p_float(2 * j + 1));
        }
        // W_mu = sum_p e^{i 2 pi q1 p/N} sum_i conj(V_im(k+q)) Z(p; mu, i)
        T wr[NM], wi[NM];
        const C2 rq = sTab[q1];
        const C2 *zs = sZ + (size_t)__umul24(vl, LY::ZB);
#pragma unroll
        for (int mu = 0; mu < NM; mu++) {
          wr[mu] = wi[mu] = 0;
#pragma unroll
          for (int j = 0; j < NW; j++) {
            const C2 z = zs[(NB - 1) * C + mu * NW + j];
            cmac_conj<T>(wr[mu], wi[mu], vrow[j].x, vrow[j].y, z.x, z.y);
          }
        }
        // two steps at a time: one copies the sums back, more spill (Al-like
        // 100^3, FP64: 174, 167, 183 ms with 1, 2, 5; Si-like 48^3: 25, 20, 20)
#pragma unroll 2
        for (int pp = NB - 2; pp >= 0; pp--) {
#pragma unroll
          for (int mu = 0; mu < NM; mu++) {
            T tr = 0, ti = 0;
            cmac<T>(tr, ti, rq.x, rq.y, wr[mu], wi[mu]);
#pragma unroll
            for (int j = 0; j < NW; j++) {
              const C2 z = zs[pp * C + mu * NW + j];
              cmac_conj<T>(tr, ti, vrow[j].x, vrow[j].y, z.x, z.y);
            }
            wr[mu] = tr;
            wi[mu] = ti;
          }
        }
        // modes: with a = |g|^2 d+, b = |g|^2 d- (d+- the Gaussians),
        // sum_nu |g|^2 [(N + f) d+ + (1 + N - f) d-] =
        // sum_nu N (a + b) + f sum_nu a + (1 - f) sum_nu b, all terms >= 0: near
        // f = 1 blocked emission must not cancel into what absorption leaves.
        // Every mode is evaluated and masked (about 5 of the 6 (nu, +-) terms of
        // a vertex are kept, so branching would not save work).
        T sa = 0, sb = 0, ct[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) ct[t] = 0;
#pragma unroll MU
        for (int nu = 0; nu < NM; nu++) {
          double w;
          C2 u[NM];
          if constexpr (sizeof(T) == 8 && NM == 3) {
            w = wq[nu];
#pragma unroll
            for (int mu = 0; mu < NM; mu++) u[mu] = uq[nu][mu];
          } else if constexpr (sizeof(T) == 8) {
            w = at_offset(om_q + nu * n2, qoff * 8u);
#pragma unroll
            for (int mu = 0; mu < NM; mu++) u[mu] = at_offset(uu_q + (nu * NM + mu) * n2, qoff * 16u);
          } else {
            w = __hiloint2double(__float_as_int(q_float(kQW + 2 * nu + 1)), __float_as_int(q_float(kQW + 2 * nu)));
#pragma unroll
            for (int mu = 0; mu < NM; mu++) u[mu] = mk<T>(q_float(2 * (nu * NM + mu)), q_float(2 * (nu * NM + mu) + 1));
          }
          const double xpd = d + w, xmd = d - w;
          const bool okp = live && fabs(xpd) <= cut, okm = live && fabs(xmd) <= cut;
          n_t += __popcll(__ballot(okp)) + __popcll(__ballot(okm));
          T gr = 0, gi = 0;
#pragma unroll
          for (int mu = 0; mu < NM; mu++) cmac<T>(gr, gi, wr[mu], wi[mu], u[mu].x, u[mu].y);
          const T g2 = fma(gr, gr, gi * gi);
          T dp, dm;
          if constexpr (sizeof(T) == 8) {
            // exp_neg(-800) is zero: no branch, so that the modes' loads and
            // chains run beside each other
            dp = exp_neg(okp ? -(xpd * inv_eta) * (xpd * inv_eta) : -800.0);
            dm = exp_neg(okm ? -(xmd * inv_eta) * (xmd * inv_eta) : -800.0);
          } else {
            // FP32 form: |g|^2, the Gaussians and the occupation weights in
            // FP32 (the arguments x are formed in FP64 from the FP64 energies)
            const float xp = (float)xpd * ex2, xm = (float)xmd * ex2;
            dp = okp ? __builtin_amdgcn_exp2f(-xp * xp) : 0.f;
            dm = okm ? __builtin_amdgcn_exp2f(-xm * xm) : 0.f;
          }
          const T ga = g2 * (dp + dm);
          sa = fma(g2, dp, sa);
          sb = fma(g2, dm, sb);
#pragma unroll
          for (int t = 0; t < NT; t++) {
            T nq;
            if constexpr (sizeof(T) == 4) {
              nq = q_float(kQN + nu * NT + t);
            } else if constexpr (NT == 1) {
              nq = at_offset(a.occ_n + (q3 * NM + nu) * n2, qoff * 8u);
            } else {
              const double2 f = at_offset(reinterpret_cast<const double2 *>(a.occ_n) + ((q3 * NM + nu) * 2 + t / 2) * n2, qoff * 16u);
              nq = t % 2 ? f.y : f.x;
            }
            ct[t] = fma(nq, ga, ct[t]);
          }
        }
#pragma unroll
        for (int t = 0; t < NT; t++) {
          T f;
          if constexpr (sizeof(T) == 4) {
            f = p_float(kPF + t);
          } else if constexpr (NT == 1) {
            f = at_offset(occ_b, (m * (uint32_t)n2 + e) * 8u);
          } else {
            const double2 f2 = at_offset(reinterpret_cast<const double2 *>(occ_b) + (t / 2) * n2, (m * (uint32_t)(2 * n2) + e) * 16u);
            f = t % 2 ? f2.y : f2.x;
          }
          ct[t] = fma(f, sa, ct[t]) + fma(-f, sb, sb);  // (1 - f) sb rounded once
        }
        if (live) {
#pragma unroll
          for (int t = 0; t < NT; t++) acc[t] += (double)ct[t];
          if constexpr (MODE == kEmit) {
            if (sRank[at] != 0xffff) {  // final state in the list: its transition rate
              const int64_t e = gpos + lbase + sRank[at];
              a.g_col[e] = at_offset(a.stidx + (p3 * n2 + p0 * N) * NW, pm * 4u);
#pragma unroll
              for (int t = 0; t < NT; t++)
                if (t < a.nt) a.g_val[(int64_t)t * a.g_stride + e] = pref * (double)ct[t];
            }
          }
        }
      }
      if constexpr (MODE == kEmit) gpos += lpre[WPB];
      // ---- the next round's queue ----
      if (!more && ++b == nbatch) break;  // workgroup-uniform
      new_z = !more;
      rot = (rot + 1) & (WPB - 1);
      sieve(par ^ 1);
    }
    __syncthreads();  // the next plane and the reductions reuse the LDS
  }
  }

  if constexpr (MODE == kCount) {  // the slab's transition rates of the state
    if (lane == 0) sCnt[wave] = n_v;
    __syncthreads();
    if (threadIdx.x == 0) {
      int64_t c = 0;
      for (int w = 0; w < WPB; w++) c += sCnt[w];
      if (a.g_slot) a.g_slot[slot * a.ns_total + s] = c;
      else a.g_cursor[s] += c;
    }
    return;
  }
  if constexpr (MODE == kEmit)
    if (threadIdx.x == 0 && !a.g_slot) a.g_cursor[s] = gpos + a.g_base;

  // ---- fixed-order reductions; slabs add up in order ----
#pragma unroll
  for (int t = 0; t < NT; t++) {
    double v = acc[t];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    if (lane == 0) sRed[wave * 8 + t] = v;
  }
  const int n_q = n_v - n_dup;
  if (nsh == 0) n_kq = count_kq ? n_q : 0;
  if (lane == 0) {
    int *c = reinterpret_cast<int *>(sRed + wave * 8 + 4);
    c[0] = n_q;
    c[1] = n_kq;
    c[2] = n_v;
    sRed[wave * 8 + 6] = __longlong_as_double(n_t);
  }
  __syncthreads();
  if ((int)threadIdx.x < NT && (int)threadIdx.x < a.nt) {
    const int t = threadIdx.x;
    double v = 0.0;
    for (int w = 0; w < WPB; w++) v += sRed[w * 8 + t];
    v *= pref;
    if (a.part_tau) {
      a.part_tau[((int64_t)slot * a.nt + t) * a.ns_total + s] = v;
    } else {
      double *dst = a.inv_tau + (int64_t)t * a.ns_total + s;
      *dst = (slab == 0 ? 0.0 : *dst) + v;
    }
  } else if (threadIdx.x >= 8 && threadIdx.x < 12) {
    const int j = threadIdx.x - 8;  // n_q, n_terms, (k,q) pairs, vertices
    int64_t v = 0;
    for (int w = 0; w < WPB; w++)
      v += j == 1 ? __double_as_longlong(sRed[w * 8 + 6]) : reinterpret_cast<const int *>(sRed + w * 8 + 4)[j == 0 ? 0 : j - 1];
    if (a.part_tau) {
      a.part_cnt[((int64_t)slot * a.ns_total + s) * 4 + j] = v;
    } else {
      int64_t *dst = (j < 2 ? a.st_counts : a.kv_counts - 2) + s * 2 + j;
      *dst = (slab == 0 ? 0 : *dst) + v;
    }
  }
}

template <class T, int NW, int NM, int NB, int NT, int MODE>
hipError_t launch_wave(const RatesArgs &a, hipStream_t st) {
  using LY = WaveLayout<T, NW, NM, NB>;
  const size_t sh = LY::total(a.N, MODE, a.slab_planes);
  if (sh > 160 * 1024) return hipErrorInvalidValue;
  auto kern = rates_wave_kernel<T, NW, NM, NB, NT, MODE>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
  if (e != hipSuccess) return e;
  constexpr int64_t kPiece = kLaunchThreads / (LY::WPB * 64);  // states
  for (int64_t i = 0; i < a.ns_launch && e == hipSuccess; i += kPiece) {
    RatesArgs b = a;
    b.s_lo = a.s_lo + i;
    b.ns_launch = a.ns_launch - i < kPiece ? a.ns_launch - i : kPiece;
    const int64_t grid = ((b.ns_launch + 7) / 8) * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid, (unsigned)(a.slab_hi - a.slab_lo)), dim3(LY::WPB * 64), sh, st, b);
    e = hipGetLastError();
  }
  return e;
}

template <class T, int NW, int NM, int NB, int MODE>
hipError_t launch_wave_t(const RatesArgs &a, hipStream_t st) {
  if constexpr (MODE == kCount) {
    return launch_wave<T, NW, NM, NB, 1, MODE>(a, st);
  } else {
    if (a.nt == 1) return launch_wave<T, NW, NM, NB, 1, MODE>(a, st);
    return launch_wave<T, NW, NM, NB, EPH_MAX_TEMPS, MODE>(a, st);
  }
}

// Launch for one (precision, modes, mode) triple: dispatch on the orbital
// count, the Rp box edge and the temperatures.
template <class T, int NM, int MODE>
hipError_t dispatch_nm(const RatesArgs &a, hipStream_t st) {
  const int nb = a.box.n[0];
#define EPH_W(NW_)                                                 \
  if (a.nw == NW_) {                                               \
    if (nb == 4) return launch_wave_t<T, NW_, NM, 4, MODE>(a, st); \
    if (nb == 6) return launch_wave_t<T, NW_, NM, 6, MODE>(a, st); \
    return hipErrorNotSupported;                                   \
  }
  EPH_W(1)
  EPH_W(2)
  EPH_W(4)
  EPH_W(8)
#undef EPH_W
  return hipErrorNotSupported;
}

}  // namespace wave
}  // namespace eph
