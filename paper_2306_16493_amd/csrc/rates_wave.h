#pragma once
// SERTA scattering rates (gfx950): the kernel template.  Instantiated per
// (precision, phonon modes, mode) in k_rates_wave_<p><nm>.hip and dispatched
// by k_rates_wave.hip.
//
// Same arithmetic as the general form (separable Rp box: Y per q3, Z per
// q-line, G per q; vertex contracted onto the final band m first, then onto
// the modes; sieve, occupations, Gaussian delta; Sec. II.B/II.C/III.A/III.C).
// One workgroup takes one initial state s = (n, k) and one q3 plane:
//   * Y_s(p1,p2; q3) is formed once per plane, straight into the registers of
//     a matrix-core operand, its (p1, channel) rows spread over the waves;
//   * Z_s(p1; q2,q3) of a batch of q-lines is one matrix product per 16 lines
//     (16x16x4 MFMA, rows (p1, channel), inner index (p2, re/im), columns the
//     lines) into LDS, where all waves read it;
//   * the q of the batch are taken 64 at a time in the order of the final
//     states p = k + q, across line ends, so no lane idles at the end of a
//     line.  Each is sieved exactly (FP64, every final band near the state's
//     energy; the compares go into wave masks, which the scalar unit joins
//     and counts), and the (p, m) with a kept term go to the wave's queue;
//   * the queues of the waves are then evaluated as one list, one vertex per
//     lane, whole passes dealt out to the waves.
// Fermi and Bose factors come from per-call grid tables, so a vertex pays one
// exp per kept term (the delta) and no other transcendental.  The phase of
// the box corner, e^{i q.lo}, is common to all terms of a vertex and leaves
// |g|^2 alone, so the three sums run over p = 0 .. NB-1, the last one by
// Horner's rule.  The lists, their order and the sums over
// lanes, waves and planes are fixed, so results are bit-reproducible.
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

// (a mod N) for 0 <= a < 2^20, N <= 512: the float quotient is off by one at most
__device__ __forceinline__ int fmod_small(int a, int N, float inv_n) {
  int r = a - N * (int)floorf((float)a * inv_n);
  r += (r < 0) ? N : 0;
  r -= (r >= N) ? N : 0;
  return r;
}

template <class T, int NW, int NM, int NB>
struct WaveLayout {
  using C2 = typename V2<T>::t;
  static constexpr int C = NW * NM;
  static constexpr int ROWS = NB * C;               // (p1, channel) rows of Y and Z
  static constexpr int MT = (ROWS + 15) / 16;       // 16-row tiles
  static constexpr int KS = (2 * NB + 3) / 4;       // 4-deep steps over (p2, re/im)
  static constexpr int WPB = (C >= 48 && sizeof(T) == 8) ? 8 : 4;  // waves per workgroup
  static constexpr int TPW = (MT + WPB - 1) / WPB;  // tiles per wave
  // lines per batch: 32 where two batches' worth of LDS is small, so that the
  // partial last pass over the queue is rare; 16 for 48 channels
  static constexpr int NL = C >= 48 ? 16 : 32;
  // one line's Z, padded by 16 bytes so that neighbouring lines start in
  // different LDS banks
  static constexpr int ZB = ROWS + (int)(16 / sizeof(C2));
  static constexpr int QC = 64 * NW + 512;          // queue entries per wave
  __host__ __device__ static size_t tab_bytes(int N) { return align16(sizeof(C2) * (size_t)N); }
  static constexpr size_t z_bytes = sizeof(C2) * (size_t)NL * ZB;
  static constexpr size_t q_bytes = 4 * (size_t)WPB * QC;
  static constexpr size_t rank_bytes = 2 * (size_t)WPB * QC;  // emit mode
  static constexpr size_t misc_bytes = 8 * (size_t)WPB * 8 + 64;
  __host__ __device__ static size_t total(int N, int mode) {
    return misc_bytes + q_bytes + (mode == kCount ? 0 : tab_bytes(N) + z_bytes) + (mode == kEmit ? rank_bytes : 0);
  }
};

// Waves per SIMD the register allocation targets.
template <class T, int NW, int NM>
__host__ __device__ constexpr int waves_per_eu() {
  return sizeof(T) == 4 ? (NW * NM >= 48 ? 3 : 4) : (NW * NM >= 48 ? 2 : 3);
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
  constexpr int C = LY::C, WPB = LY::WPB, TPW = LY::TPW, KS = LY::KS, NL = LY::NL, QC = LY::QC;
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
  const int plane = blockIdx.y, q3 = a.q3_lo + plane;

  uint32_t *sQ = reinterpret_cast<uint32_t *>(smem);            // [WPB][QC] vertices: p1 | line << 9 | m << 15 | listed << 31
  double *sRed = reinterpret_cast<double *>(smem + LY::q_bytes);  // [WPB][8] reductions; queue lengths in between
  int *sCnt = reinterpret_cast<int *>(sRed);                    // [WPB][4]: length, listed entries, more to come
  unsigned char *rest = smem + LY::q_bytes + LY::misc_bytes;
  C2 *sTab = reinterpret_cast<C2 *>(rest);                      // e^{2 pi i m/N}
  C2 *sZ = reinterpret_cast<C2 *>(rest + LY::tab_bytes(N));     // [NL][ZB]: [p1][mu][i] + pad
  uint16_t *sRank = reinterpret_cast<uint16_t *>(rest + LY::tab_bytes(N) + LY::z_bytes);  // [WPB][QC]

  if constexpr (MODE != kCount)
    for (int t = threadIdx.x; t < N; t += WPB * 64) sTab[t] = mk<T>((T)a.tab[t].x, (T)a.tab[t].y);

  const int k = a.sk[s], n = a.sn[s];
  const int k1 = k % N, k2 = (k / N) % N, k3 = k / (N * N);
  const double es = a.eps[(int64_t)k * NW + n];
  // the first state of a k point also looks for the other states' terms, so
  // that every (k, q) pair is counted once
  int nsh = 0;
  if (MODE != kCount && (s == 0 || a.sk[s - 1] != k))
    while (nsh < NW - 1 && s + 1 + nsh < a.ns_total && a.sk[s + 1 + nsh] == k) nsh++;
  const bool count_kq = s == 0 || a.sk[s - 1] != k;
  const double cut = a.sw * a.eta;
  // bands further away keep no term (the margin covers the rounding of the
  // exact test)
  const double reach = (a.wmax + cut) * (1.0 + 1e-12) + 1e-12 * fabs(es);
  const double inv_eta = 1.0 / a.eta;
  const double dnorm = 1.0 / (1.7724538509055160273 * a.eta);
  const float inv_n = 1.0f / (float)N;
  const int p3 = (k3 + q3 >= N) ? k3 + q3 - N : k3 + q3;
  // the planes of the tables that this workgroup reads
  const int64_t p_plane = (int64_t)N * N * p3, q_plane = (int64_t)N * N * q3;
  const double *eps_p = a.eps + p_plane * NW, *om_q = a.om + q_plane * NM;
  const int32_t *stidx_p = MODE == kRates ? nullptr : a.stidx + p_plane * NW;
  const C2 *evec_p, *uu_q;
  const T *occ_p, *occ_q;
  if constexpr (sizeof(T) == 8) {
    evec_p = a.evec + p_plane * (NW * NW);
    uu_q = a.uu + q_plane * (NM * NM);
    occ_p = a.occ_f + p_plane * (NW * NT);
    occ_q = a.occ_n + q_plane * (NM * NT);
  } else {
    evec_p = a.evec32 + p_plane * (NW * NW);
    uu_q = a.uu32 + q_plane * (NM * NM);
    occ_p = a.occ32_f + p_plane * (NW * NT);
    occ_q = a.occ32_n + q_plane * (NM * NT);
  }

  double acc[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) acc[t] = 0.0;
  int n_q = 0, n_t = 0, n_kq = 0, n_v = 0;  // wave-uniform counts
  int64_t gpos = 0;                         // next transition rate of the state
  if constexpr (MODE == kEmit) gpos = a.g_cursor[s] + (a.g_slot ? a.g_slot[plane * a.ns_total + s] : 0) - a.g_base;

  // ---- Y_s(p1, p2; q3) as the A operand: lane (i, g) of tile t and step ks
  //      holds row 16 t + row_of(i) = (p1, channel), inner index 4 ks + g =
  //      (p2, re/im) ----
  const int li = lane & 15, lg = lane >> 4;
  T ya[TPW][KS];
  if constexpr (MODE != kCount) {
    __syncthreads();  // phase table
    const C2 *X = reinterpret_cast<const C2 *>(a.X) + (s - a.s_base) * (int64_t)(NB * NB * NB * C);
    C2 ph3[NB];
    {
      int i3 = 0;
#pragma unroll
      for (int p = 0; p < NB; p++) {
        ph3[p] = sTab[i3];
        i3 += q3;
        i3 -= (i3 >= N) ? N : 0;
      }
    }
#pragma unroll
    for (int i = 0; i < TPW; i++) {
      const int row = 16 * (wave + WPB * i) + MM::row_of(li);
      const int p1 = row / C, c = row - p1 * C;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        const int p2 = (4 * ks + lg) >> 1;
        const bool im = lg & 1;
        T y = 0;
        if (row < LY::ROWS && p2 < NB) {
          const C2 *x = X + ((p1 * NB + p2) * NB) * C + c;
#pragma unroll
          for (int p = 0; p < NB; p++) {
            const C2 v = x[p * C];
            y = fma(ph3[p].x, im ? v.y : v.x, y);
            y = fma(ph3[p].y, im ? v.x : -v.y, y);
          }
        }
        ya[i][ks] = y;
      }
    }
  }

  const int nbatch = (N + NL - 1) / NL;
  const int nlb = (N + nbatch - 1) / nbatch;  // lines per batch, evened out
  for (int q2_0 = 0; q2_0 < N; q2_0 += nlb) {
    const int nl = min(nlb, N - q2_0);
    // ---- Z_s(p1; q2, q3) of the batch -> LDS ----
    if constexpr (MODE != kCount) {
      for (int lt = 0; lt < nl; lt += 16) {
        T br[KS], bi[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
          const C2 ph = sTab[fmod_small(__umul24(q2_0 + lt + li, (4 * ks + lg) >> 1), N, inv_n)];
          br[ks] = (lg & 1) ? -ph.y : ph.x;
          bi[ks] = (lg & 1) ? ph.x : ph.y;
        }
#pragma unroll
        for (int i = 0; i < TPW; i++) {
          const int tile = wave + WPB * i;
          if (tile < LY::MT) {  // wave-uniform
            Acc zr = Acc{0, 0, 0, 0}, zi = Acc{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
              zr = MM::mul(ya[i][ks], br[ks], zr);
              zi = MM::mul(ya[i][ks], bi[ks], zi);
            }
            const int row = 16 * tile + 4 * lg;
            C2 *z = sZ + (size_t)(lt + li) * LY::ZB + row;
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
    }

    // ---- sieve of the batch's q, in the order of p; 64 per chunk, chunk c
    //      to wave (c + rotation) % WPB ----
    const int ne = nl * N;
    const int rot = (int)((s + q2_0) & (WPB - 1));
    int base = 64 * ((wave - rot) & (WPB - 1));  // first entry of the wave's next chunk
    const uint32_t step_l = (uint32_t)(64 * WPB) / (uint32_t)N, step_p = 64 * WPB - step_l * N;
    uint32_t pl = (uint32_t)(base + lane) / (uint32_t)N, p1 = base + lane - pl * N;  // line in the batch, p1
    // table entries of the next chunk, loaded a chunk ahead; lanes past the
    // end read in bounds and are masked
    double ep[NW], om[NM];
    uint32_t item = 0, poff = 0;
    auto fetch = [&]() __attribute__((always_inline)) {
      const uint32_t l = min(pl, (uint32_t)(nl - 1)), q2 = q2_0 + l;
      const uint32_t p2 = wrap_down(k2 + q2, N), q1 = wrap_up(p1 - k1, N);
      item = p1 | (l << 9);
      poff = __umul24(p2, N) + p1;
      const uint32_t qoff = __umul24(q2, N) + q1;
#pragma unroll
      for (int m = 0; m < NW; m++) ep[m] = at_offset(eps_p + m, poff * (uint32_t)(8 * NW));
#pragma unroll
      for (int nu = 0; nu < NM; nu++) om[nu] = at_offset(om_q + nu, __umul24(qoff, 8 * NM));
      p1 += step_p;
      pl += step_l;
      pl += (p1 >= (uint32_t)N) ? 1u : 0u;
      p1 = wrap_down(p1, N);
    };
    if (base < ne) fetch();
    bool more;
    do {
      int cnt = 0, listed = 0;
      while (base < ne && cnt <= QC - 64 * NW) {
        const int nlane = ne - base;  // lanes in range
        const unsigned long long valid = nlane >= 64 ? ~0ull : (1ull << nlane) - 1ull;
        double e_[NW], w_[NM];
        unsigned long long okw[NM];  // modes above the frequency cut, lanes in range
#pragma unroll
        for (int m = 0; m < NW; m++) e_[m] = ep[m];
#pragma unroll
        for (int nu = 0; nu < NM; nu++) {
          w_[nu] = om[nu];
          okw[nu] = __ballot(om[nu] >= a.wcut) & valid;
        }
        const uint32_t item_ = item, poff_ = poff;
        base += 64 * WPB;
        if (base < ne) fetch();
        // a term (nu, +-) is kept when |d +- w| <= cut with d = es - ep: the
        // nearer of the two has |  |d| - w  |
        unsigned long long hit = 0;
#pragma unroll
        for (int m = 0; m < NW; m++) {
          const double d = es - e_[m];
          if (!(__ballot(fabs(d) <= reach) & valid)) continue;  // wave-uniform
          unsigned long long any = 0;
#pragma unroll
          for (int nu = 0; nu < NM; nu++) any |= __ballot(fabs(fabs(d) - w_[nu]) <= cut) & okw[nu];
          if (any) {
            hit |= any;
            const bool mine = __builtin_amdgcn_inverse_ballot_w64(any);
            if constexpr (MODE == kRates) {
              if (mine) sQ[wave * QC + cnt + lanes_below(any)] = item_ | ((uint32_t)m << 15);
            } else {
              const bool in_list = mine && at_offset(stidx_p + m, poff_ * (uint32_t)(4 * NW)) >= 0;
              const unsigned long long lm = __ballot(in_list);
              if constexpr (MODE == kEmit) {
                if (mine) {
                  const int at = wave * QC + cnt + lanes_below(any);
                  sQ[at] = item_ | ((uint32_t)m << 15) | (in_list ? 0x80000000u : 0u);
                  sRank[at] = (uint16_t)(listed + lanes_below(lm));
                }
              }
              listed += __popcll(lm);
            }
            cnt += (MODE == kCount) ? 0 : __popcll(any);
          }
        }
        n_q += __popcll(hit);
        for (int j = 0; j < nsh; j++) {  // the other states at this k point
          const double e2 = a.eps[(int64_t)k * NW + a.sn[s + 1 + j]];
#pragma unroll
          for (int m = 0; m < NW; m++) {
            const double d = fabs(e2 - e_[m]);
#pragma unroll
            for (int nu = 0; nu < NM; nu++) hit |= __ballot(fabs(d - w_[nu]) <= cut) & okw[nu];
          }
        }
        if (count_kq) n_kq += __popcll(hit);
      }
      if constexpr (MODE == kCount) {
        n_v += listed;
        more = false;
        continue;
      }
      n_v += cnt;
      if (lane == 0) {
        sCnt[wave * 4] = cnt;
        sCnt[wave * 4 + 1] = listed;
        sCnt[wave * 4 + 2] = base < ne ? 1 : 0;
      }
      __syncthreads();
      // ---- vertices of all queues, one per lane ----
      int pre[WPB + 1], lpre[WPB + 1];
      pre[0] = lpre[0] = 0;
      int left = 0;
#pragma unroll
      for (int w = 0; w < WPB; w++) {
        pre[w + 1] = pre[w] + __builtin_amdgcn_readfirstlane(sCnt[w * 4]);
        if constexpr (MODE == kEmit) lpre[w + 1] = lpre[w] + __builtin_amdgcn_readfirstlane(sCnt[w * 4 + 1]);
        left |= __builtin_amdgcn_readfirstlane(sCnt[w * 4 + 2]);
      }
      more = left != 0;
      const int total = pre[WPB];
      for (int v0 = 64 * ((wave - rot) & (WPB - 1)); v0 < total; v0 += 64 * WPB) {
        const bool live = v0 + lane < total;
        const int i = min(v0 + lane, total - 1);  // lanes past the end repeat the last vertex and drop it
        int at = i, lbase = 0;
#pragma unroll
        for (int w = 1; w < WPB; w++) {
          at = (i >= pre[w]) ? i - pre[w] + w * QC : at;
          if constexpr (MODE == kEmit) lbase = (i >= pre[w]) ? lpre[w] : lbase;
        }
        const uint32_t it = sQ[at];
        const uint32_t vp1 = it & 511u, vl = (it >> 9) & 63u, m = (it >> 15) & 7u;
        const uint32_t q2 = q2_0 + vl, p2 = wrap_down(k2 + q2, N), q1 = wrap_up(vp1 - k1, N);
        const uint32_t qoff = __umul24(q2, N) + q1;              // q in its plane
        const uint32_t pm = (__umul24(p2, N) + vp1) * NW + m;    // (p, m) in its plane
        const double d = es - at_offset(eps_p, pm * 8u);
        C2 vrow[NW];
#pragma unroll
        for (int j = 0; j < NW; j++) vrow[j] = at_offset(evec_p + j, pm * (uint32_t)(sizeof(C2) * NW));
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
#pragma unroll 1
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
        // modes: with a = |g|^2 (d+ + d-), b = |g|^2 (d+ - d-), c = |g|^2 d-
        // (d+- the Gaussians), sum_nu |g|^2 [(N + f) d+ + (1 + N - f) d-] =
        // sum_nu N a + f sum_nu b + sum_nu c.  Every mode is evaluated and
        // masked (about 5 of the 6 (nu, +-) terms of a vertex are kept, so
        // branching would not save work).
        T sb = 0, sc = 0, ct[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) ct[t] = 0;
#pragma unroll(MU)
        for (int nu = 0; nu < NM; nu++) {
          const double w = at_offset(om_q + nu, __umul24(qoff, 8 * NM)), xpd = d + w, xmd = d - w;
          const bool on = live && w >= a.wcut;
          const bool okp = on && fabs(xpd) <= cut, okm = on && fabs(xmd) <= cut;
          n_t += __popcll(__ballot(okp)) + __popcll(__ballot(okm));
          T gr = 0, gi = 0;
#pragma unroll
          for (int mu = 0; mu < NM; mu++) {
            const C2 u = at_offset(uu_q + nu * NM + mu, __umul24(qoff, (uint32_t)(sizeof(C2) * NM * NM)));
            cmac<T>(gr, gi, wr[mu], wi[mu], u.x, u.y);
          }
          const T g2 = fma(gr, gr, gi * gi);
          T dp, dm;
          if constexpr (sizeof(T) == 8) {
            dp = okp ? exp(-(xpd * inv_eta) * (xpd * inv_eta)) * dnorm : 0.0;
            dm = okm ? exp(-(xmd * inv_eta) * (xmd * inv_eta)) * dnorm : 0.0;
          } else {
            // FP32 form: |g|^2, the Gaussians and the occupation weights in
            // FP32 (the arguments x are formed in FP64 from the FP64 energies)
            const float xp = (float)xpd * (float)inv_eta, xm = (float)xmd * (float)inv_eta;
            dp = okp ? __expf(-xp * xp) * (float)dnorm : 0.f;
            dm = okm ? __expf(-xm * xm) * (float)dnorm : 0.f;
          }
          const T ga = g2 * (dp + dm);
          sb = fma(g2, dp - dm, sb);
          sc = fma(g2, dm, sc);
#pragma unroll
          for (int t = 0; t < NT; t++)
            ct[t] = fma(at_offset(occ_q + nu * NT + t, __umul24(qoff, (uint32_t)(sizeof(T) * NM * NT))), ga, ct[t]);
        }
#pragma unroll
        for (int t = 0; t < NT; t++) ct[t] += fma(at_offset(occ_p + t, pm * (uint32_t)(sizeof(T) * NT)), sb, sc);
        if (live) {
#pragma unroll
          for (int t = 0; t < NT; t++) acc[t] += (double)ct[t];
          if constexpr (MODE == kEmit) {
            if (it >> 31) {  // final state in the list: its transition rate
              const int64_t e = gpos + lbase + sRank[at];
              a.g_col[e] = at_offset(stidx_p, pm * 4u);
#pragma unroll
              for (int t = 0; t < NT; t++)
                if (t < a.nt) a.g_val[(int64_t)t * a.g_stride + e] = a.pref * (double)ct[t];
            }
          }
        }
      }
      if constexpr (MODE == kEmit) gpos += lpre[WPB];
      __syncthreads();  // queues and Z are rewritten
    } while (more);
  }

  if constexpr (MODE == kCount) {  // this plane's transition rates of the state
    if (lane == 0) sCnt[wave] = n_v;
    __syncthreads();
    if (threadIdx.x == 0) {
      int64_t c = 0;
      for (int w = 0; w < WPB; w++) c += sCnt[w];
      if (a.g_slot) a.g_slot[plane * a.ns_total + s] = c;
      else a.g_cursor[s] += c;
    }
    return;
  }
  if constexpr (MODE == kEmit)
    if (threadIdx.x == 0 && !a.g_slot) a.g_cursor[s] = gpos + a.g_base;

  // ---- fixed-order reductions; planes add up in order ----
#pragma unroll
  for (int t = 0; t < NT; t++) {
    double v = acc[t];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    if (lane == 0) sRed[wave * 8 + t] = v;
  }
  if (lane == 0) {
    int *c = reinterpret_cast<int *>(sRed + wave * 8 + 4);
    c[0] = n_q;
    c[1] = n_t;
    c[2] = n_kq;
    c[3] = n_v;
  }
  __syncthreads();
  if ((int)threadIdx.x < NT && (int)threadIdx.x < a.nt) {
    const int t = threadIdx.x;
    double v = 0.0;
    for (int w = 0; w < WPB; w++) v += sRed[w * 8 + t];
    v *= a.pref;
    if (a.part_tau) {
      a.part_tau[((int64_t)plane * a.nt + t) * a.ns_total + s] = v;
    } else {
      double *dst = a.inv_tau + (int64_t)t * a.ns_total + s;
      *dst = (q3 == 0 ? 0.0 : *dst) + v;
    }
  } else if (threadIdx.x >= 8 && threadIdx.x < 12) {
    const int j = threadIdx.x - 8;
    int64_t v = 0;
    for (int w = 0; w < WPB; w++) v += reinterpret_cast<const int *>(sRed + w * 8 + 4)[j];
    if (a.part_tau) {
      a.part_cnt[((int64_t)plane * a.ns_total + s) * 4 + j] = v;
    } else {
      int64_t *dst = (j < 2 ? a.st_counts : a.kv_counts - 2) + s * 2 + j;
      *dst = (q3 == 0 ? 0 : *dst) + v;
    }
  }
}

template <class T, int NW, int NM, int NB, int NT, int MODE>
hipError_t launch_wave(const RatesArgs &a, hipStream_t st) {
  using LY = WaveLayout<T, NW, NM, NB>;
  const size_t sh = LY::total(a.N, MODE);
  if (sh > 160 * 1024) return hipErrorInvalidValue;
  auto kern = rates_wave_kernel<T, NW, NM, NB, NT, MODE>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
  if (e != hipSuccess) return e;
  const int64_t grid = ((a.ns_launch + 7) / 8) * 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid, (unsigned)(a.q3_hi - a.q3_lo)), dim3(LY::WPB * 64), sh, st, a);
  return hipGetLastError();
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
