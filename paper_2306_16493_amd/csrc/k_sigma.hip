// Conductivity reduction and its energy moments (Sec. II.C), the carrier
// density, and small element-wise helpers (gfx950).
//
// M_n,ab(T) = 2 e^2/(N_k V) sum_s v_a v_b tau_s f(1-f)/(k_B T) (eps_s - mu)^n
// (n = 0 is sigma; eps in eV), or with v_b tau_s replaced by the mean free
// path F_b of the iterative solution: each block reduces a contiguous chunk of
// states at one temperature, all moments at once, with Neumaier-compensated
// per-thread sums and a fixed butterfly, writing [n][block][T][9] partials; a
// second kernel adds the partials in a fixed tree and applies the prefactor.
// The carrier density sums f over the bands of the full grid the same way.
// Results are bit-identical from run to run.
//
// What bounds it: launches and the copy of the result; 437296 states at three
// temperatures are 24 MB, 5 us of reading.  Three moments of them take 53 us
// from call to result.  One kernel per moment over all temperatures, its sums
// indexed at run time and so in scratch memory, and a serial last step took
// 509 us.
#include <algorithm>

#include "internal.h"

namespace eph {
namespace {

constexpr int kSigThreads = 256;

__device__ __forceinline__ void neumaier(double &s, double &c, double x) {
  double t = s + x;
  if (fabs(s) >= fabs(x)) c += (s - t) + x;
  else c += (x - t) + s;
  s = t;
}

struct Kts {
  double v[EPH_MAX_TEMPS];
};

// Blocks (chunk of states, temperature); NO moments; FREE: mean free paths F.
// v_a v_b and its sums are symmetric bit for bit, so six of the nine are formed.
template <int NO, bool FREE>
__global__ __launch_bounds__(kSigThreads) void sigma_kernel(int64_t ns, const double *__restrict__ e,
                                                            const double *__restrict__ v,
                                                            const double *__restrict__ inv_tau, double mu, Kts kts,
                                                            double *__restrict__ partials, int64_t chunk,
                                                            const double *__restrict__ F) {
  constexpr int NC = FREE ? 9 : 6;  // xx, xy, xz, (yx,) yy, yz, (zx, zy,) zz
  __shared__ double red[kSigThreads / 64][NO * NC];
  const int t = blockIdx.y;
  const double kt = kts.v[t];
  const int64_t b0 = blockIdx.x * chunk, b1 = min(ns, b0 + chunk);
  double s[NO][NC], c[NO][NC];
#pragma unroll
  for (int o = 0; o < NO; o++)
#pragma unroll
    for (int q = 0; q < NC; q++) s[o][q] = c[o][q] = 0.0;
  for (int64_t i = b0 + threadIdx.x; i < b1; i += kSigThreads) {
    const double it = inv_tau[t * ns + i];
    if (it == 0.0) continue;
    const double vx = v[3 * i], vy = v[3 * i + 1], vz = v[3 * i + 2];
    const double de = e[i] - mu;
    const double f = 1.0 / (exp(de / kt) + 1.0);
    double vv[NC], w0;
    if constexpr (FREE) {  // mean free paths of the iterative solution: v_a F_b in place of v_a v_b tau
      const double *fb = F + (t * ns + i) * 3;
      const double fx = fb[0], fy = fb[1], fz = fb[2];
      const double x[9] = {vx * fx, vx * fy, vx * fz, vy * fx, vy * fy, vy * fz, vz * fx, vz * fy, vz * fz};
#pragma unroll
      for (int q = 0; q < NC; q++) vv[q] = x[q];
      w0 = f * (1.0 - f) / kt;
    } else {
      const double x[6] = {vx * vx, vx * vy, vx * vz, vy * vy, vy * vz, vz * vz};
#pragma unroll
      for (int q = 0; q < NC; q++) vv[q] = x[q];
      w0 = f * (1.0 - f) / kt / it;
    }
#pragma unroll
    for (int o = 0; o < NO; o++) {
      const double w = o == 0 ? w0 : w0 * (o == 1 ? de : de * de);
#pragma unroll
      for (int q = 0; q < NC; q++) neumaier(s[o][q], c[o][q], vv[q] * w);
    }
  }
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
#pragma unroll
  for (int o = 0; o < NO; o++)
#pragma unroll
    for (int q = 0; q < NC; q++) {
      double x = s[o][q] + c[o][q];
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
      if (lane == 0) red[wave][o * NC + q] = x;
    }
  __syncthreads();
  if (threadIdx.x < NO * 9) {
    const int o = threadIdx.x / 9, q = threadIdx.x % 9, a = min(q / 3, q % 3), b = max(q / 3, q % 3);
    const int col = o * NC + (FREE ? q : a == 0 ? b : a + b + 1);
    double x = 0.0;
    for (int w = 0; w < kSigThreads / 64; w++) x += red[w][col];
    partials[((int64_t)o * gridDim.x + blockIdx.x) * (EPH_MAX_TEMPS * 9) + t * 9 + q] = x;
  }
}

// out[y][q] = pref * sum_b partials[y][b][q], q < nq of ld, zero past nq: 16
// lanes per q, each a run of the blocks, joined by a fixed butterfly.  (One
// lane per q waits for one block's partial after the other: 67 us for 256.)
__global__ void final_kernel(int nblk, int ld, int nq, const double *__restrict__ partials, double pref,
                             double *__restrict__ out) {
  const int q = threadIdx.x / 16, l = threadIdx.x % 16;
  const double *p = partials + (int64_t)blockIdx.y * nblk * ld;
  double s = 0.0, c = 0.0;
  if (q < nq) {
    const int per = (nblk + 15) / 16, b1 = min(nblk, (l + 1) * per);
#pragma unroll 16
    for (int b = l * per; b < b1; b++) neumaier(s, c, p[(int64_t)b * ld + q]);
  }
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    // both lanes of a pair form the same sum: the lower one's comes first
    const double so = __shfl_xor(s, m, 16), co = __shfl_xor(c, m, 16);
    double a = (l & m) ? so : s;
    c += co;
    neumaier(a, c, (l & m) ? s : so);
    s = a;
  }
  if (l == 0 && q < ld) out[blockIdx.y * ld + q] = pref * (s + c);
}

// sum over k of f(eps_nk) for band_lo <= n <= band_hi, per temperature
__global__ __launch_bounds__(kSigThreads) void density_kernel(int64_t nk, int64_t n2, int nw, const double *__restrict__ eps,
                                                               int blo, int bhi, double mu, int nt, Kts kts,
                                                               double *__restrict__ partials, int64_t chunk) {
  __shared__ double red[kSigThreads / 64][EPH_MAX_TEMPS];
  const int64_t b0 = blockIdx.x * chunk, b1 = min(nk, b0 + chunk);
  double s[EPH_MAX_TEMPS], c[EPH_MAX_TEMPS];
#pragma unroll
  for (int t = 0; t < EPH_MAX_TEMPS; t++) s[t] = c[t] = 0.0;
  for (int64_t k = b0 + threadIdx.x; k < b1; k += kSigThreads)
    for (int n = blo; n <= bhi; n++) {
      const double e = eps[plane_at(k, n, nw, n2)];
#pragma unroll
      for (int t = 0; t < EPH_MAX_TEMPS; t++)
        if (t < nt) neumaier(s[t], c[t], 1.0 / (exp((e - mu) / kts.v[t]) + 1.0));
    }
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
#pragma unroll
  for (int t = 0; t < EPH_MAX_TEMPS; t++) {
    double x = s[t] + c[t];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    if (lane == 0) red[wave][t] = x;
  }
  __syncthreads();
  if (threadIdx.x < EPH_MAX_TEMPS) {
    double x = 0.0;
    for (int w = 0; w < kSigThreads / 64; w++) x += red[w][threadIdx.x];
    partials[blockIdx.x * EPH_MAX_TEMPS + threadIdx.x] = x;
  }
}

__global__ void to_f32_kernel(int64_t n, const double2 *__restrict__ in, float2 *__restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

}  // namespace

hipError_t launch_sigma(int64_t ns, const double *e, const double *v, const double *inv_tau, double mu, int nt,
                        const double *kts_host, double pref, double *partials, int nblk, double *out,
                        hipStream_t st, int n_orders, const double *F) {
  const int64_t chunk = std::max<int64_t>(1, (ns + nblk - 1) / nblk);
  Kts k;
  for (int t = 0; t < EPH_MAX_TEMPS; t++) k.v[t] = t < nt ? kts_host[t] : 1.0;
  const dim3 grid(nblk, nt);
  if (F && n_orders == 1)
    hipLaunchKernelGGL((sigma_kernel<1, true>), grid, dim3(kSigThreads), 0, st, ns, e, v, inv_tau, mu, k, partials, chunk, F);
  else if (!F && n_orders == 1)
    hipLaunchKernelGGL((sigma_kernel<1, false>), grid, dim3(kSigThreads), 0, st, ns, e, v, inv_tau, mu, k, partials, chunk, F);
  else if (!F && n_orders == 3)
    hipLaunchKernelGGL((sigma_kernel<3, false>), grid, dim3(kSigThreads), 0, st, ns, e, v, inv_tau, mu, k, partials, chunk, F);
  else
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(final_kernel, dim3(1, n_orders), dim3(16 * EPH_MAX_TEMPS * 9), 0, st, nblk, EPH_MAX_TEMPS * 9, nt * 9,
                     partials, pref, out);
  return hipGetLastError();
}

hipError_t launch_density(int N, int nw, const double *eps, int blo, int bhi, double mu, int nt,
                          const double *kts_host, double pref, double *partials, int nblk, double *out,
                          hipStream_t st) {
  const int64_t nk = (int64_t)N * N * N;
  const int64_t chunk = std::max<int64_t>(1, (nk + nblk - 1) / nblk);
  Kts k;
  for (int t = 0; t < EPH_MAX_TEMPS; t++) k.v[t] = t < nt ? kts_host[t] : 1.0;
  hipLaunchKernelGGL(density_kernel, dim3(nblk), dim3(kSigThreads), 0, st, nk, (int64_t)N * N, nw, eps, blo, bhi, mu, nt, k,
                     partials, chunk);
  hipLaunchKernelGGL(final_kernel, dim3(1), dim3(64), 0, st, nblk, EPH_MAX_TEMPS, nt, partials, pref, out);
  return hipGetLastError();
}

hipError_t launch_to_f32(int64_t n, const double2 *in, float2 *out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = std::min<int64_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(to_f32_kernel, dim3((unsigned)nb), dim3(256), 0, st, n, in, out);
  return hipGetLastError();
}

}  // namespace eph
