// Small device helpers: fills, a max reduction and the per-call count
// summary (gfx950).  Fills use a kernel rather than hipMemsetAsync so the
// library never records memset nodes if a caller captures its stream.
#include <algorithm>

#include "internal.h"

namespace eph {
namespace {

__global__ void zero_kernel(int64_t n64, unsigned long long *__restrict__ p) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n64) p[i] = 0ull;
}

// max of non-negative doubles through their (monotone) bit patterns; elements
// below cut are set to +inf
__global__ void max_nonneg_kernel(int64_t n, double *__restrict__ x, double cut, unsigned long long *__restrict__ out) {
  __shared__ unsigned long long red[256];
  unsigned long long m = 0ull;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double v = x[i];
    if (v < cut) x[i] = __builtin_huge_val();
    if (v > 0.0) {
      unsigned long long b = (unsigned long long)__double_as_longlong(v);
      m = b > m ? b : m;
    }
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = red[threadIdx.x] > red[threadIdx.x + s] ? red[threadIdx.x] : red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicMax(out, red[0]);
}

// out[1] += sum n_q_valid, out[2] += sum n_terms, out[3] += #(inv_tau[0][s] == 0);
// with kv_counts out[0] += (k,q) pairs, out[4] += vertices
__global__ void summarize_kernel(int64_t ns, const int64_t *__restrict__ st_counts,
                                 const int64_t *__restrict__ kv_counts, const double *__restrict__ inv_tau0,
                                 unsigned long long *__restrict__ out) {
  __shared__ unsigned long long red[5][256];
  unsigned long long v[5] = {0, 0, 0, 0, 0};
  for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < ns; s += (int64_t)gridDim.x * blockDim.x) {
    v[1] += (unsigned long long)st_counts[2 * s];
    v[2] += (unsigned long long)st_counts[2 * s + 1];
    v[3] += inv_tau0[s] == 0.0 ? 1ull : 0ull;
    if (kv_counts) {
      v[0] += (unsigned long long)kv_counts[2 * s];
      v[4] += (unsigned long long)kv_counts[2 * s + 1];
    }
  }
  for (int q = 0; q < 5; q++) red[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s)
      for (int q = 0; q < 5; q++) red[q][threadIdx.x] += red[q][threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < 5 && red[threadIdx.x][0]) atomicAdd(out + threadIdx.x, red[threadIdx.x][0]);
}

struct Kts {
  double v[EPH_MAX_TEMPS];
};

// Element i = (plane, component, point) of a table whose planes hold n2 points
// per component: its two pairs of temperatures in the wave kernel's layout.
__device__ __forceinline__ int64_t pair_at(int64_t i, int64_t n2, int t) {
  return (((i / n2) * 2 + t / 2) * n2 + i % n2) * 2 + t % 2;
}

__global__ void occupation_kernel(int64_t nq, int64_t n2, int nw, int nm, const double *__restrict__ eps,
                                  const double *__restrict__ om, double mu, int nt, Kts kts, double wcut, int rows,
                                  double *__restrict__ occ_f, double *__restrict__ occ_n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int nv = rows ? EPH_MAX_TEMPS : occ_stride(nt);
  for (int t = 0; t < nv; t++) {
    const int64_t at = rows ? i * EPH_MAX_TEMPS + t : nv == 1 ? i : pair_at(i, n2, t);
    if (i < nq * nw) occ_f[at] = t < nt ? 1.0 / (exp((eps[i] - mu) / kts.v[t]) + 1.0) : 0.0;
    if (i < nq * nm) {
      const double w = om[i];
      occ_n[at] = (t < nt && w >= wcut && w > 0.0) ? 1.0 / expm1(w / kts.v[t]) : 0.0;
    }
  }
}

// 16 lanes per group of 16 p of a p3 plane (groups counted from the first p
// of each batch of lines): the range of every band's energies.
__global__ __launch_bounds__(256) void band_range_kernel(int N, int nw, int nlb, int plane_groups,
                                                         const double *__restrict__ eps, float2 *__restrict__ out) {
  const int64_t g = (blockIdx.x * (int64_t)256 + threadIdx.x) >> 4;
  if (g >= (int64_t)N * plane_groups) return;  // whole groups
  const int lane = threadIdx.x & 15;
  const int p3 = (int)(g / plane_groups), c = (int)(g - (int64_t)p3 * plane_groups);
  const int gb = (nlb * N + 15) >> 4, b = c / gb;
  const int ne = min(nlb, N - b * nlb) * N;
  const int64_t n2 = (int64_t)N * N, p = (int64_t)b * nlb * N + min(16 * (c - b * gb) + lane, ne - 1);
  for (int m = 0; m < nw; m++) {
    const double e = eps[(p3 * nw + m) * n2 + p];
    double lo = e, hi = e;
    for (int d = 8; d >= 1; d >>= 1) {
      lo = fmin(lo, __shfl_xor(lo, d, 16));
      hi = fmax(hi, __shfl_xor(hi, d, 16));
    }
    if (lane == 0) out[g * nw + m] = make_float2(__double2float_rd(lo), __double2float_ru(hi));
  }
}

// Record r of point x, component c0 on, into the chunk layout.
template <class R>
__device__ __forceinline__ void put_chunks(const R &r, float4 *__restrict__ out, int64_t plane_comp, int64_t n2, int64_t x) {
  const float4 *src = reinterpret_cast<const float4 *>(&r);
#pragma unroll
  for (int c = 0; c < (int)(sizeof(R) / 16); c++) out[(plane_comp + c) * n2 + x] = src[c];
}

template <int NW, int NT>
__global__ void p_record_kernel(int64_t n, int64_t n2, const double *__restrict__ eps,
                                const double2 *__restrict__ evec, double mu, int nt, Kts kts, float4 *__restrict__ out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;  // element of eps
  if (i >= n) return;
  const int64_t pm = i / n2, x = i % n2;  // plane and band
  PRec<NW, NT> r = {};
#pragma unroll
  for (int j = 0; j < NW; j++) {
    const double2 v = evec[(pm * NW + j) * n2 + x];
    r.v[j] = make_float2((float)v.x, (float)v.y);
  }
  r.e = eps[i];
#pragma unroll
  for (int t = 0; t < NT; t++) r.f[t] = t < nt ? (float)(1.0 / (exp((r.e - mu) / kts.v[t]) + 1.0)) : 0.f;
  put_chunks(r, out, pm * (int64_t)(sizeof(r) / 16), n2, x);
}

template <int NM, int NT>
__global__ void q_record_kernel(int64_t n, int64_t n2, const double *__restrict__ om, const double2 *__restrict__ uu,
                                int nt, Kts kts, double wcut, float4 *__restrict__ out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;  // q
  if (i >= n) return;
  const int64_t pl = i / n2, x = i % n2;
  QRec<NM, NT> r = {};
#pragma unroll
  for (int e = 0; e < NM * NM; e++) {
    const double2 u = uu[(pl * (NM * NM) + e) * n2 + x];
    r.u[e] = make_float2((float)u.x, (float)u.y);
  }
#pragma unroll
  for (int nu = 0; nu < NM; nu++) {
    const double w = om[(pl * NM + nu) * n2 + x];
    r.w[nu] = w >= wcut ? w : __builtin_huge_val();
#pragma unroll
    for (int t = 0; t < NT; t++)
      r.n[nu * NT + t] = (t < nt && w >= wcut && w > 0.0) ? (float)(1.0 / expm1(w / kts.v[t])) : 0.f;
  }
  put_chunks(r, out, pl * (int64_t)(sizeof(r) / 16), n2, x);
}

template <int NM, int NT>
size_t rec_sizes(int nw, int64_t nq, size_t *q_offset) {
  const size_t p = nw == 1   ? sizeof(PRec<1, NT>)
                   : nw == 2 ? sizeof(PRec<2, NT>)
                   : nw == 4 ? sizeof(PRec<4, NT>)
                             : sizeof(PRec<8, NT>);
  *q_offset = p * nw * nq;
  return *q_offset + sizeof(QRec<NM, NT>) * nq;
}

template <int NT>
hipError_t wave_records(int N, int nw, int nm, const double *eps, const double *om, const double2 *evec,
                        const double2 *uu, double mu, int nt, const Kts &k, double wcut, void *out, hipStream_t st) {
  const int64_t n2 = (int64_t)N * N, nq = n2 * N;
  size_t qo;
  (void)wave_rec_bytes(nw, nm, nt, nq, &qo);
  const dim3 gp((unsigned)((nq * nw + 255) / 256)), gq((unsigned)((nq + 255) / 256));
  float4 *p = static_cast<float4 *>(out), *q = p + qo / 16;
#define EPH_PREC(NW_) \
  if (nw == NW_) hipLaunchKernelGGL((p_record_kernel<NW_, NT>), gp, dim3(256), 0, st, nq * nw, n2, eps, evec, mu, nt, k, p);
  EPH_PREC(1)
  EPH_PREC(2)
  EPH_PREC(4)
  EPH_PREC(8)
#undef EPH_PREC
  if (nm == 3) hipLaunchKernelGGL((q_record_kernel<3, NT>), gq, dim3(256), 0, st, nq, n2, om, uu, nt, k, wcut, q);
  else hipLaunchKernelGGL((q_record_kernel<6, NT>), gq, dim3(256), 0, st, nq, n2, om, uu, nt, k, wcut, q);
  return hipGetLastError();
}

}  // namespace

int wave_batch_lines(int N) {
  const int nb = (N + kWaveLines - 1) / kWaveLines;
  return (N + nb - 1) / nb;  // evened out over the batches
}

// Planes per workgroup: enough for about 20000 q (10000 in FP64, whose tables
// are twice as large), so that what a workgroup does once (tables, reductions)
// stays small beside them, while the states still make 8192 workgroups.  More
// q per workgroup cost more than they save, the q-side tables of the planes in
// flight no longer fit the L2s (Al-like, FP32, 71^3: 387 ms at 20000 q, 407 at
// 10000, 402 at 40000; FP64, 100^3, 4 % of the states: 185 ms at 10000, 194 at
// 20000, 205 at 40000).
int wave_slab_planes(int N, int64_t ns, bool fp64) {
  const int64_t n2 = (int64_t)N * N, p = std::min(((fp64 ? 10000 : 20000) + n2 / 2) / n2, ns * N / 8192);
  return (int)std::max<int64_t>(1, std::min<int64_t>(p, N));
}

int wave_plane_groups(int N) {
  const int nlb = wave_batch_lines(N), full = N / nlb, rest = N - full * nlb;
  return full * ((nlb * N + 15) / 16) + (rest * N + 15) / 16;
}

hipError_t launch_band_ranges(int N, int nw, const double *eps, float2 *out, hipStream_t st) {
  const int pc = wave_plane_groups(N);
  hipLaunchKernelGGL(band_range_kernel, dim3((unsigned)(((int64_t)N * pc + 15) / 16)), dim3(256), 0, st, N, nw,
                     wave_batch_lines(N), pc, eps, out);
  return hipGetLastError();
}

size_t wave_rec_bytes(int nw, int nm, int nt, int64_t nq, size_t *q_offset) {
  if (occ_stride(nt) == 1) return nm == 3 ? rec_sizes<3, 1>(nw, nq, q_offset) : rec_sizes<6, 1>(nw, nq, q_offset);
  return nm == 3 ? rec_sizes<3, EPH_MAX_TEMPS>(nw, nq, q_offset) : rec_sizes<6, EPH_MAX_TEMPS>(nw, nq, q_offset);
}

hipError_t launch_wave_records(int N, int nw, int nm, const double *eps, const double *om, const double2 *evec,
                               const double2 *uu, double mu, int nt, const double *kts_host, double wcut, void *out,
                               hipStream_t st) {
  Kts k;
  for (int t = 0; t < EPH_MAX_TEMPS; t++) k.v[t] = t < nt ? kts_host[t] : 1.0;
  if (occ_stride(nt) == 1) return wave_records<1>(N, nw, nm, eps, om, evec, uu, mu, nt, k, wcut, out, st);
  return wave_records<EPH_MAX_TEMPS>(N, nw, nm, eps, om, evec, uu, mu, nt, k, wcut, out, st);
}

hipError_t launch_occupations(int N, int nw, int nm, const double *eps, const double *om, double mu, int nt,
                              const double *kts_host, double wcut, bool rows, double *occ_f, double *occ_n,
                              hipStream_t st) {
  Kts k;
  for (int t = 0; t < EPH_MAX_TEMPS; t++) k.v[t] = t < nt ? kts_host[t] : 1.0;
  const int64_t n2 = (int64_t)N * N, nq = n2 * N, n = nq * (nw > nm ? nw : nm);
  hipLaunchKernelGGL(occupation_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, nq, n2, nw, nm, eps, om,
                     mu, nt, k, wcut, rows ? 1 : 0, occ_f, occ_n);
  return hipGetLastError();
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t st) {
  int64_t n64 = (int64_t)((bytes + 7) / 8);
  if (n64 <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n64 + 255) / 256)), dim3(256), 0, st, n64,
                     static_cast<unsigned long long *>(p));
  return hipGetLastError();
}

hipError_t launch_max_nonneg(int64_t n, double *x, double cut, unsigned long long *out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(max_nonneg_kernel, dim3((unsigned)blocks), dim3(256), 0, st, n, x, cut, out);
  return hipGetLastError();
}

hipError_t launch_summarize(int64_t ns, const int64_t *st_counts, const int64_t *kv_counts, const double *inv_tau0,
                            unsigned long long *out, hipStream_t st) {
  if (ns <= 0) return hipSuccess;
  int64_t blocks = (ns + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(summarize_kernel, dim3((unsigned)blocks), dim3(256), 0, st, ns, st_counts, kv_counts,
                     inv_tau0, out);
  return hipGetLastError();
}

}  // namespace eph
