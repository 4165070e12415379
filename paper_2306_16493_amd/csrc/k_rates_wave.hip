// SERTA scattering rates, wave form: shape selection and dispatch to the
// per-(precision, modes) instances of the kernel in rates_wave.h, and the sums
// over the slabs of a launch.
#include "internal.h"

namespace eph {
namespace wave {
template <class T, int NM, int MODE>
hipError_t dispatch_nm(const RatesArgs &a, hipStream_t st);
extern template hipError_t dispatch_nm<double, 3, kRates>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<double, 6, kRates>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<float, 3, kRates>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<float, 6, kRates>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<double, 3, kCount>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<double, 6, kCount>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<double, 3, kEmit>(const RatesArgs &, hipStream_t);
extern template hipError_t dispatch_nm<double, 6, kEmit>(const RatesArgs &, hipStream_t);
}  // namespace wave

namespace {

// blockIdx.y: a temperature or one of the four counters
__global__ void add_slabs_kernel(RatesArgs a) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= a.ns_launch) return;
  const int64_t s = a.s_lo + i;
  const int np = a.slab_hi - a.slab_lo, t = blockIdx.y, c = t - a.nt;
  if (c < 0) {
    double *dst = a.inv_tau + (int64_t)t * a.ns_total + s;
    double v = a.slab_lo == 0 ? 0.0 : *dst;
#pragma unroll 8
    for (int j = 0; j < np; j++) v += a.part_tau[((int64_t)j * a.nt + t) * a.ns_total + s];
    *dst = v;
  } else {
    int64_t *dst = (c < 2 ? a.st_counts : a.kv_counts - 2) + 2 * s + c;
    int64_t v = a.slab_lo == 0 ? 0 : *dst;
#pragma unroll 8
    for (int j = 0; j < np; j++) v += a.part_cnt[((int64_t)j * a.ns_total + s) * 4 + c];
    *dst = v;
    if (c == 0 && a.g_slot) a.g_cursor[s] += a.g_slot[(int64_t)np * a.ns_total + s];
  }
}

__global__ void slab_counts_kernel(RatesArgs a, int total) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= a.ns_launch) return;
  const int64_t s = a.s_lo + i;
  const int np = a.slab_hi - a.slab_lo;
  int64_t run = 0;
  for (int j = 0; j < np; j++) {
    int64_t *p = a.g_slot + (int64_t)j * a.ns_total + s;
    const int64_t c = *p;
    if (!total) *p = run;
    run += c;
  }
  if (total) a.g_cursor[s] += run;
  else a.g_slot[(int64_t)np * a.ns_total + s] = run;
}

}  // namespace

hipError_t launch_add_slabs(const RatesArgs &a, hipStream_t st) {
  if (a.ns_launch <= 0) return hipSuccess;
  hipLaunchKernelGGL(add_slabs_kernel, dim3((unsigned)((a.ns_launch + 255) / 256), a.nt + 4), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_slab_counts(const RatesArgs &a, int total, hipStream_t st) {
  if (a.ns_launch <= 0) return hipSuccess;
  hipLaunchKernelGGL(slab_counts_kernel, dim3((unsigned)((a.ns_launch + 255) / 256)), dim3(256), 0, st, a, total);
  return hipGetLastError();
}

// Shapes served by the wave kernel: a cubic Rp box of edge 4 or
// 6 and final-state lines of at most 2048 energies (N * n_wann).  Returns
// the states per group, 0 when the shape is not served.
int rates_wave_group(int nw, int nm, RpBox box, int N, int precision) {
  const bool cube = box.n[0] == box.n[1] && box.n[1] == box.n[2] && (box.n[0] == 4 || box.n[0] == 6);
  if (!cube || N * nw > kMaxLine) return 0;
  (void)precision;
  if (nm == 3 && (nw == 1 || nw == 2 || nw == 4)) return 2;
  if (nm == 3 && nw == 8) return 1;
  if (nm == 6 && (nw == 1 || nw == 2)) return 2;
  if (nm == 6 && (nw == 4 || nw == 8)) return 1;
  return 0;
}

// mode kCount / kEmit (transition rates) are FP64 only.
hipError_t launch_rates_wave(int precision, const RatesArgs &a, hipStream_t st, int mode) {
  if (a.ns_launch <= 0) return hipSuccess;
  const bool m3 = a.nm == 3;
  if (mode == kCount) {
    if (precision != EPH_FP64) return hipErrorNotSupported;
    return m3 ? wave::dispatch_nm<double, 3, kCount>(a, st) : wave::dispatch_nm<double, 6, kCount>(a, st);
  }
  if (mode == kEmit) {
    if (precision != EPH_FP64) return hipErrorNotSupported;
    return m3 ? wave::dispatch_nm<double, 3, kEmit>(a, st) : wave::dispatch_nm<double, 6, kEmit>(a, st);
  }
  if (precision == EPH_FP64) return m3 ? wave::dispatch_nm<double, 3, kRates>(a, st) : wave::dispatch_nm<double, 6, kRates>(a, st);
  return m3 ? wave::dispatch_nm<float, 3, kRates>(a, st) : wave::dispatch_nm<float, 6, kRates>(a, st);
}

}  // namespace eph
