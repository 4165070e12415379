// Re transform fused with the j -> n band rotation (gfx950):
//   X_s(Rp, mu, i) = sum_{Re, j} g_ij^mu(Re, Rp) e^{i k_s.Re} V_{j n_s}(k_s)
// i.e. the innermost bracket (g P^el(k) U^+(k)) of the q-batch order of
// Sec. III.C, evaluated per initial state s = (n, k).  It is a complex GEMM
// X[s][col] = sum_kk B[s][kk] W[kk][col] with kk = (Re, j) and
// col = (Rp, mu, i); the state-side operand B (a phase times one
// eigenvector component) is generated on the fly into LDS.
//
// What bounds it: the matrix cores.  FP64 products run there at the vector
// units' rate, FP32 ones at twice that of single (non-packed) instructions,
// and both read a sixteenth of the LDS per operation.  A
// workgroup makes a 64 x 64 tile of X, each of its four waves 2 x 2 blocks of
// 16 x 16 complex elements, four real products per complex one.  A thread's
// elements of B share their state and (with 4 or 8 bands) their R vector, so
// one phase, looked up in LDS by 32-bit arithmetic, serves four of them; with
// 64-bit remainders per element, generating B took as long as the products.
// FP64, 2651 states of 8 bands, 512 x 216 cells: 14.8 ms, 61 TFLOP/s of the
// 73 of a large product (28 ms with vector operations); FP32, 156516 states
// of 4 bands, 216 x 216 cells: 24.5 ms, 114 TFLOP/s of 151 (51.7).
#include "dev_util.h"
#include "internal.h"

namespace eph {
namespace {

constexpr int BM = 64, BN = 64, BK = 16;
constexpr int kSlots = BM * BK / 256;  // elements of B per thread and step, consecutive in kk

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// 16 x 16 x 4 products: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
// and holds column l % 16 of D, in register r its row(l / 16, r)
template <class T>
struct Mat;
template <>
struct Mat<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mat<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int row(int g, int r) { return g + 4 * r; }
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// T = accumulation/operand type (double for the FP64 form, float for FP32).
template <class T, int NW>
__global__ __launch_bounds__(256) void xform_kernel(int64_t ns, const int32_t *__restrict__ sk,
                                                    const int32_t *__restrict__ sn, int N, int64_t n2, int nre,
                                                    const int *__restrict__ re, int ncol, int64_t nrow_blocks,
                                                    int64_t nblocks, const typename V2<T>::t *__restrict__ wt,
                                                    const double2 *__restrict__ evec,
                                                    const double2 *__restrict__ tab,
                                                    typename V2<T>::t *__restrict__ X) {
  using C2 = typename V2<T>::t;
  using MM = Mat<T>;
  constexpr int PH = NW >= kSlots ? 1 : kSlots / NW;  // R vectors of a thread's elements
  __shared__ C2 sB[BM][BK + 1];
  __shared__ C2 sW[BK][BN];
  extern __shared__ __align__(16) double2 sTab[];
  // consecutive workgroups go round-robin to the 8 XCDs: give each a run of
  // tiles along the states, which read the same columns of W
  const int64_t per_xcd = (nblocks + 7) / 8;
  const int64_t blk = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if ((int64_t)(blockIdx.x / 8) >= per_xcd || blk >= nblocks) return;  // workgroup-uniform
  const int64_t s0 = blk % nrow_blocks * BM;
  const int c0 = (int)(blk / nrow_blocks) * BN;
  const int K = nre * NW;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  for (int t = tid; t < N; t += 256) sTab[t] = tab[t];

  // the thread's share of B: state sl, elements kq .. kq + kSlots - 1 of a step
  const int sl = tid / (BK / kSlots), kq = tid % (BK / kSlots) * kSlots;
  const bool has_state = s0 + sl < ns;
  double2 v[kSlots];
  int k1 = 0, k2 = 0, k3 = 0;
#pragma unroll
  for (int q = 0; q < kSlots; q++) v[q] = make_double2(0.0, 0.0);
  if (has_state) {
    const int k = sk[s0 + sl], n = sn[s0 + sl];
    k1 = k % N;
    k2 = (k / N) % N;
    k3 = k / (N * N);
#pragma unroll
    for (int q = 0; q < kSlots; q++) v[q] = evec[plane_at(k, n * NW + (kq + q) % NW, NW * NW, n2)];
  }
  const float inv_n = 1.0f / (float)N;

  int rv[PH][3];
  C2 w[BK * BN / 256];
  auto load_step = [&](int kk0) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < PH; h++) {
      const int r = min((kk0 + kq) / NW + h, nre - 1);
#pragma unroll
      for (int a = 0; a < 3; a++) rv[h][a] = re[3 * r + a];
    }
#pragma unroll
    for (int i = 0; i < BK * BN / 256; i++) {
      const int kk = kk0 + (tid + 256 * i) / BN, c = c0 + (tid + 256 * i) % BN;
      w[i] = (kk < K && c < ncol) ? wt[(size_t)kk * ncol + c] : mk<T>(0, 0);
    }
  };

  typename MM::acc xr[2][2], xi[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) xr[i][j] = xi[i][j] = typename MM::acc{0, 0, 0, 0};

  load_step(0);
  for (int kk0 = 0; kk0 < K; kk0 += BK) {
    __syncthreads();  // the last step's products (the first time: the phase table)
#pragma unroll
    for (int h = 0; h < PH; h++) {
      // k . R mod N: below 3 N^2 < 2^20, so the float quotient is off by one at most
      const int a = k1 * imod(rv[h][0], N) + k2 * imod(rv[h][1], N) + k3 * imod(rv[h][2], N);
      int m = a - (int)((float)a * inv_n) * N;
      m += (m < 0) ? N : 0;
      m -= (m >= N) ? N : 0;
      const double2 ph = sTab[m];
#pragma unroll
      for (int q = h * (kSlots / PH); q < (h + 1) * (kSlots / PH); q++) {
        double2 b = cmul(ph, v[q]);  // in FP64, then T
        if (kk0 + kq + q >= K) b = make_double2(0.0, 0.0);
        sB[sl][kq + q] = mk<T>((T)b.x, (T)b.y);
      }
    }
#pragma unroll
    for (int i = 0; i < BK * BN / 256; i++) sW[(tid + 256 * i) / BN][(tid + 256 * i) % BN] = w[i];
    __syncthreads();
    if (kk0 + BK < K) load_step(kk0 + BK);  // while the products run
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      C2 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; i++) {
        a[i] = sB[wm + 16 * i + li][ks + lg];
        b[i] = sW[ks + lg][wn + 16 * i + li];
      }
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
          xr[i][j] = MM::mul(a[i].x, b[j].x, xr[i][j]);
          xi[i][j] = MM::mul(a[i].x, b[j].y, xi[i][j]);
          xr[i][j] = MM::mul(-a[i].y, b[j].y, xr[i][j]);
          xi[i][j] = MM::mul(a[i].y, b[j].x, xi[i][j]);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int col = c0 + wn + 16 * j + li;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int64_t s = s0 + wm + 16 * i + MM::row(lg, r);
        if (s < ns && col < ncol) X[s * ncol + col] = mk<T>(xr[i][j][r], xi[i][j][r]);
      }
    }
}

template <class T>
hipError_t launch(int64_t ns, const int32_t *sk, const int32_t *sn, int N, int64_t n2, int nw, int nre, const int *re, int ncol,
                  const typename V2<T>::t *wt, const double2 *evec, const double2 *tab, typename V2<T>::t *X,
                  hipStream_t st) {
  if (ns <= 0) return hipSuccess;
  const int64_t nrow = (ns + BM - 1) / BM, nblocks = nrow * ((ncol + BN - 1) / BN);
  const dim3 grid((unsigned)((nblocks + 7) / 8 * 8));
  const size_t sh = sizeof(double2) * N;
#define EPH_XF(NW)                                                                                                  \
  case NW:                                                                                                          \
    hipLaunchKernelGGL((xform_kernel<T, NW>), grid, dim3(256), sh, st, ns, sk, sn, N, n2, nre, re, ncol, nrow,     \
                       nblocks, wt, evec, tab, X);                                                                  \
    return hipGetLastError();
  switch (nw) {
    EPH_XF(1)
    EPH_XF(2)
    EPH_XF(4)
    EPH_XF(8)
  }
#undef EPH_XF
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_xform64(int64_t ns, const int32_t *sk, const int32_t *sn, int N, int64_t n2, int nw, int nre, const int *re,
                          int ncol, const double2 *wt, const double2 *evec, const double2 *tab, double2 *X,
                          hipStream_t st) {
  return launch<double>(ns, sk, sn, N, n2, nw, nre, re, ncol, wt, evec, tab, X, st);
}

hipError_t launch_xform32(int64_t ns, const int32_t *sk, const int32_t *sn, int N, int64_t n2, int nw, int nre, const int *re,
                          int ncol, const float2 *wt, const double2 *evec, const double2 *tab, float2 *X,
                          hipStream_t st) {
  return launch<float>(ns, sk, sn, N, n2, nw, nre, re, ncol, wt, evec, tab, X, st);
}

}  // namespace eph
