// Online linear estimators (Sec. 3.3.1) for gfx950: ordinary least-squares
// fits refined as samples are fed back.  The state of an estimator set is the
// sufficient statistics of every fit, in device memory, float64:
//   gram[e][F][F] = sum x x^T,  mom[e][F] = sum x y,  count[e].
//
// est_accumulate  a group of lanes per estimator (sized to the batch's average
//                 samples per estimator): its lanes stride over the estimator's
//                 samples (grouped by estimator), sum in registers, and reduce
//                 across the group in a fixed order (results do not depend on
//                 scheduling), then add to the state.  Bound: HBM, once the
//                 reduction is cheap: 20 sums of 64 lanes through LDS shuffles
//                 cost more than reading the samples, so a group is at most
//                 16 lanes (a DPP row: rotations on the VALU) while that
//                 fills the chip (8,388,608 samples of 65,536 five-feature
//                 estimators, 435.7 MB: 189 us with groups of 64, 120 us with
//                 16, 3.6 TB/s).
// est_solve       one lane per estimator: Cholesky factorisation of the Gram
//                 matrix and two triangular solves for the coefficients, all
//                 in registers, a wave to a block.  Bound: latency of the
//                 strided loads and of the divisions and roots in turn (the
//                 same estimators: 21 us with indexed arrays, 6.3 us).
// est_predict     one lane per query: integer microseconds for the simulator;
//                 a query's features and coefficients in flight together.
//                 Bound: the gathered coefficients' lines (1,048,576 queries
//                 40 us with one feature after the other, 23 us).
#include <climits>
#include <cmath>

#include "ss_internal.h"

struct ss_est {
  int device = 0;
  int64_t n_est = 0, n_feat = 0;
  double *gram = nullptr, *mom = nullptr;  // [n_est][F][F], [n_est][F]
  int64_t *count = nullptr;                // [n_est]
};

namespace {

constexpr int kWave = 64;
constexpr double kPivotRtol = 1e-12;  // relative pivot below which a Gram matrix is singular

// Sum of v over each aligned group of kL lanes, in every lane of the group.
// Within a row of 16 lanes by rotation (a DPP move on the VALU), beyond that
// through the LDS permute network.
template <int kCtrl>
__device__ __forceinline__ double row_move(double v) {
  const uint64_t x = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, kCtrl, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), kCtrl, 0xF, 0xF, false);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

template <int kL>
__device__ __forceinline__ double group_sum(double v) {
  // quad_perm {1,0,3,2} and {2,3,0,1}; row_half_mirror and row_mirror, whose
  // partners hold the other half's sum; then across rows
  if (kL >= 2) v += row_move<0xB1>(v);
  if (kL >= 4) v += row_move<0x4E>(v);
  if (kL >= 8) v += row_move<0x141>(v);
  if (kL >= 16) v += row_move<0x140>(v);
  if (kL >= 32) v += __shfl_xor(v, 16, kWave);
  if (kL >= 64) v += __shfl_xor(v, 32, kWave);
  return v;
}

// kL lanes per estimator (a power of two dividing 64): each wave serves
// 64 / kL estimators, lane t of a group takes samples t, t + kL, ...; the
// group then reduces by a fixed butterfly, so the sums do not depend on how
// the device schedules the work.
template <int F, int kL>
__global__ __launch_bounds__(kWave) void est_accumulate(int64_t n_est, const int64_t *__restrict__ ptr,
                                                        int64_t n_samples, const double *__restrict__ x,
                                                        const double *__restrict__ y, double *__restrict__ gram,
                                                        double *__restrict__ mom, int64_t *__restrict__ count) {
  const int lane = threadIdx.x, t = lane & (kL - 1);
  const int64_t e = (int64_t)blockIdx.x * (kWave / kL) + lane / kL;
  const bool live = e < n_est;
  const int64_t ec = live ? e : n_est - 1;
  // the estimator's samples, clamped to [0, n_samples)
  const int64_t s0 = min(max(ptr[ec], (int64_t)0), n_samples);
  const int64_t s1 = live ? min(max(ptr[ec + 1], s0), n_samples) : s0;
  double g[F * (F + 1) / 2], m[F];
#pragma unroll
  for (int i = 0; i < F * (F + 1) / 2; ++i) g[i] = 0.0;
#pragma unroll
  for (int i = 0; i < F; ++i) m[i] = 0.0;
  for (int64_t s = s0 + t; s < s1; s += kL) {
    double v[F];
#pragma unroll
    for (int i = 0; i < F; ++i) v[i] = x[s * F + i];
    const double yt = y[s];
    int k = 0;
#pragma unroll
    for (int i = 0; i < F; ++i) {
      m[i] = fma(v[i], yt, m[i]);
#pragma unroll
      for (int j = i; j < F; ++j, ++k) g[k] = fma(v[i], v[j], g[k]);
    }
  }
  double *ge = gram + ec * F * F, *me = mom + ec * F;
  const bool writer = live && t == 0;
  int k = 0;
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const double mi = group_sum<kL>(m[i]);
    if (writer) me[i] += mi;
#pragma unroll
    for (int j = i; j < F; ++j, ++k) {
      const double gij = group_sum<kL>(g[k]);
      if (writer) {
        ge[i * F + j] += gij;
        if (j != i) ge[j * F + i] += gij;
      }
    }
  }
  if (writer) count[ec] += s1 - s0;
}

template <int F>
__global__ __launch_bounds__(kWave) void est_solve(int64_t n_est, const double *__restrict__ gram,
                                                   const double *__restrict__ mom, const int64_t *__restrict__ count,
                                                   double *__restrict__ coef, int32_t *__restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * kWave + threadIdx.x;
  if (e >= n_est) return;
  double L[F][F], z[F], beta[F];
  const double *a = gram + e * F * F, *b = mom + e * F;
#pragma unroll
  for (int i = 0; i < F; ++i) {
    z[i] = b[i];
#pragma unroll
    for (int j = 0; j <= i; ++j) L[i][j] = a[i * F + j];
  }
  int st = count[e] < F ? SS_EST_UNDERDETERMINED : SS_EST_FITTED;
#pragma unroll
  for (int j = 0; j < F; ++j) {
    const double ajj = L[j][j];
    double d = ajj;
#pragma unroll
    for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
    if (st == SS_EST_FITTED && (!(d > kPivotRtol * fabs(ajj)) || ajj <= 0.0)) st = SS_EST_SINGULAR;
    L[j][j] = sqrt(d);  // (what follows a refused pivot is not used)
#pragma unroll
    for (int i = j + 1; i < F; ++i) {
      double s = L[i][j];
#pragma unroll
      for (int k = 0; k < j; ++k) s -= L[i][k] * L[j][k];
      L[i][j] = s / L[j][j];
    }
  }
#pragma unroll
  for (int i = 0; i < F; ++i) {  // L z = mom
    double s = z[i];
#pragma unroll
    for (int k = 0; k < i; ++k) s -= L[i][k] * z[k];
    z[i] = s / L[i][i];
  }
#pragma unroll
  for (int i = F - 1; i >= 0; --i) {  // L^T beta = z
    double s = z[i];
#pragma unroll
    for (int k = i + 1; k < F; ++k) s -= L[k][i] * beta[k];
    beta[i] = s / L[i][i];
  }
#pragma unroll
  for (int i = 0; i < F; ++i) coef[e * F + i] = st == SS_EST_FITTED ? beta[i] : 0.0;
  status[e] = st;
}

template <int F>
__global__ __launch_bounds__(256) void est_predict(const double *__restrict__ coef, int64_t n_est,
                                                   const int32_t *__restrict__ est_of, const double *__restrict__ x,
                                                   int64_t M, int64_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  const int32_t e = est_of[i];
  if (e < 0 || e >= n_est) {
    out[i] = 0;  // unknown estimator
    return;
  }
  double v[F], c[F];
#pragma unroll
  for (int j = 0; j < F; ++j) {
    v[j] = x[i * F + j];
    c[j] = coef[(int64_t)e * F + j];
  }
  // products and sums rounded one by one, in feature order (no fused
  // multiply-add): the integer decision below is then reproducible bit for bit
  double t = 0.0;
#pragma unroll
  for (int j = 0; j < F; ++j) t = __dadd_rn(t, __dmul_rn(v[j], c[j]));
  const double r = ceil(t);
  out[i] = !(r < 4.611686018427388e18) ? 0 : r < 1.0 ? 1 : (int64_t)r;  // not finite or >= 2^62: 0
}

int hip_fail(hipError_t err, const char *what) {
  return ss_set_error(err == hipErrorOutOfMemory ? SS_ERR_OOM : SS_ERR_DEVICE,
                      std::string(what) + ": " + hipGetErrorString(err));
}

template <int F, int kL>
void launch_group(const ss_est *E, const int64_t *ptr, int64_t S, const double *x, const double *y,
                  hipStream_t stream) {
  constexpr int64_t per = kWave / kL;  // estimators per wave
  hipLaunchKernelGGL((est_accumulate<F, kL>), dim3((unsigned)((E->n_est + per - 1) / per)), dim3(kWave), 0, stream,
                     E->n_est, ptr, S, x, y, E->gram, E->mom, E->count);
}

// Lanes per estimator from the average samples per estimator of the batch
// (4 .. 16, so that most lanes have a sample).  32 and 64 for batches of fewer
// estimators, whose groups of 16 would leave the chip's waves idle, and the
// more estimators the longer the sums that outweigh the wider reduction; that
// grows with the features, so the lines lie at fewer estimators for more of
// them.  Measured, 16, 32 and 64 lanes in us: 2,048 estimators of three
// features with 1,000 samples each 26.9, 17.0 and 14.5, with 4,000 129, 66 and
// 41; 4,096 with 4,000 155, 98 and 93; 6,000 with 1,500 60, 44 and 51; 8,192
// with 1,500 76, 71 and 73, with 400 19.3, 20.8 and 22.7; of eight features
// 2,048 with 1,000 39, 32 and 35, 6,000 with 800 66, 69 and 85; of five 8,192
// with 1,000 73, 76 and 79.
template <int F>
void launch_accumulate(const ss_est *E, const int64_t *ptr, int64_t S, const double *x, const double *y,
                       hipStream_t stream) {
  const int64_t avg = S / E->n_est;
  const int64_t n = E->n_est;
  if (avg >= 48 && (n < 2048 || (avg >= 600 && n * F < 12288) || (avg >= 3000 && n < 6144)))
    launch_group<F, 64>(E, ptr, S, x, y, stream);
  else if (avg >= 24 && (n < 4096 || (avg >= 1000 && n < 8192 && n * F < 40960) || (avg >= 1500 && n < 12288)))
    launch_group<F, 32>(E, ptr, S, x, y, stream);
  else if (avg >= 12)
    launch_group<F, 16>(E, ptr, S, x, y, stream);
  else if (avg >= 6)
    launch_group<F, 8>(E, ptr, S, x, y, stream);
  else
    launch_group<F, 4>(E, ptr, S, x, y, stream);
}

template <int F>
void launch_solve(const ss_est *E, double *coef, int32_t *status, hipStream_t stream) {
  hipLaunchKernelGGL(est_solve<F>, dim3((unsigned)((E->n_est + kWave - 1) / kWave)), dim3(kWave), 0, stream, E->n_est, E->gram,
                     E->mom, E->count, coef, status);
}

template <int F>
void launch_predict(const double *coef, int64_t n_est, const int32_t *est_of, const double *x, int64_t M,
                    int64_t *out, hipStream_t stream) {
  hipLaunchKernelGGL(est_predict<F>, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, stream, coef, n_est, est_of, x,
                     M, out);
}

}  // namespace

int ss_run_est_create(int64_t n_est, int64_t n_feat, ss_est **out) {
  auto *E = new ss_est();
  E->n_est = n_est;
  E->n_feat = n_feat;
  hipError_t err = hipGetDevice(&E->device);
  const size_t g = (size_t)n_est * n_feat * n_feat * sizeof(double), m = (size_t)n_est * n_feat * sizeof(double),
               c = (size_t)n_est * sizeof(int64_t);
  void *mem = nullptr;
  if (err == hipSuccess) err = hipMalloc(&mem, g + m + c + 8);
  if (err == hipSuccess) err = hipMemset(mem, 0, g + m + c + 8);
  if (err == hipSuccess) err = hipDeviceSynchronize();
  if (err != hipSuccess) {
    if (mem) (void)hipFree(mem);
    delete E;
    return hip_fail(err, "allocating the estimator state");
  }
  E->gram = static_cast<double *>(mem);
  E->mom = E->gram + (size_t)n_est * n_feat * n_feat;
  E->count = reinterpret_cast<int64_t *>(E->mom + (size_t)n_est * n_feat);
  *out = E;
  return SS_OK;
}

void ss_run_est_free(ss_est *E) {
  int prev = 0;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(E->device);
  (void)hipDeviceSynchronize();
  (void)hipFree(E->gram);
  (void)hipSetDevice(prev);
  delete E;
}

int ss_run_est_info(const ss_est *E, int64_t *n_est, int64_t *n_feat, int *device) {
  if (n_est) *n_est = E->n_est;
  if (n_feat) *n_feat = E->n_feat;
  if (device) *device = E->device;
  return SS_OK;
}

int ss_run_est_add(const ss_est *E, const int64_t *ptr, int64_t S, const double *x, const double *y,
                   hipStream_t stream) {
  if (E->n_est == 0) return SS_OK;
  using L = void (*)(const ss_est *, const int64_t *, int64_t, const double *, const double *, hipStream_t);
  static const L table[SS_EST_MAX_FEAT] = {launch_accumulate<1>, launch_accumulate<2>, launch_accumulate<3>,
                                           launch_accumulate<4>, launch_accumulate<5>, launch_accumulate<6>,
                                           launch_accumulate<7>, launch_accumulate<8>};
  SsTimingRec *t = ss_timing_start(SS_KERNEL_ESTIMATOR, stream);
  table[E->n_feat - 1](E, ptr, S, x, y, stream);
  ss_timing_stop(t, stream);
  const hipError_t err = hipGetLastError();
  return err == hipSuccess ? SS_OK : hip_fail(err, "est_accumulate launch");
}

int ss_run_est_solve(const ss_est *E, double *coef, int32_t *status, hipStream_t stream) {
  if (E->n_est == 0) return SS_OK;
  using L = void (*)(const ss_est *, double *, int32_t *, hipStream_t);
  static const L table[SS_EST_MAX_FEAT] = {launch_solve<1>, launch_solve<2>, launch_solve<3>, launch_solve<4>,
                                           launch_solve<5>, launch_solve<6>, launch_solve<7>, launch_solve<8>};
  SsTimingRec *t = ss_timing_start(SS_KERNEL_ESTIMATOR, stream);
  table[E->n_feat - 1](E, coef, status, stream);
  ss_timing_stop(t, stream);
  const hipError_t err = hipGetLastError();
  return err == hipSuccess ? SS_OK : hip_fail(err, "est_solve launch");
}

int ss_run_est_predict(const double *coef, int64_t n_est, int64_t n_feat, const int32_t *est_of, const double *x,
                       int64_t M, int64_t *out, hipStream_t stream) {
  if (M == 0) return SS_OK;
  using L = void (*)(const double *, int64_t, const int32_t *, const double *, int64_t, int64_t *, hipStream_t);
  static const L table[SS_EST_MAX_FEAT] = {launch_predict<1>, launch_predict<2>, launch_predict<3>, launch_predict<4>,
                                           launch_predict<5>, launch_predict<6>, launch_predict<7>, launch_predict<8>};
  SsTimingRec *t = ss_timing_start(SS_KERNEL_ESTIMATOR, stream);
  table[n_feat - 1](coef, n_est, est_of, x, M, out, stream);
  ss_timing_stop(t, stream);
  const hipError_t err = hipGetLastError();
  return err == hipSuccess ? SS_OK : hip_fail(err, "est_predict launch");
}
