// k_grpo.hip — the senior-only GRPO loss pieces over a batch of tandem
// rollouts (section 3.4, the L_TRL equation; Algorithm 1's update half).
//
// Per rollout s = j G + i: the group-relative advantage of its binary reward,
// normalised by the sample standard deviation of the group's G rewards
// (+1e-6).  Per position t < length[s] that the senior emitted (owner != 0):
// rho = exp(logp_new - logp_old) and GRPO's clipped term
// min(rho A, clip(rho, 1 - eps, 1 + eps) A).  The loss is minus the mean of
// those terms over every masked position of the batch; its gradient with
// respect to logp_new is -rho A / N where the unclipped term is the minimum
// and 0 elsewhere (junior positions, positions past the length, clipped
// terms).
//
// Two launches, streaming over the [S][T] arenas, with nothing exchanged inside
// a launch.  The first takes a workgroup per rollout: advantage, masked count,
// the sum of its terms and -rho A as the gradient before its division by N.  The
// second, by the batch's masked count N = the sum of the rollouts' counts,
// divides the gradient and (its first workgroup) sums the rollouts' terms in
// double in a fixed order, so the loss is deterministic.  The gradient is read and
// written once more than with a count pass ahead of everything, but that pass
// needed a ticket to find the last partial sum, and its release and acquire in
// every workgroup were most of the time.  Both launches, 128 rollouts of at most
// 3000 positions: 18.4 -> 7.8 us.  Calls in a row, that kernel pair / these: 128 x 3000
// 18.3 / 16.9 us, 512 x 4096 58.9 / 17.0 (both bound by the host's 17 us), 2048 x 4096
// 242 / 41, 8 rows of a million 1251 / 269.
#include <mutex>

#include "common.h"
#include "kernels.h"

namespace tandem {
namespace {

constexpr int kGrpoNT = 256;                 // threads of the second launch
constexpr int kGrpoPer = 8;                  // gradient entries per thread there

// arena rows start at any multiple of their element size
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_any __attribute__((aligned(1), may_alias));

// One workgroup per rollout, four positions per thread and pass.  Bound by the
// latency of one chain (lengths and authorship, log-probs, sums): a row of up to
// 4 NT positions is one pass, whose loads are issued together.
template <int NT>
__global__ __launch_bounds__(NT) void grpo_terms_kernel(GrpoArgs a) {
  constexpr int NW = NT / kWave;
  __shared__ double red_s[NW];
  __shared__ float red_c[NW];
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int len = min(max(a.length[s], 0), a.T);
  const size_t row = (size_t)s * a.T;
  const float* lnew = a.logp_new ? a.logp_new : a.logp_old;
  // four positions from t on; those at or past len are left out
  auto load = [&](int t, uint32_t& own, float* lo, float* ln) {
    own = 0;
    if (t >= len) return;
    if (t + 3 < a.T) {
      own = *reinterpret_cast<const u32_any*>(a.owner + row + t);
      const f32x4_any o = *reinterpret_cast<const f32x4_any*>(a.logp_old + row + t);
      const f32x4_any n = *reinterpret_cast<const f32x4_any*>(lnew + row + t);
#pragma unroll
      for (int e = 0; e < 4; ++e) { lo[e] = o[e]; ln[e] = n[e]; }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t + e < a.T) {
          own |= (uint32_t)a.owner[row + t + e] << (8 * e);
          lo[e] = a.logp_old[row + t + e];
          ln[e] = lnew[row + t + e];
        }
    }
  };
  uint32_t own;
  float lo[4] = {}, ln[4] = {};
  load(4 * tid, own, lo, ln);

  // the advantage, by every wave for itself
  const int j0 = (s / a.G) * a.G;
  float sr = 0.f, sq = 0.f;
  for (int i = lane; i < a.G; i += kWave) sr += a.rewards[j0 + i];
  const float mean = wave_sum(sr) / (float)a.G;
  for (int i = lane; i < a.G; i += kWave) {
    const float d = a.rewards[j0 + i] - mean;
    sq += d * d;
  }
  sq = wave_sum(sq);
  const float sd = a.G > 1 ? sqrtf(sq / (float)(a.G - 1)) : 0.f;
  const float A = (a.rewards[s] - mean) / (sd + 1e-6f);
  const float lo_c = 1.f - a.eps, hi_c = 1.f + a.eps;

  double acc = 0.0;
  int cnt = 0;
  for (int t = 4 * tid; t < a.T; t += 4 * NT) {
    if (t != 4 * tid) load(t, own, lo, ln);
    float sum = 0.f, g[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      g[e] = 0.f;
      if (t + e < len && ((own >> (8 * e)) & 0xFFu) != 0) {
        const float rho = expf(ln[e] - lo[e]);
        const float un = rho * A;
        const float cl = fminf(fmaxf(rho, lo_c), hi_c) * A;
        sum += fminf(un, cl);
        g[e] = un <= cl ? -un : 0.f;
        ++cnt;
      }
    }
    acc += (double)sum;
    if (!a.grad) continue;
    if (t + 3 < a.T) {
      *reinterpret_cast<f32x4_any*>(a.grad + row + t) = f32x4_any{g[0], g[1], g[2], g[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t + e < a.T) a.grad[row + t + e] = g[e];
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kWave);
  const float wc = wave_sum((float)cnt);     // counts are exact: below 2^24
  if (lane == 0) { red_s[wave] = acc; red_c[wave] = wc; }
  __syncthreads();
  if (tid == 0) {
    double sum = 0.0;
    float n = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      sum += red_s[w];
      n += red_c[w];
    }
    a.adv[s] = A;
    a.cnt[s] = (int32_t)n;
    const float hi = (float)sum;
    a.part[s] = hi;
    // an infinite sum (a ratio that overflows) leaves no remainder: inf - inf is NaN
    if (a.part_lo) a.part_lo[s] = fabsf(hi) < INFINITY ? (float)(sum - (double)hi) : 0.f;
  }
}

// The gradient divided by the masked count, kGrpoPer entries per thread; the
// first workgroup also writes the loss.
__global__ __launch_bounds__(kGrpoNT) void grpo_scale_kernel(GrpoArgs a) {
  __shared__ float red[kGrpoNT / kWave];
  const int tid = threadIdx.x;
  const size_t total = (size_t)a.S * a.T;
  const size_t i0 = (size_t)blockIdx.x * kGrpoNT * kGrpoPer + 4 * tid;
  f32x4_any g[kGrpoPer / 4];
#pragma unroll
  for (int k = 0; k < kGrpoPer / 4; ++k) {
    const size_t i = i0 + (size_t)k * 4 * kGrpoNT;
    if (a.grad && i + 3 < total) g[k] = *reinterpret_cast<const f32x4_any*>(a.grad + i);
  }
  float n = 0.f;                             // exact: the batch holds < 2^24 positions
  for (int i = tid; i < a.S; i += kGrpoNT) n += (float)a.cnt[i];
  n = block_sum<kGrpoNT>(n, red);
  const float inv_n = n > 0.f ? 1.f / n : 0.f;
  if (a.grad) {
#pragma unroll
    for (int k = 0; k < kGrpoPer / 4; ++k) {
      const size_t i = i0 + (size_t)k * 4 * kGrpoNT;
      if (i + 3 < total) {
        *reinterpret_cast<f32x4_any*>(a.grad + i) = g[k] * inv_n;
      } else {
        for (size_t j = i; j < total; ++j) a.grad[j] *= inv_n;
      }
    }
  }
  if (blockIdx.x != 0) return;
  __shared__ double dred[kGrpoNT];
  double sum = 0.0;
  for (int i = tid; i < a.S; i += kGrpoNT) sum += (double)a.part[i] + (a.part_lo ? (double)a.part_lo[i] : 0.0);
  dred[tid] = sum;
  __syncthreads();
  for (int w = kGrpoNT / 2; w > 0; w >>= 1) {
    if (tid < w) dred[tid] += dred[tid + w];
    __syncthreads();
  }
  if (tid == 0) {
    a.loss[0] = n > 0.f ? (float)(-dred[0] / (double)n) : 0.f;
    a.n_masked[0] = (int32_t)n;
  }
}

// The allocation-free entry point's workspace: one array per device, kept
// until the process ends.  Host code uses its device address from
// hipGetSymbolAddress (taken once per device), never the array's name.
static __device__ __align__(256) unsigned char scratch[kGrpoStaticBytes];

}  // namespace

hipError_t grpo_static_workspace(void** ptr) {
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_grpo(const GrpoArgs& a, hipStream_t st) {
  // a row of up to 1024 positions is one pass of 256 threads, up to 4096 of 1024
  if (a.T <= 1024)
    grpo_terms_kernel<256><<<a.S, 256, 0, st>>>(a);
  else
    grpo_terms_kernel<1024><<<a.S, 1024, 0, st>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t per = (size_t)kGrpoNT * kGrpoPer;
  const size_t blocks = a.grad ? ((size_t)a.S * a.T + per - 1) / per : 1;
  grpo_scale_kernel<<<(unsigned)blocks, kGrpoNT, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace tandem
