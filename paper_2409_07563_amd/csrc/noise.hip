// Step (a1): fill eps[T][m][ldk] with sigma_j * N(0, 1) draws.
//
// One thread per (sample k, Philox call c): a call yields the four normals
// n = 4c .. 4c+3 of sample k (n = t*m + j).  Lanes of a wave hold consecutive
// samples, so each of the four stores of a wave is one contiguous 256-byte
// row segment of the [T*m][ldk] layout (k fastest).  The kernel is VALU-bound
// (Philox + two Box-Muller pairs, ~35 VALU operations per normal) rather than
// bound by its HBM writes.
//
// Large draws take four samples per thread: with one, a wave lives for one
// call, about 150 operations, behind a chain of scalar loads (arguments,
// iteration word, deviations); four samples pay that once, and their rows are
// stored 16 bytes a lane.  One and four samples per thread: K 65536, T 200,
// m 4 66 and 46 us (the stores alone take 31, the arithmetic alone 40);
// K 32768, T 200, m 2 20 and 16 us.
#include "common.h"
#include "noise.h"

namespace mppi {

// FOUR: four samples per thread; calls: Philox calls per thread and sample.
// A workgroup covers one group of 256 samples (grouped so that their rollout
// finds them in its L2): one thread per sample, or (FOUR) 64 lanes of four
// samples per wave, the waves taking different calls.  WIDE: 1024 samples of
// the same calls.
template <bool FOUR, bool WIDE>
__global__ __launch_bounds__(256) void noise_kernel(uint32_t key0, uint32_t key1,
                                                    const uint32_t* __restrict__ d_iteration,
                                                    uint32_t iteration, uint32_t instance,
                                                    int K, int TM, int m, Sigma8 sigma,
                                                    float* __restrict__ eps, int64_t ldk,
                                                    int calls, const float* __restrict__ sigma_t,
                                                    int mean_sample, uint32_t* d_word_out) {
  const int slice = blockIdx.y;
  const int t = threadIdx.x;
  const int k = WIDE ? (blockIdx.x * 256 + t) * 4
                     : blockIdx.x * kGroupSamples + (FOUR ? t % kWave * 4 : t);
  if (k >= K) return;
  const uint32_t it = d_iteration ? *d_iteration + iteration : iteration;
  if (d_word_out && blockIdx.x == 0 && slice == 0 && t == 0) *d_word_out = it;
  const int ncall = (TM + 3) / 4;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int c0 = (FOUR && !WIDE ? slice * 4 + wave : slice) * calls;
  const bool zero = mean_sample && k == 0;
  for (int c = c0; c < c0 + calls && c < ncall; ++c) {
    if constexpr (FOUR)
      noise::emit_call4(key0, key1, it, instance, k, K, c, TM, m, sigma.v, eps, ldk, sigma_t,
                        zero);
    else
      noise::emit_call(key0, key1, it, instance, k, c, TM, m, sigma.v, eps, ldk, sigma_t, zero);
  }
}
static_assert(kGroupSamples == 256 && kGroupSamples == 4 * kWave, "one group per workgroup");

// Four samples per thread from this many Philox calls in all (four waves per
// SIMD then, on 256 CUs: 9.6 us with one sample per thread, 8.3 with four;
// below, too few waves are left to cover the loads), where the rows can be
// stored 16 bytes a lane.
constexpr int64_t kFourMinCalls = int64_t{1} << 20;
// 1024 samples per workgroup from this many bytes of noise, of which the L2s
// (32 MB) can keep little: whole rows are then written one after the other,
// which the update's pass over the rows gains more from.  Sampling and rollout |
// one iteration, us, quadrotor, 256 and 1024 samples per workgroup: K 32768
// T 64 57 and 65 | 61 and 61; K 65536 T 64 65 and 71 | 74 and 75; K 65536 T 100
// 93 and 99 | 117 and 115; K 65536 T 200 179 and 183 | 216 and 212.
constexpr int64_t kWideMinBytes = int64_t{80} << 20;

hipError_t launch_noise(uint64_t seed, const uint32_t* d_iteration, uint32_t iteration,
                        uint32_t instance, int K, int T, int m, const float* sigma,
                        float* d_eps, int64_t ldk, hipStream_t stream, int calls,
                        const float* d_sigma_t, bool mean_sample, uint32_t* d_word_out) {
  if (calls < 1) return hipErrorInvalidValue;
  const int TM = T * m;
  const int ncall = (TM + 3) / 4;
  Sigma8 s{};
  for (int j = 0; j < m; ++j) s.v[j] = sigma[j];
  const bool four = static_cast<int64_t>(K) * ncall >= kFourMinCalls && ldk % 4 == 0 &&
                    reinterpret_cast<uintptr_t>(d_eps) % sizeof(float4) == 0;
  const bool wide = four && int64_t{4} * ldk * TM >= kWideMinBytes;
  const int per = four && !wide ? 4 * calls : calls;  // calls per workgroup
  const int ny = (ncall + per - 1) / per;
  const auto kernel = wide ? noise_kernel<true, true>
                           : four ? noise_kernel<true, false> : noise_kernel<false, false>;
  const int nx = wide ? static_cast<int>((int64_t{K} + 1023) / 1024) : sample_groups(K);
  hipLaunchKernelGGL(kernel, dim3(nx, ny), dim3(256), 0, stream, static_cast<uint32_t>(seed),
                     static_cast<uint32_t>(seed >> 32), d_iteration, iteration, instance, K, TM, m,
                     s, d_eps, ldk, calls, d_sigma_t, mean_sample ? 1 : 0, d_word_out);
  return hipGetLastError();
}

// Every possible Box-Muller factor: r[j1-1] for j1 in [1, 2^24], (c, s)[j2]
// for j2 in [0, 2^24).
__global__ __launch_bounds__(256) void noise_tables_kernel(float* __restrict__ r,
                                                           float* __restrict__ c,
                                                           float* __restrict__ s) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= (1u << 24)) return;
  r[j] = noise::radius(j + 1u);
  float cc, ss;
  noise::angle(j, cc, ss);
  c[j] = cc;
  s[j] = ss;
}

hipError_t launch_noise_tables(float* d_r, float* d_c, float* d_s, hipStream_t stream) {
  hipLaunchKernelGGL(noise_tables_kernel, dim3((1u << 24) / 256), dim3(256), 0, stream, d_r,
                     d_c, d_s);
  return hipGetLastError();
}

}  // namespace mppi
