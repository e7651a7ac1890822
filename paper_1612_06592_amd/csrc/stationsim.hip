// Station simulator, ADC stage (Winchen et al. 2016, Sec. 2: each station
// samples its antennas at 5 ns; Sec. 5: the simulation chain).  Every input
// (station x polarisation) gets, at absolute sample n,
//   noise = sum_{r < R} (popcount(w_r) - 16)
// with w_r the 32-bit words of Philox4x32-10 (Salmon, Moraes, Dror & Shaw,
// SC 2011) under key (seed lo, seed hi) and counter (n lo, n hi, input,
// group of four words): Binomial(32 R, 1/2) centred, variance 8 R, in
// integer arithmetic, so the codes are reproducible bit for bit anywhere.
// An optional float pulse waveform per input is rounded half to even and
// added; the sum saturates to the ADC's signed range.  The station
// filterbank that turns these codes into subbands is lp_station_ppf.
#include <cmath>

#include "lp_internal.h"

namespace lp {

constexpr int kSimPer = 4;  // samples per thread (a workgroup covers 1024)

constexpr unsigned kPhM0 = 0xD2511F53u, kPhM1 = 0xCD9E8D57u;  // multipliers
constexpr unsigned kPhW0 = 0x9E3779B9u, kPhW1 = 0xBB67AE85u;  // key increments

__device__ __forceinline__ unsigned xor3(unsigned a, unsigned b, unsigned c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
// One 32 x 32 -> 64-bit product gives both halves.
__device__ __forceinline__ void mul_hl(unsigned m, unsigned v, unsigned &hi,
                                       unsigned &lo) {
  const unsigned long long p = (unsigned long long)m * v;
  hi = (unsigned)(p >> 32);
  lo = (unsigned)p;
}

// Philox4x32 with 10 rounds multiplies, in each round, words 0 and 2 by the
// two round multipliers, mixes the high halves with words 1 and 3 and the
// key, and advances the key.  The groups of one sample differ in counter
// word 3 alone, which enters round 1 by a xor and reaches every word only in
// round 3: of the first three rounds' six products, four are the sample's.
struct PhiloxSample {
  unsigned h0;          // round 1: high half of M0 c0
  unsigned c1y;         // round 1, word 1 (the input's alone)
  unsigned c2w;         // round 2, word 3
  unsigned h3, c3y;     // round 3: high half of M1 c2, word 1
  __device__ __forceinline__ PhiloxSample(unsigned lo, unsigned hi,
                                          unsigned inp, unsigned k0,
                                          unsigned k1) {
    unsigned l0, h1, h2, c2z;
    mul_hl(kPhM0, lo, h0, l0);
    mul_hl(kPhM1, inp, h1, c1y);
    mul_hl(kPhM0, xor3(h1, hi, k0), h2, c2w);
    c2z = xor3(h2, l0, k1 + kPhW1);
    mul_hl(kPhM1, c2z, h3, c3y);
  }
};

// The four words of group g.
__device__ __forceinline__ void philox_words(const PhiloxSample &s, unsigned g,
                                             unsigned k0, unsigned k1,
                                             unsigned *w) {
  unsigned h, c2y, x, y = s.c3y, z, v;
  mul_hl(kPhM1, xor3(s.h0, g, k1), h, c2y);
  mul_hl(kPhM0, xor3(h, s.c1y, k0 + kPhW0), h, v);
  x = xor3(s.h3, c2y, k0 + 2 * kPhW0);
  z = xor3(h, s.c2w, k1 + 2 * kPhW1);
#pragma unroll
  for (int r = 3; r < 10; ++r) {
    unsigned h0, l0, h1, l1;
    mul_hl(kPhM0, x, h0, l0);
    mul_hl(kPhM1, z, h1, l1);
    x = xor3(h1, y, k0 + r * kPhW0);
    z = xor3(h0, v, k1 + r * kPhW1);
    y = l1;
    v = l0;
  }
  w[0] = x;
  w[1] = y;
  w[2] = z;
  w[3] = v;
}

// What bounds it is integer issue: every instruction here takes a quad-cycle,
// so the mixes are three-input xors and a sample's products are shared by its
// groups (16 words per sample, 402 M samples: 2495 -> 1737 us).
__global__ __launch_bounds__(256) void sim_adc_kernel(
    unsigned k0, unsigned k1, int R, int lim, long n0, long n_samp,
    const float *__restrict__ pulse, long pulse_n0, long pulse_len,
    short *__restrict__ adc) {
  const unsigned inp = blockIdx.y;
  long t = (long)blockIdx.x * (256 * kSimPer) + threadIdx.x;
  for (int i = 0; i < kSimPer && t < n_samp; ++i, t += 256) {
    const unsigned long long n = (unsigned long long)(n0 + t);
    const PhiloxSample s((unsigned)n, (unsigned)(n >> 32), inp, k0, k1);
    int acc = -16 * R;
    int g = 0;
    for (; 4 * g + 16 <= R; g += 4) {  // four groups side by side
      unsigned w[16];
#pragma unroll
      for (int j = 0; j < 4; ++j) philox_words(s, g + j, k0, k1, w + 4 * j);
#pragma unroll
      for (int j = 0; j < 16; ++j) acc += __popc(w[j]);
    }
    for (; 4 * g < R; ++g) {
      unsigned w[4];
      philox_words(s, g, k0, k1, w);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * g + j < R) acc += __popc(w[j]);
    }
    const long pi = n0 + t - pulse_n0;
    if (pulse && pi >= 0 && pi < pulse_len) {
      // |pulse| is bounded before the conversion (beyond any ADC range).
      const float v =
          fminf(fmaxf(pulse[(long)inp * pulse_len + pi], -1e6f), 1e6f);
      acc += (int)rintf(v);
    }
    acc = min(max(acc, -lim), lim - 1);
    adc[(long)inp * n_samp + t] = (short)acc;
  }
}

}  // namespace lp

using namespace lp;

extern "C" lp_status lp_sim_adc(lp_ctx *ctx, const lp_sim_cfg *cfg, int64_t n0,
                                int64_t n_samp, const float *pulse,
                                int64_t pulse_n0, int64_t pulse_len,
                                int16_t *adc, void *hip_stream) {
  if (!ctx || !cfg || !adc)
    return set_error(LP_EINVAL, "lp_sim_adc: NULL argument");
  if (cfg->n_in < 1 || cfg->n_in > 65535)
    return set_error(LP_EINVAL, "lp_sim_adc: n_in %d", cfg->n_in);
  if (cfg->noise_words < 0 || cfg->noise_words > 256)
    return set_error(LP_EINVAL, "lp_sim_adc: noise_words %d not in 0..256",
                     cfg->noise_words);
  if (cfg->adc_bits < 2 || cfg->adc_bits > 16)
    return set_error(LP_EINVAL, "lp_sim_adc: adc_bits %d not in 2..16",
                     cfg->adc_bits);
  if (n0 < 0 || n_samp <= 0)
    return set_error(LP_EINVAL, "lp_sim_adc: bad sample range");
  if (pulse && pulse_len <= 0)
    return set_error(LP_EINVAL, "lp_sim_adc: pulse_len must be positive");
  if ((n_samp + 255) / 256 > 0x7fffffffL)
    return set_error(LP_EINVAL, "lp_sim_adc: n_samp too large");
  lp_status rc = set_device(ctx);
  if (rc) return rc;
  const unsigned k0 = (unsigned)(cfg->seed & 0xffffffffu);
  const unsigned k1 = (unsigned)(cfg->seed >> 32);
  constexpr long per = 256 * kSimPer;
  dim3 grid((unsigned)((n_samp + per - 1) / per), cfg->n_in);
  hipLaunchKernelGGL(sim_adc_kernel, grid, dim3(256), 0,
                     static_cast<hipStream_t>(hip_stream), k0, k1,
                     cfg->noise_words, 1 << (cfg->adc_bits - 1), (long)n0,
                     (long)n_samp, pulse, (long)pulse_n0,
                     pulse ? (long)pulse_len : 0L,
                     reinterpret_cast<short *>(adc));
  LP_HIP(hipGetLastError());
  return LP_OK;
}
