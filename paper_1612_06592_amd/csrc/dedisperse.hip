// Ionospheric de-dispersion (Winchen et al. 2016, Sec. 3, dispersion
// paragraph): per beam and subband the series is multiplied in the
// frequency domain by the complex weight of the trial STEC.  Overlap-save:
// each hop of 2048 new samples forms a 4096-point buffer with the previous
// 2048 samples, is transformed once, and for every trial is multiplied by
//   exp(-2 pi i [kappa T / (f_k + nu_q) + q_s D / 4096])
// and transformed back; the last 2048 outputs are kept.
//
// One 256-thread workgroup per (beam, subband, hop).  Each thread owns 16
// points; the 4096-point transform is three radix-16 Stockham passes with
// two exchanges through a padded 34 KB LDS tile.  The butterflies take the
// powers 1, 2, 4 and 8 of a pass's twiddle from the context's table: pass 1's
// through LDS, pass 2's per thread (tables of all 15 powers were measured
// slower: this kernel is close to bound by LDS instructions as well as VALU).
// Those powers are squares of each other in FP32, and their rounding is most
// of the outputs' error (5.7e-7 relative): rounded from the exact values they
// would give 2.6e-7, but every output would move by 6e-7, and a series' SNR by
// up to 9e-7, from what this transform has returned since its powers were
// formed as products in the kernel.
// The forward spectrum stays in registers across all trials.  A trial's chirp
// phase is formed per bin from FP64-reduced constants and taken through the
// hardware sine and cosine; on a uniform grid only the first trial's is, and
// trial t + 1's chirp is trial t's times a per-bin factor read from a table
// formed in FP64 (a table of every trial's factors, one complex load per bin
// and trial instead of the phase, made the single-trial workloads slower: C3
// 2.70 -> 2.79 ms).
#include <cmath>

#include "fft_dev.h"
#include "lp_internal.h"

namespace lp {

constexpr int kDdThreads = 256;
constexpr int kDdLds = 4096 + 128;  // slot of element 4095 is 4222

// Pass-1 twiddles of one workgroup (w = exp(-2 pi i / 4096)): w^(16 a) and
// its powers 2, 4, 8 for a < 16.
struct DdTw {
  Tw16 p1[16];
};

// 4096-point transform of v[r] = in[j + 256 r] (j = thread); on return
// v[r] = out[j + 256 r] (HI: only r >= 8).  Unnormalised; INV selects
// exp(+2 pi i ...).
// pass2_twiddle(j) gives w^j and its powers.  START: pass 0's first stage
// (the pairs v[n], v[n + 8]) is done.
template <bool INV, bool HI, bool START, typename Pass2>
__device__ __forceinline__ void fft4096(float2 *v, float2 *lds,
                                        const DdTw &tw, Pass2 pass2_twiddle,
                                        int j) {
  // Element e sits at slot e + e / 32 (one pad slot per 32: every access
  // pattern below puts the 64 lanes' 8-byte words evenly on the banks, for
  // 32 or 64 banks).  In closed form (j < 256, r < 16):
  //   16 j + r -> 16 j + j / 2 + r,  j + 256 r -> j + j / 32 + 264 r,
  //   (j / 16) 256 + j mod 16 + 16 r -> (j / 16) 264 + j mod 16 + 16 r + r / 2.
  const int sj = j + (j >> 5);
  // Pass 0 (Ns = 1): no twiddle; write to (16 j + r) once every thread has
  // read the previous transform's last exchange.
  if (START)
    dft16_tail<INV, 16>(v);
  else
    dft16_fma<INV>(v);
  __syncthreads();
  {
    const int b0 = 16 * j + (j >> 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) lds[b0 + r] = v[r];
  }
  __syncthreads();
  // Pass 1 (Ns = 16): twiddle w^(16 (j mod 16) r).
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = lds[sj + 264 * r];
  dft16_twiddled<INV>(v, tw.p1[j & 15].conj_if<INV>());
  const Tw16 w2p = pass2_twiddle(j);
  __syncthreads();
  {
    const int b2 = (j >> 4) * 264 + (j & 15);
#pragma unroll
    for (int r = 0; r < 16; ++r) lds[b2 + 16 * r + (r >> 1)] = v[r];
  }
  __syncthreads();
  // Pass 2 (Ns = 256): twiddle w^(j r); output index j + 256 r stays in
  // registers.
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = lds[sj + 264 * r];
  dft16_twiddled<INV, HI>(v, w2p.conj_if<INV>());
}

// Chirp factor exp(-2 pi i c) for a phase c in cycles, |c| <= 1/2 after the
// reduction; the hardware sine and cosine take revolutions.
__device__ __forceinline__ float2 chirp(float c) {
  c -= rintf(c);
  return make_float2(__builtin_amdgcn_cosf(c), -__builtin_amdgcn_sinf(c));
}

// base + e folded into [-1/2, 1/2] with one rounding: e (a multiple of 1/4)
// less a whole number is exact.  Near zero a phase keeps more bits.
__device__ __forceinline__ float fold_phase(float base, float e) {
  return base + (e - rintf(base + e));
}

// Eight outputs of a thread, 256 samples apart.  Where all outputs exceed the
// cache they are written past it, else left there for their reader: one beam x
// 244 subbands x 16 hops at 4 trials, 256 MB, up to the synthesis, 455 us
// against 461 us past it; 2 beams at 16 trials, 2 GB, 2610 against 2600 us.
__device__ __forceinline__ void store_half(float2 *out, const float2 *v,
                                           bool stream) {
  if (stream) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float o[2] = {v[r].x, v[r].y};
      nt_store<2>(out + 256 * r, o);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 8; ++r) out[256 * r] = v[r];
  }
}

// REC: the trials are uniformly spaced, so the first trial's chirp comes
// from its phase and each next one is the previous one times
// rstep[s][q] (float2 [S][N_fft]).
template <bool REC>
__global__ __launch_bounds__(kDdThreads)
__attribute__((amdgpu_waves_per_eu(4, 8))) void dd_kernel(
    const float2 *__restrict__ y, float2 *__restrict__ tail, int update_tail,
    float2 *__restrict__ d, const float2 *__restrict__ tw,
    const float *__restrict__ base, const float *__restrict__ afac,
    const float2 *__restrict__ rstep, const float *__restrict__ gq, int n_sb,
    int n_tec, long n_t, int n_hop, long n_blocks, int stream) {
  __shared__ float2 lds[kDdLds];
  __shared__ DdTw tws;
  const Tw16 *twp = reinterpret_cast<const Tw16 *>(tw + kTwPowers);
  if (threadIdx.x < 16) tws.p1[threadIdx.x] = twp[16 * threadIdx.x];
  // The pass-2 twiddle w^j: kept in registers, except beside the trial
  // steps' 32 (REC), where each pass reads it again (8 KB, from the caches)
  // ahead of the exchange.
  const Tw16 w2p = twp[threadIdx.x];
  const __amdgpu_buffer_rsrc_t twrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float2 *>(tw), 0, kTwEntries * 8, kRawBufferWord3);
  auto pass2_twiddle = [&](int jo) {
    if constexpr (!REC) return w2p;
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const u4 a = __builtin_amdgcn_raw_buffer_load_b128(twrs, 32 * jo,
                                                       8 * kTwPowers, 0),
             b = __builtin_amdgcn_raw_buffer_load_b128(twrs, 32 * jo,
                                                       8 * kTwPowers + 16, 0);
    auto f2 = [](unsigned x, unsigned y) {
      return make_float2(__uint_as_float(x), __uint_as_float(y));
    };
    return Tw16{f2(a.x, a.y), f2(a.z, a.w), f2(b.x, b.y), f2(b.z, b.w)};
  };
  // (the barrier inside the first transform orders these before use)
  const long bid = xcd_remap(blockIdx.x, n_blocks);
  const int h = (int)(bid % n_hop);
  const long bs = bid / n_hop;          // beam * n_sb + subband
  const int s = (int)(bs % n_sb);
  const int b = (int)(bs / n_sb);
  const int j = threadIdx.x;
  const float2 *ys = y + bs * n_t;
  float2 *tl = tail + bs * kHist;
  const long hs = (long)h * kHop;

  float2 v[16];
#pragma unroll
  for (int r = 0; r < 8; ++r)
    v[r] = (h == 0) ? tl[j + 256 * r] : ys[hs - kHist + j + 256 * r];
#pragma unroll
  for (int r = 8; r < 16; ++r) v[r] = ys[hs + j + 256 * (r - 8)];

  fft4096<false, false, false>(v, lds, tws, pass2_twiddle, j);

  // Hop 0 read the old tail above (and every thread has passed the
  // barriers inside the transform), so it can now store the new one.
  if (update_tail && h == 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) tl[j + 256 * r] = ys[n_t - kHist + j + 256 * r];
  }

  // The inverse transform's 1 / 4096 applied to the spectrum (a power of
  // two: exact, so every later rounding is the same as scaling the output).
  float2 U[16];
#pragma unroll
  for (int r = 0; r < 16; ++r)
    U[r] = make_float2(v[r].x * (1.0f / 4096.0f), v[r].y * (1.0f / 4096.0f));
  // Chirp phase of bin q (signed q_s) for trial t, in cycles:
  //   frac(kappa T / (f_k + nu_q)) + q_s D / 4096
  //     = frac(A) - A g_q + (q_s mod 4) / 4   (mod 1),
  // with A = kappa T / f_k, g_q = x / (1 + x), x = nu_q / f_k from the plan
  // table, and q_s mod 4 = j mod 4 for every bin of thread j.  The residual
  // A g_q is below ~0.4 cycles.
  const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(gq), 0, n_sb * kNfft * 4, kRawBufferWord3);
  const float e = 0.25f * (float)(j & 3);
  float2 *outb = d + ((long)b * n_tec * n_sb + s) * n_t + hs + j;
  const long trial_stride = (long)n_sb * n_t;
  if (REC) {
    // U becomes the first trial's chirped spectrum; R the per-trial factor.
    const float bse = fold_phase(base[s], e), A = afac[s];
    const float2 *rs = rstep + s * kNfft + j;
    float2 R[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float g = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
          grs, 4 * (s * kNfft + j), 1024 * r, 0));
      U[r] = cmul(U[r], chirp(fmaf(-A, g, bse)));
      R[r] = rs[256 * r];
    }
    for (int jt = 0; jt < n_tec; ++jt) {
      const int jo = opaque(j);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        v[r] = U[r];
        U[r] = cmul(U[r], R[r]);
      }
      fft4096<true, true, false>(v, lds, tws, pass2_twiddle, jo);
      store_half(outb + jt * trial_stride, v + 8, stream);
    }
  } else {
    for (int jt = 0; jt < n_tec; ++jt) {
      const int jo = opaque(j);
      const float bse = fold_phase(base[jt * n_sb + s], e),
                  A = afac[jt * n_sb + s];
      const int goff = 4 * (s * kNfft + jo);
      // The chirped spectrum and the inverse's first stage together: the
      // chirp factor of bin n + 8 is the twiddle of that butterfly.
      auto factor = [&](int r) {
        const float g = __uint_as_float(
            __builtin_amdgcn_raw_buffer_load_b32(grs, goff, 1024 * r, 0));
        return chirp(fmaf(-A, g, bse));
      };
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        v[n] = cmul(U[n], factor(n));
        v[n + 8] = U[n + 8];
        bf2(v[n], v[n + 8], factor(n + 8));
      }
      fft4096<true, true, true>(v, lds, tws, pass2_twiddle, jo);
      store_half(outb + jt * trial_stride, v + 8, stream);
    }
  }
}

// The same with one trial: a workgroup walks a run of hops of one series.
// The next hop's samples are read while this one is transformed, and the half
// that it shares with this one is kept instead of read again (61 beams x 244
// subbands x 16 hops: 2476 -> 2365 us, 3.3 TB/s).  What bounds both kernels is
// the latency between the barriers, four waves per SIMD issuing an instruction
// per 4 cycles where 2.1 would do; tried and slower: one wave per hop with 64
// points per lane and one exchange without barriers (two waves per SIMD, 2972
// us), and an unpadded tile for five workgroups per CU (spills at 96
// registers).
__global__ __launch_bounds__(kDdThreads)
__attribute__((amdgpu_waves_per_eu(4, 8))) void dd_single_kernel(
    const float2 *__restrict__ y, float2 *__restrict__ tail, int update_tail,
    float2 *__restrict__ d, const float2 *__restrict__ tw,
    const float *__restrict__ base, const float *__restrict__ afac,
    const float *__restrict__ gq, int n_sb, long n_t, int n_hop, int per_wg,
    int runs, long n_blocks) {
  __shared__ float2 lds[kDdLds];
  __shared__ DdTw tws;
  const int j = threadIdx.x;
  const long bid = xcd_remap(blockIdx.x, n_blocks);
  const int h0 = (int)(bid % runs) * per_wg;
  const int h1 = min(h0 + per_wg, n_hop);
  const long bs = bid / runs;  // beam * n_sb + subband
  const int s = (int)(bs % n_sb);
  const float2 *ys = y + bs * n_t + j;
  float2 *tl = tail + bs * kHist + j;
  float2 *out = d + bs * n_t + j;

  // Samples and outputs pass the cache by: each is 256 MB or more here (19
  // beams x 488 subbands x 4 hops: 411 -> 389 us; 32 x 128 x 4, 256 MB, 196 ->
  // 186, with the synthesis that reads them 617 -> 609).
  float2 last[8], next[8];
  auto read = [&](int h) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float o[2];
      nt_load<2>(ys + (long)h * kHop + 256 * r, o);
      next[r] = make_float2(o[0], o[1]);
    }
  };
#pragma unroll
  for (int r = 0; r < 8; ++r)
    last[r] = h0 == 0 ? tl[256 * r] : ys[(long)(h0 - 1) * kHop + 256 * r];
  read(h0);
  const Tw16 *twp = reinterpret_cast<const Tw16 *>(tw + kTwPowers);
  if (j < 16) tws.p1[j] = twp[16 * j];
  // (the barrier inside the first transform orders these before use)
  const Tw16 w2p = twp[j];
  auto pass2_twiddle = [&](int) { return w2p; };
  const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(gq), 0, n_sb * kNfft * 4, kRawBufferWord3);
  const float bse = fold_phase(base[s], 0.25f * (float)(j & 3)), A = afac[s];
  // This thread read its part of the old tail above: the new one can go there.
  if (update_tail && h0 == 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) tl[256 * r] = ys[n_t - kHist + 256 * r];
  }
  for (int h = h0; h < h1; ++h) {
    const int jo = opaque(j);
    float2 v[16];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      v[r] = last[r];
      v[8 + r] = last[r] = next[r];
    }
    if (h + 1 < h1) read(h + 1);
    fft4096<false, false, false>(v, lds, tws, pass2_twiddle, jo);
    const int goff = 4 * (s * kNfft + jo);
    auto factor = [&](int r) {
      const float g = __uint_as_float(
          __builtin_amdgcn_raw_buffer_load_b32(grs, goff, 1024 * r, 0));
      return chirp(fmaf(-A, g, bse));
    };
    auto scaled = [&](int r) {
      return make_float2(v[r].x * (1.0f / 4096.0f), v[r].y * (1.0f / 4096.0f));
    };
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      v[n] = cmul(scaled(n), factor(n));
      v[n + 8] = scaled(n + 8);
      bf2(v[n], v[n + 8], factor(n + 8));
    }
    fft4096<true, true, true>(v, lds, tws, pass2_twiddle, jo);
    store_half(out + (long)h * kHop, v + 8, true);
  }
}

}  // namespace lp

using namespace lp;

extern "C" lp_status lp_dedisperse(lp_ctx *ctx, const lp_band *band,
                                   const double *tec_tecu, int32_t n_tec,
                                   const void *y, int32_t n_beams,
                                   int64_t n_t, void *tail, int32_t flags,
                                   void *d, void *hip_stream) {
  if (!ctx || !tec_tecu || !y || !tail || !d)
    return set_error(LP_EINVAL, "lp_dedisperse: NULL argument");
  lp_status rc = check_band(band);
  if (rc) return rc;
  if (n_tec <= 0 || n_tec > 4096)
    return set_error(LP_EINVAL, "lp_dedisperse: n_tec %d", n_tec);
  for (int j = 0; j < n_tec; ++j)
    if (!(tec_tecu[j] >= 0.0 && tec_tecu[j] <= 1000.0))
      return set_error(LP_EINVAL, "lp_dedisperse: TEC %g outside [0, 1000]",
                       tec_tecu[j]);
  if (n_beams <= 0)
    return set_error(LP_EINVAL, "lp_dedisperse: n_beams %d", n_beams);
  if (n_t <= 0 || n_t % kHop != 0)
    return set_error(LP_EINVAL,
                     "lp_dedisperse: n_t %lld not a positive multiple of %d",
                     (long long)n_t, kHop);
  if (flags & ~LP_DD_KEEP_TAIL)
    return set_error(LP_EINVAL, "lp_dedisperse: unknown flags 0x%x", flags);
  if ((rc = set_device(ctx))) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  PlanRef<DdPlan> p;
  if ((rc = get_dd_plan(ctx, band, tec_tecu, n_tec, st, p))) return rc;
  return dd_launch(ctx, p.get(), band->n_sb, y, n_beams, n_t, tail,
                   !(flags & LP_DD_KEEP_TAIL), d, 0, n_tec, st);
}

namespace lp {
lp_status dd_launch(lp_ctx *ctx, DdPlan *p, int n_sb, const void *y,
                    int n_beams, long n_t, void *tail, bool update_tail,
                    void *d, int j0, int nj, hipStream_t st) {
  lp_status rc;
  if ((rc = plan_wait(p, st))) return rc;
  const int n_hop = (int)(n_t / kHop);
  const long nb = (long)n_beams * n_sb * n_hop;
  if (nb > 0x7fffffffL)
    return set_error(LP_EINVAL, "lp_dedisperse: grid too large");
  if (j0 < 0 || nj <= 0 || j0 + nj > p->n_tec)
    return set_error(LP_EINVAL, "de-dispersion: trials %d..%d of %d", j0,
                     j0 + nj - 1, p->n_tec);
  const size_t jo = (size_t)j0 * n_sb;
  // One trial and many hops: runs of hops, each workgroup's long enough that
  // the samples read ahead pay for the start, with sixteen workgroups per CU
  // so that the last ones cost little.  Shorter runs lose: 244 series of 32
  // hops took 81 us in runs of 2 against 77 us hop by hop.
  // Results below 256 MB, which a device of fewer than 256 CUs would reach
  // here, stay hop by hop, and with that in the cache for their reader.
  const int per_wg = (int)std::min<long>(n_hop, nb / (16L * ctx->n_cu));
  const size_t bytes = (size_t)nb * nj * kHop * sizeof(float2);
  if (nj == 1 && per_wg >= 4 && bytes >= kMallBytes) {
    const int runs = (n_hop + per_wg - 1) / per_wg;
    const long n_wg = (long)n_beams * n_sb * runs;
    hipLaunchKernelGGL(dd_single_kernel, dim3((unsigned)n_wg),
                       dim3(kDdThreads), 0, st, static_cast<const float2 *>(y),
                       static_cast<float2 *>(tail), update_tail ? 1 : 0,
                       static_cast<float2 *>(d), ctx->tw4096.as<const float2>(),
                       p->base.as<const float>() + jo,
                       p->afac.as<const float>() + jo, p->gq.as<const float>(),
                       n_sb, n_t, n_hop, per_wg, runs, n_wg);
    LP_HIP(hipGetLastError());
    return LP_OK;
  }
  auto kern = p->uniform && nj >= 2 ? dd_kernel<true> : dd_kernel<false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(kDdThreads), 0, st,
                     static_cast<const float2 *>(y), static_cast<float2 *>(tail),
                     update_tail ? 1 : 0, static_cast<float2 *>(d),
                     ctx->tw4096.as<const float2>(),
                     p->base.as<const float>() + jo,
                     p->afac.as<const float>() + jo,
                     p->rstep.as<const float2>(),
                     p->gq.as<const float>(), n_sb, nj, n_t, n_hop, nb,
                     bytes > kMallBytes);
  LP_HIP(hipGetLastError());
  return LP_OK;
}
}  // namespace lp
