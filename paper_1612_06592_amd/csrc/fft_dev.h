// Register-level DFT butterflies and Stockham passes shared by the
// de-dispersion (4096-point) and synthesis (1024-point) kernels.
//
// A Stockham pass of radix R over an N-point transform, with Ns the size
// of the sub-transforms already formed, lets butterfly j (0 <= j < N/R)
// read in[j + r N/R], twiddle element r by exp(s 2 pi i (j mod Ns) r /
// (Ns R)), do an R-point DFT and write out[(j / Ns) Ns R + (j mod Ns) +
// r Ns]; Ns = 1, R1, R1 R2, ... yields the natural-order DFT.
#pragma once

#include <hip/hip_runtime.h>

namespace lp {

__device__ __forceinline__ float2 cadd(float2 a, float2 b) {
  return make_float2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ float2 csub(float2 a, float2 b) {
  return make_float2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// 4-point DFT in place; INV selects the +i kernel.
template <bool INV>
__device__ __forceinline__ void dft4(float2 &a, float2 &b, float2 &c,
                                     float2 &d) {
  float2 t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), t3 = csub(b, d);
  a = cadd(t0, t2);
  c = csub(t0, t2);
  if (!INV) {  // X1 = t1 - i t3, X3 = t1 + i t3
    b = make_float2(t1.x + t3.y, t1.y - t3.x);
    d = make_float2(t1.x - t3.y, t1.y + t3.x);
  } else {
    b = make_float2(t1.x - t3.y, t1.y + t3.x);
    d = make_float2(t1.x + t3.y, t1.y - t3.x);
  }
}

// exp(-2 pi i m / 16) for m = 0..15 (cos, -sin).
__device__ __forceinline__ float2 w16(int m) {
  constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508977f,
                  c2 = 0.70710678118654752f;
  switch (m & 15) {
    case 0: return make_float2(1.f, 0.f);
    case 1: return make_float2(c1, -s1);
    case 2: return make_float2(c2, -c2);
    case 3: return make_float2(s1, -c1);
    case 4: return make_float2(0.f, -1.f);
    case 5: return make_float2(-s1, -c1);
    case 6: return make_float2(-c2, -c2);
    case 7: return make_float2(-c1, -s1);
    case 8: return make_float2(-1.f, 0.f);
    case 9: return make_float2(-c1, s1);
    case 10: return make_float2(-c2, c2);
    case 11: return make_float2(-s1, c1);
    case 12: return make_float2(0.f, 1.f);
    case 13: return make_float2(s1, c1);
    case 14: return make_float2(c2, c2);
    default: return make_float2(c1, s1);
  }
}

// v * W16^m (INV: times its conjugate).  W16^4 = -i is a swap and a sign
// change (a general complex product by (0, -1) keeps two products by zero,
// which IEEE arithmetic does not let the compiler drop).
template <bool INV>
__device__ __forceinline__ float2 tw16(float2 v, int m) {
  if (m == 4)
    return INV ? make_float2(-v.y, v.x) : make_float2(v.y, -v.x);
  const float2 w = w16(m);
  return INV ? cmulc(v, w) : cmul(v, w);
}

// 16-point DFT in place, natural order in and out (4 x 4 decomposition:
// n = 4 n1 + n2, k = k1 + 4 k2).
template <bool INV>
__device__ __forceinline__ void dft16(float2 *v) {
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2)
    dft4<INV>(v[n2], v[4 + n2], v[8 + n2], v[12 + n2]);
  // v[n2 + 4 k1] now holds A[n2][k1]; apply W16^(n2 k1).
#pragma unroll
  for (int n2 = 1; n2 < 4; ++n2) {
#pragma unroll
    for (int k1 = 1; k1 < 4; ++k1)
      v[n2 + 4 * k1] = tw16<INV>(v[n2 + 4 * k1], n2 * k1);
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
    dft4<INV>(v[4 * k1 + 0], v[4 * k1 + 1], v[4 * k1 + 2], v[4 * k1 + 3]);
  // v[4 k1 + k2] holds X[k1 + 4 k2]: transpose the 4 x 4 index.
  float2 t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = v[i];
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = t[4 * k1 + k2];
}

// Radix-2 butterflies in fused multiply-adds: (a, b) <- (a + w b, a - w b).
// The sum takes two FMAs per component and the difference is 2 a minus the
// sum, one more: 6 instructions with the twiddle's product in them, where a
// complex product and two sums take 8.  A DFT built of these (decimation in
// time) needs no products by its external twiddles: input r is to be
// multiplied by w^r, and w^8, w^4, w^2 and w go into the four stages.
__device__ __forceinline__ void bf2(float2 &a, float2 &b, float2 w) {
  const float x = fmaf(w.x, b.x, fmaf(-w.y, b.y, a.x));
  const float y = fmaf(w.x, b.y, fmaf(w.y, b.x, a.y));
  b = make_float2(fmaf(2.f, a.x, -x), fmaf(2.f, a.y, -y));
  a = make_float2(x, y);
}
// a - w b alone (b takes it).
__device__ __forceinline__ void bf2_diff(float2 a, float2 &b, float2 w) {
  b = make_float2(fmaf(-w.x, b.x, fmaf(w.y, b.y, a.x)),
                  fmaf(-w.x, b.y, fmaf(-w.y, b.x, a.y)));
}
// -i w (INV: +i w): the quarter-turn of a stage's twiddles.
template <bool INV>
__device__ __forceinline__ float2 quarter(float2 w) {
  return INV ? make_float2(-w.y, w.x) : make_float2(w.y, -w.x);
}
// W8 w (INV: times its conjugate).
template <bool INV>
__device__ __forceinline__ float2 eighth(float2 w) {
  constexpr float c = 0.70710678118654752f;
  return INV ? make_float2(c * (w.x - w.y), c * (w.x + w.y))
             : make_float2(c * (w.x + w.y), c * (w.y - w.x));
}
// The same butterflies for w = W16^m alone (m = 0..7), without its trivial
// products.
template <bool INV>
__device__ __forceinline__ void bf2_w16(float2 &a, float2 &b, int m) {
  const float2 p = a, q = b;
  if (m == 0) {
    a = cadd(p, q);
    b = csub(p, q);
  } else if (m == 4) {
    const float2 iq = quarter<INV>(q);
    a = cadd(p, iq);
    b = csub(p, iq);
  } else if (m == 2 || m == 6) {  // c (s, d) or c (d', -s') of the sums
    constexpr float c = 0.70710678118654752f;
    const float s = q.x + q.y, d = q.y - q.x;
    // W16^2 q = c (s, d), W16^6 q = c (d, -s); conjugated: c (-d, s) and
    // c (-s, -d).
    const float2 e = m == 2 ? (INV ? make_float2(-d, s) : make_float2(s, d))
                            : (INV ? make_float2(-s, -d) : make_float2(d, -s));
    a = make_float2(fmaf(c, e.x, p.x), fmaf(c, e.y, p.y));
    b = make_float2(fmaf(-c, e.x, p.x), fmaf(-c, e.y, p.y));
  } else {
    const float2 w = w16(m);
    bf2(a, b, INV ? make_float2(w.x, -w.y) : w);
  }
}

// Stages 2 to 4 of the untwiddled 16-point DFT (stage 1, the pairs (n, n +
// 8), done), natural order out.  NZ as in dft16_fma.
template <bool INV, int NZ>
__device__ __forceinline__ void dft16_tail(float2 *v) {
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    if (n + 4 < NZ) {
      bf2_w16<INV>(v[n], v[n + 4], 0);
      bf2_w16<INV>(v[n + 8], v[n + 12], 4);
    } else {
      v[n + 4] = v[n];
      v[n + 12] = v[n + 8];
    }
  }
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    bf2_w16<INV>(v[n], v[n + 2], 0);
    bf2_w16<INV>(v[n + 8], v[n + 10], 2);
    bf2_w16<INV>(v[n + 4], v[n + 6], 4);
    bf2_w16<INV>(v[n + 12], v[n + 14], 6);
  }
  float2 t[16];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    // C_0[k], C_1[k] sit at the bit reversal of k (four bits, low one 0).
    const int p = 8 * (k & 1) + 4 * ((k >> 1) & 1) + 2 * (k >> 2);
    bf2_w16<INV>(v[p], v[p + 1], k);
    t[k] = v[p];
    t[k + 8] = v[p + 1];
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = t[i];
}

// 16-point DFT in place, natural order in and out, of which only inputs 0 ..
// NZ-1 can be nonzero (NZ 4..8 or 16; the others are not read).
template <bool INV, int NZ = 16>
__device__ __forceinline__ void dft16_fma(float2 *v) {
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    if (NZ == 16)
      bf2_w16<INV>(v[n], v[n + 8], 0);
    else
      v[n + 8] = v[n];
  }
  dft16_tail<INV, NZ>(v);
}

// The external twiddle of a radix-16 butterfly: w and its powers 2, 4 and 8.
struct Tw16 {
  float2 w, w2, w4, w8;
  template <bool CONJ>
  __device__ __forceinline__ Tw16 conj_if() const {
    if (!CONJ) return *this;
    return {make_float2(w.x, -w.y), make_float2(w2.x, -w2.y),
            make_float2(w4.x, -w4.y), make_float2(w8.x, -w8.y)};
  }
};

// 16-point DFT of v[r] w^r (r = 0..15), natural order in and out; HI: only
// outputs 8..15 are formed.  w is the twiddle as it multiplies (conjugated
// by the caller for an inverse transform).
template <bool INV, bool HI = false>
__device__ __forceinline__ void dft16_twiddled(float2 *v, const Tw16 &tw) {
  const float2 w = tw.w, w2 = tw.w2, w4 = tw.w4, w8 = tw.w8;
#pragma unroll
  for (int n = 0; n < 8; ++n) bf2(v[n], v[n + 8], w8);
  const float2 w4q = quarter<INV>(w4);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    bf2(v[n], v[n + 4], w4);
    bf2(v[n + 8], v[n + 12], w4q);
  }
  const float2 w2e = eighth<INV>(w2), w2q = quarter<INV>(w2),
               w2s = quarter<INV>(w2e);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    bf2(v[n], v[n + 2], w2);
    bf2(v[n + 8], v[n + 10], w2e);
    bf2(v[n + 4], v[n + 6], w2q);
    bf2(v[n + 12], v[n + 14], w2s);
  }
  float2 t[16], wk[8];
  wk[0] = w;
  wk[1] = INV ? cmulc(w, w16(1)) : cmul(w, w16(1));
  wk[2] = eighth<INV>(w);
  wk[3] = INV ? cmulc(w, w16(3)) : cmul(w, w16(3));
#pragma unroll
  for (int k = 0; k < 4; ++k) wk[k + 4] = quarter<INV>(wk[k]);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int p = 8 * (k & 1) + 4 * ((k >> 1) & 1) + 2 * (k >> 2);
    if (HI)
      bf2_diff(v[p], v[p + 1], wk[k]);
    else
      bf2(v[p], v[p + 1], wk[k]);
    t[k] = v[p];
    t[k + 8] = v[p + 1];
  }
#pragma unroll
  for (int i = HI ? 8 : 0; i < 16; ++i) v[i] = t[i];
}

// 4-point DFT of (a, b w, c w^2, d w^3), w2 = w^2.
template <bool INV>
__device__ __forceinline__ void dft4_twiddled(float2 &a, float2 &b, float2 &c,
                                              float2 &d, float2 w, float2 w2) {
  bf2(a, c, w2);
  bf2(b, d, w2);
  bf2(a, b, w);                // outputs 0, 2
  bf2(c, d, quarter<INV>(w));  // outputs 1, 3
  const float2 t = b;
  b = c;
  c = t;
}

// Returns x unchanged but hides that from the optimiser, so that loads
// indexed by it are not hoisted out of an enclosing loop (which would keep
// tables of twiddles or taps live in registers across the whole loop).
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// LDS index with one pad slot every 16 entries (spreads banks).
__device__ __forceinline__ int pad16(int i) { return i + (i >> 4); }

// Row swaps across the wavefront (gfx950 v_permlane32/16_swap): with rows
// of 16 lanes, swap_rows32 exchanges rows 2, 3 of a with rows 0, 1 of b;
// swap_rows16 exchanges rows 1, 3 of a with rows 0, 2 of b.
__device__ __forceinline__ void swap_rows32(float2 &a, float2 &b) {
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a.x),
                                                  __float_as_uint(b.x), false,
                                                  false);
  const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(a.y),
                                                  __float_as_uint(b.y), false,
                                                  false);
  a = make_float2(__uint_as_float(x[0]), __uint_as_float(y[0]));
  b = make_float2(__uint_as_float(x[1]), __uint_as_float(y[1]));
}
__device__ __forceinline__ void swap_rows16(float2 &a, float2 &b) {
  const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.x),
                                                  __float_as_uint(b.x), false,
                                                  false);
  const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.y),
                                                  __float_as_uint(b.y), false,
                                                  false);
  a = make_float2(__uint_as_float(x[0]), __uint_as_float(y[0]));
  b = make_float2(__uint_as_float(x[1]), __uint_as_float(y[1]));
}

// After pass 1 of the 1024-point per-wave transform (radix 16, 16, 4), lane
// j holds output (j / 16) 256 + j mod 16 + 16 r in v[r]; the radix-4
// butterfly j + 64 q of pass 2 needs elements j + 64 q + 256 m (m < 4),
// held in v[4 q + j / 16] of lanes j mod 16 + 16 m.  Transposing, in each
// group of four registers, the lane's row of 16 against the register's low
// two bits (two swap steps across rows, no LDS) leaves element
// j + 64 q + 256 m in v[4 q + m].
__device__ __forceinline__ void pass2_gather(float2 *v) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    swap_rows32(v[4 * q], v[4 * q + 2]);
    swap_rows32(v[4 * q + 1], v[4 * q + 3]);
    swap_rows16(v[4 * q], v[4 * q + 1]);
    swap_rows16(v[4 * q + 2], v[4 * q + 3]);
  }
}

}  // namespace lp
