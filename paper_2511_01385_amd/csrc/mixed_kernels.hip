// mixed_kernels.hip -- rdFFT rows whose half-length has factors 3 and 5.
//
// Even n = 2N with N = 2^a 3^b 5^c that is not a power of two, N <= 16384.  The
// transform is the one of the power-of-two kernels (Sec. 4.1): the N-point complex DFT of
// z_m = x_{2m} + i x_{2m+1} followed by the post-pass that pairs bins k and N-k, and the
// inverse pre-pass (1/n folded in) followed by the conjugate passes.  A row's N complex
// points pass through LDS between Stockham passes whose radices (up to 16: the composite 6,
// 9, 10, 12 and 15 beside the powers of two) a host plan picks at run time; a butterfly's first
// and fourth twiddle powers come from Taylor sums of sine and cosine (the fourth of 16-bit rows, at
// radix 9 and more, from the hardware functions) and the others from products, so these plans need no table.
//
// What bounds them: VALU work and the waits between passes in 16-bit storage, HBM in float32.
// n = 6144 (16 16 12, 12 points a thread, about 1010 VALU instructions per wave), 16384 rows, takes 95
// us forward and 113 us inverse in bf16 (4.2 and 3.6 TB/s), 149 us each in float32 (5.4 TB/s).  Radices up to
// 8, always 16 points per thread and the row staged through LDS before its
// first and after its last pass (five passes, 1740 instructions for 16 points) took 200 and 208 us,
// 231 and 192 us; 65536 rows of n = 96, each in a workgroup of its own then, 48 us against 9 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fft_device.hpp"
#include "launch.hpp"

namespace rdfft {

namespace {

constexpr int kMixedMaxPasses = 16;
constexpr int kMixedLdsF2 = 160 * 1024 / 8;  // float2 of LDS per workgroup

// One Stockham pass: butterfly j < B = N/R reads in[j + r*B], multiplies input r by
// W_{Ns*R}^{r*k} (k = j mod Ns), runs the R-point DFT and writes out[(j/Ns)*Ns*R + k + r*Ns].
// In LDS, every block of Ns*R outputs is followed by `pad` unused slots (element e lies at
// e + pad*floor(e/(Ns*R))), which spreads the strided writes over the banks; as the next pass's
// stride N/R' is a multiple of Ns*R, its reads stay at a base plus r times one step.
struct MixedPass {
  int R, B, Ns, pad_in, pad_out, step_in;  // step_in: LDS slots between inputs r and r+1
  float inv_ns, inv_den;                   // 1/Ns, 1/(Ns*R)
};
struct MixedPlan {
  int n_half;   // N
  int passes;
  int tpr;      // threads of a row, for the variant that the launch picks
  int log_tpr;  // of a row that shares its workgroup (a power of two), else -1
  int rows_wg;  // rows per workgroup
  int lds_f2;   // LDS slots of a row
  int waves[3];      // by variant (kHold...): waves of a row's workgroup, 0 where 16 do not do
  int per_cu[2][3];  // by direction and variant: workgroups per CU
  MixedPass pass[kMixedMaxPasses];
};

// -i * a (forward) or +i * a (inverse)
template <bool INV>
__device__ __forceinline__ float2 mul_mi(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

template <int R, bool INV>
__device__ __forceinline__ void dft_any(float2* v);

template <int R, bool INV>
struct DftOdd;

// 3 points: y1, y2 = (v0 - (v1+v2)/2) -+ i (sqrt(3)/2) (v1 - v2)
template <bool INV>
struct DftOdd<3, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    constexpr float s3 = 0.866025403784438646763723f;  // sin(2 pi / 3)
    const float2 a = c_add(v[1], v[2]), d = mul_mi<INV>(c_sub(v[1], v[2]));
    const float2 t = make_float2(fmaf(-0.5f, a.x, v[0].x), fmaf(-0.5f, a.y, v[0].y));
    v[0] = c_add(v[0], a);
    v[1] = make_float2(fmaf(s3, d.x, t.x), fmaf(s3, d.y, t.y));
    v[2] = make_float2(fmaf(-s3, d.x, t.x), fmaf(-s3, d.y, t.y));
  }
};

// 5 points with c1 = cos(2 pi/5), c2 = cos(4 pi/5), s1 = sin(2 pi/5), s2 = sin(4 pi/5):
//   y1, y4 = v0 + c1 (v1+v4) + c2 (v2+v3) -+ i (s1 (v1-v4) + s2 (v2-v3))
//   y2, y3 = v0 + c2 (v1+v4) + c1 (v2+v3) -+ i (s2 (v1-v4) - s1 (v2-v3))
template <bool INV>
struct DftOdd<5, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    constexpr float c1 = 0.309016994374947424102293f, c2 = -0.809016994374947424102293f;
    constexpr float s1 = 0.951056516295153572116439f, s2 = 0.587785252292473129168706f;
    const float2 a1 = c_add(v[1], v[4]), a2 = c_add(v[2], v[3]);
    const float2 b1 = c_sub(v[1], v[4]), b2 = c_sub(v[2], v[3]);
    const float2 v0 = v[0];
    const float2 t1 = make_float2(fmaf(c2, a2.x, fmaf(c1, a1.x, v0.x)), fmaf(c2, a2.y, fmaf(c1, a1.y, v0.y)));
    const float2 t2 = make_float2(fmaf(c1, a2.x, fmaf(c2, a1.x, v0.x)), fmaf(c1, a2.y, fmaf(c2, a1.y, v0.y)));
    const float2 u1 = make_float2(fmaf(s2, b2.x, s1 * b1.x), fmaf(s2, b2.y, s1 * b1.y));
    const float2 u2 = make_float2(fmaf(-s1, b2.x, s2 * b1.x), fmaf(-s1, b2.y, s2 * b1.y));
    v[0] = c_add(v0, c_add(a1, a2));
    const float2 iu1 = mul_mi<INV>(u1), iu2 = mul_mi<INV>(u2);
    v[1] = c_add(t1, iu1);
    v[4] = c_sub(t1, iu1);
    v[2] = c_add(t2, iu2);
    v[3] = c_sub(t2, iu2);
  }
};

// 9 points as 3 x 3 (n = 3 n1 + n2, k = k1 + 3 k2): W_9^{n2 k1} between the two layers
template <bool INV>
struct DftOdd<9, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    // exp(-2 pi i m / 9), m = 1, 2, 4
    constexpr float2 w1 = {0.766044443118978035202393f, -0.642787609686539326322643f};
    constexpr float2 w2 = {0.173648177666930348851717f, -0.984807753012208059366743f};
    constexpr float2 w4 = {-0.939692620785908384054109f, -0.342020143325668733044100f};
    float2 u[3][3];
    static_for<3>([&](auto n2c) {
      constexpr int n2 = decltype(n2c)::value;
      static_for<3>([&](auto n1c) { u[n2][decltype(n1c)::value] = v[3 * decltype(n1c)::value + n2]; });
      DftOdd<3, INV>::run(u[n2]);
    });
    u[1][1] = c_mul<INV>(u[1][1], w1);
    u[1][2] = c_mul<INV>(u[1][2], w2);
    u[2][1] = c_mul<INV>(u[2][1], w2);
    u[2][2] = c_mul<INV>(u[2][2], w4);
    static_for<3>([&](auto k1c) {
      constexpr int k1 = decltype(k1c)::value;
      float2 w[3] = {u[0][k1], u[1][k1], u[2][k1]};
      DftOdd<3, INV>::run(w);
      static_for<3>([&](auto k2c) { v[k1 + 3 * decltype(k2c)::value] = w[decltype(k2c)::value]; });
    });
  }
};

// A*C points for coprime A and C without twiddles (Good's prime-factor mapping): input
// n = (C n1 + A n2) mod AC; output k with k mod A = k1 and k mod C = k2.
template <int A, int C, bool INV>
struct DftCoprime {
  static constexpr int out_index(int k1, int k2) {
    for (int k = 0; k < A * C; ++k)
      if (k % A == k1 && k % C == k2) return k;
    return 0;
  }
  __device__ __forceinline__ static void run(float2* v) {
    float2 u[C][A];
    static_for<C>([&](auto n2c) {
      constexpr int n2 = decltype(n2c)::value;
      static_for<A>([&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value;
        u[n2][n1] = v[(C * n1 + A * n2) % (A * C)];
      });
      // sum over n1 of W^{C n1 k} = W_A^{n1 k}: an A-point DFT in k mod A
      dft_any<A, INV>(u[n2]);
    });
    static_for<A>([&](auto k1c) {
      constexpr int k1 = decltype(k1c)::value;
      float2 w[C];
      static_for<C>([&](auto n2c) { w[decltype(n2c)::value] = u[decltype(n2c)::value][k1]; });
      dft_any<C, INV>(w);
      static_for<C>([&](auto k2c) { v[out_index(k1, decltype(k2c)::value)] = w[decltype(k2c)::value]; });
    });
  }
};

template <int R, bool INV>
__device__ __forceinline__ void dft_any(float2* v) {
  if constexpr (R == 3 || R == 5 || R == 9) DftOdd<R, INV>::run(v);
  else if constexpr (R == 6) DftCoprime<2, 3, INV>::run(v);
  else if constexpr (R == 10) DftCoprime<2, 5, INV>::run(v);
  else if constexpr (R == 12) DftCoprime<4, 3, INV>::run(v);
  else if constexpr (R == 15) DftCoprime<3, 5, INV>::run(v);
  else Dft<R, INV>::run(v);
}

// cosine and sine of f quarter turns, |f| <= 1/2, as Taylor sums (remainders below 2e-9): the
// coefficients are (pi/2)^k / k! with alternating signs
__device__ __forceinline__ float2 cos_sin_quarters(float f) {
  const float z = f * f;
  const float s = f * fmaf(z, fmaf(z, fmaf(z, fmaf(z, 1.60441184787359822e-4f, -4.68175413531868810e-3f),
                                           7.96926262461670452e-2f), -6.45964097506246253e-1f), 1.57079632679489662f);
  const float c = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, -2.52020423730606055e-5f, 9.19260274839426581e-4f),
                                               -2.08634807633529609e-2f), 2.53669507901048014e-1f),
                               -1.23370055013616983f), 1.0f);
  return make_float2(c, s);
}

// exp(-+ 2 pi i num / den) for 0 <= num < den; the caller passes inv_den = 1/den.  FINE: the angle
// is reduced to |f| <= 1/2 quarter turns in integers, so that its rounding is relative to f.  Else the
// hardware sine and cosine of the angle in revolutions, a few 1e-7 off.
template <bool INV, bool FINE>
__device__ __forceinline__ float2 unit_root(int num, int den, float inv_den) {
  if constexpr (FINE) {
    const int q = (int)rintf((float)(4 * num) * inv_den);  // nearest quarter turn
    const float2 w = cos_sin_quarters((float)(4 * num - q * den) * inv_den);
    const bool odd = (q & 1) != 0;
    const float x = odd ? w.y : w.x, y = odd ? w.x : w.y;
    const uint32_t flip_x = (uint32_t)((q + 1) & 2) << 30, flip_y = (uint32_t)((q & 2) ^ (INV ? 0 : 2)) << 30;
    return make_float2(__uint_as_float(__float_as_uint(x) ^ flip_x), __uint_as_float(__float_as_uint(y) ^ flip_y));
  } else {
    const float x = (float)num * inv_den;  // revolutions
    const float s = __builtin_amdgcn_sinf(x), c = __builtin_amdgcn_cosf(x);
    return make_float2(c, INV ? s : -s);
  }
}

// Multiplies input r of a butterfly of radix R by w^r, w = exp(-+ 2 pi i k / (Ns R)), k < Ns.
// Products carry a root's error once per factor: so w comes from Taylor sums in every storage type
// (from radix 8 on it lies within 1/8 turn and needs no reduction), and from radix 6 on w^4 is a
// root of its own, so that w^15 = (w^4)^3 w^3 has six errors, not fifteen: by Taylor sums too, but for
// 16-bit rows of radix 9 and more, which the hardware functions serve within the old error (below) and 3 %
// sooner.
// (With the hardware functions for w and all powers from it, n = 6144 had a float32 error of 6.7e-7, and
// 0.32 % of its float16 results fell on the wrong side of a rounding, plans of radices up to 8 before:
// 4.3e-7 and 0.22 %; now 1.6e-7 and 0.15 %.  2^26 bf16 values, forward and inverse: 119 us then and now.)
template <bool INV, int R, bool FINE>
__device__ __forceinline__ void twiddle(float2* v, int k, int den, float inv_den) {
  float2 w[R];
  if constexpr (R < 8) {
    w[1] = unit_root<INV, true>(k, den, inv_den);
  } else {
    const float2 cs = cos_sin_quarters((float)(4 * k) * inv_den);
    w[1] = make_float2(cs.x, INV ? cs.y : -cs.y);
  }
  if constexpr (R > 5) w[4] = unit_root<INV, FINE || R <= 8>(4 * k, den, inv_den);
  static_for<R - 1>([&](auto rc) {
    constexpr int r = decltype(rc)::value + 1;
    if constexpr (r == 2 || (r == 4 && R == 5) || r == 8) w[r] = c_mul<false>(w[r / 2], w[r / 2]);
    else if constexpr (r == 3) w[r] = c_mul<false>(w[2], w[1]);
    else if constexpr (r == 12) w[r] = c_mul<false>(w[8], w[4]);
    else if constexpr (r > 4) w[r] = c_mul<false>(w[r & ~3], w[r & 3]);
    v[r] = c_mul<false>(v[r], w[r]);
  });
}

// Pairs of the pre-pass whose loads a thread has in flight at a time: one pair at a time left the
// inverse waiting for HBM (n = 6144 bf16, 16384 rows: 160 us; 116 us with four).  The forward's
// post-pass reads LDS and gained nothing from it.
constexpr int kMixedAhead = 4;

// The kernel's variants: butterflies of one pass that a thread can hold.  One; as many as 16
// values make; or one more where 16 is no multiple of the radix, which fits any row in 1024 threads.
enum { kHoldOne, kHoldSome, kHoldMany };
constexpr int held(int R, int hold) { return hold == kHoldOne ? 1 : hold == kHoldSome ? 16 / R : (15 + R) / R; }
// waves per SIMD that the registers of a variant leave
constexpr int held_waves(int hold, bool inv) { return hold == kHoldOne ? 7 : hold == kHoldMany ? 4 : inv ? 6 : 5; }

// read(r-th input position) / write as functors of an LDS slot or global pair index; a pass
// that reads or writes LDS on both sides has a barrier between its reads and its writes.
template <int R, bool INV, int HOLD, bool FROM_GLOBAL, bool TO_GLOBAL, class Acc>
__device__ __forceinline__ void mixed_pass(const MixedPass& p, int t, int tpr, bool active, float2* lds, const Acc& acc) {
  constexpr int MB = held(R, HOLD);
  constexpr bool FINE = std::is_same<typename Acc::raw_t, float2>::value;
  float2 v[MB][R];
  int kk[MB], qq[MB];
#pragma unroll
  for (int s = 0; s < MB; ++s) {
    const int j = t + s * tpr;
    // j / Ns: exact, as (j + 1/2) / Ns stays 1/(2 Ns) away from any integer and j < 2^14
    qq[s] = FROM_GLOBAL ? j : (int)(((float)j + 0.5f) * p.inv_ns);
    kk[s] = FROM_GLOBAL ? 0 : j - qq[s] * p.Ns;
    if (j < p.B) {
      if constexpr (FROM_GLOBAL) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[s][r] = acc.load(j + r * p.B);
      } else {
        const float2* in = lds + j + qq[s] * p.pad_in;
#pragma unroll
        for (int r = 0; r < R; ++r) v[s][r] = in[r * p.step_in];
      }
    }
  }
  if constexpr (!FROM_GLOBAL) __syncthreads();
#pragma unroll
  for (int s = 0; s < MB; ++s) {
    const int j = t + s * tpr;
    if (j < p.B) {
      if constexpr (!FROM_GLOBAL) {
        if (p.Ns > 1) twiddle<INV, R, FINE>(v[s], kk[s], p.Ns * R, p.inv_den);
      }
      dft_any<R, INV>(v[s]);
      const int o = (j - kk[s]) * R + kk[s];
      if constexpr (TO_GLOBAL) {
        if (active) {
#pragma unroll
          for (int r = 0; r < R; ++r) acc.store(o + r * p.Ns, v[s][r]);
        }
      } else {
        float2* out = lds + o + qq[s] * p.pad_out;
#pragma unroll
        for (int r = 0; r < R; ++r) out[FROM_GLOBAL ? r : r * p.Ns] = v[s][r];
      }
    }
  }
  if constexpr (!TO_GLOBAL) __syncthreads();
}

template <bool INV, int HOLD, bool FROM_GLOBAL, bool TO_GLOBAL, class Acc>
__device__ __forceinline__ void mixed_pass_any(const MixedPass& p, int t, int tpr, bool active, float2* lds,
                                               const Acc& acc) {
  switch (p.R) {
    case 2: mixed_pass<2, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 3: mixed_pass<3, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 4: mixed_pass<4, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 5: mixed_pass<5, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 6: mixed_pass<6, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 8: mixed_pass<8, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 9: mixed_pass<9, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 10: mixed_pass<10, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 12: mixed_pass<12, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    case 15: mixed_pass<15, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
    default: mixed_pass<16, INV, HOLD, FROM_GLOBAL, TO_GLOBAL>(p, t, tpr, active, lds, acc); break;
  }
}

// A workgroup owns rows_wg rows of tpr threads each.  The forward's first pass reads the row
// from global memory and its post-pass writes it; the inverse's pre-pass reads it and its
// last pass writes it.  Every load of a row precedes its first store (barriers between).
// HC: the spectrum (the forward's output, the inverse's input) in the halfcomplex layout.
template <class Acc, class Elem, bool INV, bool HC, int HOLD>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(held_waves(HOLD, INV))))
mixed_rows_kernel(Elem* buf, int64_t rows, MixedPlan plan) {
  extern __shared__ float2 mixed_lds[];
  constexpr bool FINE = std::is_same<typename Acc::raw_t, float2>::value;
  const int N = plan.n_half, T = plan.tpr;
  const int rho = plan.log_tpr >= 0 ? (int)threadIdx.x >> plan.log_tpr : 0;
  const int t = (int)threadIdx.x - rho * T;
  const int64_t row = (int64_t)blockIdx.x * plan.rows_wg + rho;
  const bool active = row < rows;
  float2* const lds = mixed_lds + (size_t)rho * plan.lds_f2;
  Elem* const rp = buf + (active ? row : 0) * (int64_t)N;
  const Acc sig{rp};                                // the signal pairs (x_{2m}, x_{2m+1})
  const auto spec = spectrum_view<HC, Acc>(rp, N);  // the packed spectrum
  if constexpr (!INV) {
    mixed_pass_any<INV, HOLD, true, false>(plan.pass[0], t, T, active, lds, sig);
    for (int q = 1; q < plan.passes; ++q) mixed_pass_any<INV, HOLD, false, false>(plan.pass[q], t, T, active, lds, sig);
    if (!active) return;
    // post-pass: Y_k = s/2 + (-i W_n^k / 2) d, Y_{N-k} = conj(s/2 - (-i W_n^k / 2) d) with
    // s = Z_k + conj(Z_{N-k}), d = Z_k - conj(Z_{N-k}); slot 0 = (Y_0, Y_{n/2})
    const float inv_n = 1.0f / (float)(2 * N);
    for (int k = t; 2 * k <= N; k += T) {
      const float2 a = lds[k];
      if (k == 0) {
        spec.store(0, make_float2(a.x + a.y, a.x - a.y));
        continue;
      }
      const float2 b = c_conj(lds[N - k]);
      const float2 s = c_add(a, b), d = c_sub(a, b);
      const float2 w = unit_root<false, FINE>(k, 2 * N, inv_n);  // W_n^k
      const float2 q = c_mul<false>(d, make_float2(0.5f * w.y, -0.5f * w.x));  // -i W_n^k d / 2
      spec.store(k, make_float2(fmaf(s.x, 0.5f, q.x), fmaf(s.y, 0.5f, q.y)));
      if (2 * k != N) spec.store(N - k, make_float2(fmaf(s.x, 0.5f, -q.x), -fmaf(s.y, 0.5f, -q.y)));
    }
  } else {
    // pre-pass: Z~_m = (s + i conj(W_n^m) d) / n, Z~_{N-m} = conj(s - i conj(W_n^m) d) / n with
    // s = Y_m + conj(Y_{N-m}), d = Y_m - conj(Y_{N-m}); slot 0 holds (Y_0, Y_{n/2})
    const float sc = 1.0f / (2.0f * N), inv_n = 1.0f / (float)(2 * N);
    for (int m0 = t; 2 * m0 <= N; m0 += kMixedAhead * T) {
      typename Acc::raw_t ra[kMixedAhead], rb[kMixedAhead];
      static_for<kMixedAhead>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        const int m = m0 + u * T;
        const bool in = 2 * m <= N;
        ra[u] = spec.load_raw(in ? m : 0);
        rb[u] = spec.load_raw(in && m != 0 ? N - m : 0);
      });
      static_for<kMixedAhead>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        const int m = m0 + u * T;
        if (2 * m <= N) {
          const float2 ya = Acc::widen(ra[u]), yb = c_conj(Acc::widen(rb[u]));
          const float2 s = c_add(ya, yb), d = c_sub(ya, yb);
          const float2 w = unit_root<true, FINE>(m, 2 * N, inv_n);         // conj(W_n^m)
          const float2 q = c_mul<false>(d, make_float2(-sc * w.y, sc * w.x));  // i conj(W_n^m) d / n
          const float2 lo = make_float2(fmaf(s.x, sc, q.x), fmaf(s.y, sc, q.y));
          lds[m] = m == 0 ? make_float2(sc * (ya.x + ya.y), sc * (ya.x - ya.y)) : lo;
          if (m != 0 && 2 * m != N) lds[N - m] = make_float2(fmaf(s.x, sc, -q.x), -fmaf(s.y, sc, -q.y));
        }
      });
    }
    __syncthreads();
    for (int q = 0; q + 1 < plan.passes; ++q)
      mixed_pass_any<INV, HOLD, false, false>(plan.pass[q], t, T, active, lds, sig);
    mixed_pass_any<INV, HOLD, false, true>(plan.pass[plan.passes - 1], t, T, active, lds, sig);
  }
}

// The variant for rows with a workgroup each.  What a variant with few butterflies per thread gains in
// waves it loses in rows per CU, whose passes cover one another's barriers and loads; and its waves
// are mostly idle but in the pass with the most butterflies.  So: the first variant that holds all
// rows at once or, beyond that, the one with the most rows per CU, the first among equals.
// (2^26 float32 values, inverse, one butterfly per thread -- in plans of radices up to 8 and 4 to 16 waves
// -- by this rule: n = 8000 (5 10 8 10) 176 -- 97 -- 95 us; n = 6250 (fives) 172 -- 107 -- 101 us; n = 9000
// (15 10 6 5) 190 -- 151 -- 101 us.  Rows per CU are no more than an estimate of the time: n = 5832 bf16 forward
// takes 95 us by it, 73 with one butterfly per thread.)
int pick_hold(const int* per_cu, int64_t rows, int num_cu) {
  int best = kHoldMany;
  for (int h : {kHoldMany, kHoldSome, kHoldOne}) {
    if (per_cu[h] == 0) continue;
    if (per_cu[h] >= per_cu[best] || rows <= (int64_t)num_cu * per_cu[h]) best = h;
  }
  return best;
}

template <class K>
hipError_t allow_lds(K kernel) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             160 * 1024);
}

template <class Acc, class Elem, bool INV, bool HC, int HOLD>
hipError_t launch_mixed_t(void* buf, int64_t rows, const MixedPlan& plan, hipStream_t stream) {
  static const hipError_t attr = allow_lds(mixed_rows_kernel<Acc, Elem, INV, HC, HOLD>);
  if (attr != hipSuccess) return attr;
  const int threads = plan.tpr * plan.rows_wg;
  const size_t lds = (size_t)plan.lds_f2 * plan.rows_wg * sizeof(float2);
  Elem* base = static_cast<Elem*>(buf);
  const int64_t max_rows = kMaxGridThreads / threads * plan.rows_wg;
  for (int64_t r0 = 0; r0 < rows; r0 += max_rows) {
    const int64_t nr = std::min<int64_t>(max_rows, rows - r0);
    hipLaunchKernelGGL((mixed_rows_kernel<Acc, Elem, INV, HC, HOLD>),
                       dim3((unsigned)((nr + plan.rows_wg - 1) / plan.rows_wg)), dim3(threads), lds, stream,
                       base + r0 * plan.n_half, nr, plan);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template <class Acc, class Elem, bool INV, bool HC>
hipError_t launch_mixed(void* buf, int64_t rows, const MixedPlan& made, hipStream_t stream, int num_cu) {
  MixedPlan plan = made;
  int hold = kHoldOne;
  if (plan.tpr == 0) {  // rows with a workgroup of their own
    hold = pick_hold(plan.per_cu[INV], rows, num_cu);
    plan.tpr = 64 * plan.waves[hold];
  }
  // few short rows: no more of them to a workgroup than fill a wave, while some CU has none
  // (n = 384, 341 float32 rows: 22 workgroups 5.2 us, 86 4.8 us; one row each 6.5 us)
  while (plan.rows_wg > 1 && plan.rows_wg * plan.tpr > 64 && rows < (int64_t)num_cu * plan.rows_wg) plan.rows_wg /= 2;
  if (hold == kHoldOne) return launch_mixed_t<Acc, Elem, INV, HC, kHoldOne>(buf, rows, plan, stream);
  if (hold == kHoldSome) return launch_mixed_t<Acc, Elem, INV, HC, kHoldSome>(buf, rows, plan, stream);
  return launch_mixed_t<Acc, Elem, INV, HC, kHoldMany>(buf, rows, plan, stream);
}

constexpr int kMixedRadices[] = {16, 15, 12, 10, 9, 8, 6, 5, 4, 3, 2};

// VALU instructions of a radix-R butterfly: its DFT, R-1 twiddle products and the R-2 powers
// they need, and its LDS addresses, plus the fixed cost of a pass per butterfly
double butterfly_cost(int R) {
  static const double dft[17] = {0, 0, 4, 14, 16, 36, 40, 0, 52, 100, 92, 0, 104, 0, 0, 178, 148};
  return dft[R] + 8.0 * (R - 1) + 2.0 * R + 30.0;
}

// Radices of a plan (fixed storage: plans are made inside the C entry points, which must not throw)
struct Radices {
  int count = 0;
  int r[kMixedMaxPasses];
};

// The cheapest factorisation of m into radices no larger than kMixedRadices[from] (largest first)
void best_radices(int n_half, int m, int from, double cost, Radices* cur, Radices* best, double* best_cost) {
  if (cost >= *best_cost) return;
  if (m == 1) {
    *best = *cur;
    *best_cost = cost;
    return;
  }
  if (cur->count == kMixedMaxPasses) return;
  for (int i = from; i < (int)(sizeof(kMixedRadices) / sizeof(int)); ++i) {
    const int R = kMixedRadices[i];
    if (m % R != 0) continue;
    cur->r[cur->count++] = R;
    best_radices(n_half, m / R, i, cost + (double)(n_half / R) * butterfly_cost(R), cur, best, best_cost);
    --cur->count;
  }
}

// The plan of N = 2^a 3^b 5^c.  Radices: the cheapest factorisation by VALU instructions.  An
// odd radix comes first when there is one (its outputs, R apart, then need no padding), the
// others in falling order.  Short rows share a workgroup, with one butterfly per thread in the pass
// with the most of them; longer ones get the threads of each variant of the kernel (pick_hold).
bool make_plan(int64_t n_half, MixedPlan* plan) {
  if (n_half < 1 || n_half > kMixedMaxHalf || (n_half & (n_half - 1)) == 0) return false;
  int m = (int)n_half;
  for (int f : {2, 3, 5})
    while (m % f == 0) m /= f;
  if (m != 1) return false;
  const int N = (int)n_half;
  Radices cur, radices;
  double cost = 1e30;
  best_radices(N, N, 0, 0.0, &cur, &radices, &cost);
  if (radices.count == 0) return false;
  for (int i = 0; i < radices.count; ++i)
    if (radices.r[i] & 1) {
      std::swap(radices.r[0], radices.r[i]);
      break;
    }
  plan->n_half = N;
  plan->passes = radices.count;
  int Ns = 1, pad_in = 0, lds = N;
  int need[3] = {0, 0, 0};  // threads of a row that holds one, some or many butterflies each
  for (int q = 0; q < plan->passes; ++q) {
    MixedPass& p = plan->pass[q];
    const int R = radices.r[q], M = Ns * R;
    p.R = R;
    p.B = N / R;
    p.Ns = Ns;
    p.inv_ns = 1.0f / (float)Ns;
    p.inv_den = 1.0f / (float)M;
    p.pad_in = pad_in;
    p.step_in = p.B + pad_in * (p.B / Ns);
    // the writes of neighbouring lanes: runs of Ns slots M apart.  Sixteen lanes cover 16 slots of
    // two banks each: with M + pad = Ns (mod 16) the runs follow one another on the banks
    int pad = 0;
    if (q + 1 < plan->passes && Ns < 16) {
      pad = (((Ns - M) % 16) + 16) % 16;
      if (pad * 8 > M) pad = M % 2 == 0 ? 1 : 0;
      if (Ns == 1) pad = R % 2 == 0 ? 1 : 0;
      if (N + pad * (N / M) > kMixedLdsF2) pad = 0;
    }
    p.pad_out = pad_in = pad;
    lds = std::max(lds, N + pad * (N / M));
    for (int h : {kHoldOne, kHoldSome, kHoldMany}) need[h] = std::max(need[h], (p.B + held(R, h) - 1) / held(R, h));
    Ns = M;
  }
  plan->lds_f2 = lds;
  plan->tpr = 0;
  plan->rows_wg = 1;
  plan->log_tpr = -1;
  if (need[kHoldOne] <= 128) {
    plan->log_tpr = 0;
    while ((1 << plan->log_tpr) < need[kHoldOne]) ++plan->log_tpr;
    plan->tpr = 1 << plan->log_tpr;
    while (plan->rows_wg * 2 * plan->tpr <= 256 && plan->rows_wg * 2 * lds <= kMixedLdsF2 / 4) plan->rows_wg *= 2;
    return true;
  }
  const int by_lds = kMixedLdsF2 / lds;
  for (int h : {kHoldOne, kHoldSome, kHoldMany}) {
    int waves = (need[h] + 63) / 64;
    // (a workgroup's waves are spread evenly over the four SIMDs)
    auto per_cu = [&](bool inv) {
      const int held = held_waves(h, inv);
      return std::min(by_lds, waves < 4 && h != kHoldMany ? 4 * held / waves : held / ((waves + 3) / 4));
    };
    // waves that the registers leave beside those workgroups shorten every pass
    if (h == kHoldMany) waves = std::max(waves, 4 * (held_waves(h, false) / per_cu(false)));
    plan->waves[h] = waves <= 16 ? waves : 0;
    for (bool inv : {false, true}) plan->per_cu[inv][h] = waves <= 16 ? per_cu(inv) : 0;
  }
  return true;
}

// The plans of all supported lengths, made once
constexpr int kMixedLengths = 186;  // 2^a 3^b 5^c up to kMixedMaxHalf but the powers of two
struct MixedPlans {
  int count = 0;
  MixedPlan plan[kMixedLengths];
};
const MixedPlan* find_plan(int64_t n_half) {
  static const MixedPlans plans = [] {
    MixedPlans v;
    for (int64_t h = 1; h <= kMixedMaxHalf && v.count < kMixedLengths; ++h)
      if (make_plan(h, &v.plan[v.count])) ++v.count;
    return v;
  }();
  const MixedPlan* end = plans.plan + plans.count;
  const MixedPlan* it =
      std::lower_bound(plans.plan, end, n_half, [](const MixedPlan& p, int64_t h) { return p.n_half < h; });
  return it != end && it->n_half == n_half ? it : nullptr;
}

// In-place pairs <-> halfcomplex conversion of one row per workgroup (the permutation of
// the power-of-two converters), staged through LDS so that every slot is read before any
// is written.  Pair slot k maps to the real slots (k, n-k), and slot 0 to (0, N).
template <class Pair, class Scalar, bool TO_HC>
__global__ void __launch_bounds__(1024) mixed_layout_kernel(Scalar* buf, int n_half) {
  extern __shared__ float2 mixed_lds[];
  Pair* lds = reinterpret_cast<Pair*>(mixed_lds);
  const int N = n_half, T = blockDim.x, t = threadIdx.x;
  Scalar* const s = buf + (int64_t)blockIdx.x * (2 * N);
  Pair* const p = reinterpret_cast<Pair*>(s);
  for (int k = t; k < N; k += T) {
    if constexpr (TO_HC) {
      lds[k] = p[k];
    } else {
      Pair v;
      v.x = s[k];
      v.y = s[k == 0 ? N : 2 * N - k];
      lds[k] = v;
    }
  }
  __syncthreads();
  for (int k = t; k < N; k += T) {
    const Pair v = lds[k];
    if constexpr (TO_HC) {
      s[k] = v.x;
      s[k == 0 ? N : 2 * N - k] = v.y;
    } else {
      p[k] = v;
    }
  }
}

struct alignas(4) Half2 {
  uint16_t x, y;
};

template <class Pair, class Scalar, bool TO_HC>
hipError_t launch_mixed_layout_t(void* buf, int64_t rows, int n_half, int threads, hipStream_t stream) {
  static const hipError_t attr = allow_lds(mixed_layout_kernel<Pair, Scalar, TO_HC>);
  if (attr != hipSuccess) return attr;
  const size_t lds = (size_t)n_half * sizeof(Pair);
  Scalar* base = static_cast<Scalar*>(buf);
  const int64_t max_rows = kMaxGridThreads / threads;
  for (int64_t r0 = 0; r0 < rows; r0 += max_rows) {
    const int64_t nr = std::min<int64_t>(max_rows, rows - r0);
    hipLaunchKernelGGL((mixed_layout_kernel<Pair, Scalar, TO_HC>), dim3((unsigned)nr), dim3(threads), lds, stream,
                       base + r0 * 2 * n_half, n_half);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// threads of a converter's workgroup: about 16 slots each
int threads_for(int64_t n_half) {
  return (int)std::min<int64_t>(1024, std::max<int64_t>(64, ((n_half + 16 * 64 - 1) / (16 * 64)) * 64));
}

}  // namespace

bool mixed_length_supported(int64_t n) {
  return n % 2 == 0 && find_plan(n / 2) != nullptr;
}

hipError_t launch_mixed_rows(void* buf, int64_t rows, int64_t n, int storage, bool inv, bool halfcomplex,
                             hipStream_t stream, int num_cu) {
  const MixedPlan* plan = find_plan(n / 2);
  if (plan == nullptr) return hipErrorInvalidValue;
  using Fn = hipError_t (*)(void*, int64_t, const MixedPlan&, hipStream_t, int);
  static const Fn table[2][3][2] = {
      {{&launch_mixed<GlobalF32, float2, false, false>, &launch_mixed<GlobalF32, float2, true, false>},
       {&launch_mixed<GlobalBF16, uint32_t, false, false>, &launch_mixed<GlobalBF16, uint32_t, true, false>},
       {&launch_mixed<GlobalF16, uint32_t, false, false>, &launch_mixed<GlobalF16, uint32_t, true, false>}},
      {{&launch_mixed<GlobalF32, float2, false, true>, &launch_mixed<GlobalF32, float2, true, true>},
       {&launch_mixed<GlobalBF16, uint32_t, false, true>, &launch_mixed<GlobalBF16, uint32_t, true, true>},
       {&launch_mixed<GlobalF16, uint32_t, false, true>, &launch_mixed<GlobalF16, uint32_t, true, true>}}};
  return table[halfcomplex ? 1 : 0][storage][inv ? 1 : 0](buf, rows, *plan, stream, num_cu);
}

}  // namespace rdfft

namespace rdfft {

hipError_t launch_mixed_layout(void* buf, int64_t rows, int64_t n, bool half16, bool to_halfcomplex,
                               hipStream_t stream) {
  if (!mixed_length_supported(n)) return hipErrorInvalidValue;
  using Fn = hipError_t (*)(void*, int64_t, int, int, hipStream_t);
  static const Fn table[2][2] = {
      {&launch_mixed_layout_t<float2, float, false>, &launch_mixed_layout_t<float2, float, true>},
      {&launch_mixed_layout_t<Half2, uint16_t, false>, &launch_mixed_layout_t<Half2, uint16_t, true>}};
  return table[half16 ? 1 : 0][to_halfcomplex ? 1 : 0](buf, rows, (int)(n / 2), threads_for(n / 2), stream);
}

}  // namespace rdfft
