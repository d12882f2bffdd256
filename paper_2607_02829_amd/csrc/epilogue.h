// GELU and the per-element GEMM epilogues (listed in gemm.hip), shared by the bf16 and fp32 GEMMs.
#pragma once
#include "common.h"
#include "sr_internal.h"

namespace sr {

// GELU(z) = z Phi(z) and GELU'(z) = Phi(z) + z phi(z) with the standard normal CDF Phi and
// density phi (exact GELU, not the tanh form).  Phi comes from erfc in the Chebyshev-fitted form
// of Press et al. (Numerical Recipes, Sec. 6.2): with x = |z|/sqrt(2) and t = 1/(1 + x/2),
// erfc(x) = t exp(-x^2 + q(t)); here q is a least-squares polynomial fit of
// log2(erfc(x) e^{x^2} / t) on t in (0, 1] (coefficients of our own fits), of degree 9 for fp32
// activations and 5 for bf16 ones.  Evaluated in fp32 the relative error of erfc is, at degree 9,
// below 2e-7 for x <= 4 and grows to 1.4e-5 near x = 8, where the rounding of the exponent
// argument (about -92) dominates; at degree 5 it stays below 4.8e-5 for x <= 8.  bf16 outputs
// round at 2e-3, forty times coarser, and the fp32 mode's gradients need the degree-9 fit.
// Branch-free, one reciprocal and one exp2; the tails have relative, not absolute, accuracy.
template <int DEG>
SR_DEV float half_erfc_of(float z, float zz) {   // 0.5 erfc(|z|/sqrt(2)), zz = z*z
  static_assert(DEG == 5 || DEG == 9, "fit degree");
  const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(z), 0.35355339059327376f, 1.0f));
  float q;
  if constexpr (DEG == 9) {
    q = 0.24651731550693512f;
    q = fmaf(q, t, -1.1861149072647095f);
    q = fmaf(q, t, 2.147474527359009f);
    q = fmaf(q, t, -1.6377531290054321f);
    q = fmaf(q, t, 0.40232160687446594f);
    q = fmaf(q, t, -0.2687568664550781f);
    q = fmaf(q, t, 0.13963006436824799f);
    q = fmaf(q, t, 0.5397006273269653f);
    q = fmaf(q, t, 1.4427292346954346f);
    q = fmaf(q, t, -2.8257482051849365f);   // constant term minus 1: the factor 1/2
  } else {
    q = 0.278960645198822f;
    q = fmaf(q, t, -0.8764582872390747f);
    q = fmaf(q, t, 0.52732914686203f);
    q = fmaf(q, t, 0.44432464241981506f);
    q = fmaf(q, t, 1.451727271080017f);
    q = fmaf(q, t, -2.82594895362854f);     // constant term minus 1: the factor 1/2
  }
  return t * __builtin_amdgcn_exp2f(fmaf(zz, -0.72134752044448170f, q));
}
// fit degree for an activation storage type
template <typename Ta>
constexpr int gelu_deg() {
  return sizeof(Ta) == 2 ? 5 : 9;
}
template <int DEG>
SR_DEV float norm_cdf(float z, float zz) {
  const float h = half_erfc_of<DEG>(z, zz);
  return z >= 0.f ? 1.0f - h : h;
}
template <int DEG>
SR_DEV float gelu_f(float z) {
  return z * norm_cdf<DEG>(z, z * z);
}
template <int DEG>
SR_DEV float gelu_grad_f(float z) {
  const float zz = z * z;
  // phi(z) = 2^(-z^2 log2(e)/2 - log2(sqrt(2 pi)))
  return norm_cdf<DEG>(z, zz) + z * __builtin_amdgcn_exp2f(fmaf(zz, -0.72134752044448170f, -1.3257480647361593f));
}

template <int EPI, typename T, typename Ta>
SR_DEV void epilogue(const EpiArgs& e, int m, int n, float v) {
  const size_t o = (size_t)m * e.ldo + n;
  if constexpr (EPI == EPI_BIAS_ACT) {
    ((Ta*)e.out_act)[o] = from_f32<Ta>(v + to_f32<T>(((const T*)e.bias)[n]));
  } else if constexpr (EPI == EPI_RESID) {
    float t = v + to_f32<T>(((const T*)e.bias)[n]);
    if (e.gate) {
      ((Ta*)e.a_save)[o] = from_f32<Ta>(t);
      t *= e.gate[(size_t)(m / e.S) * e.gate_stride + n];
    }
    const float r = e.resid[o] + t;
    if (e.out_f32) e.out_f32[o] = r;
    if (e.out_st) ((T*)e.out_st)[o] = from_f32<T>(r);
    if (e.sc_x) {
      const int b = m / e.S, s = m - b * e.S;
      const int i = e.sc_idx[(e.sc_shared ? 0 : b) * e.S + s];
      T* xp = (T*)e.sc_x + ((size_t)b * e.sc_L + i) * e.ldo + n;
      const float x0 = to_f32<T>(*xp);
      *xp = from_f32<T>(__fadd_rn(x0, __fsub_rn(to_f32<T>(from_f32<T>(r)), x0)));
    }
  } else if constexpr (EPI == EPI_GELU) {
    const Ta z = from_f32<Ta>(v + to_f32<T>(((const T*)e.bias)[n]));
    ((Ta*)e.out_act)[o] = z;
    ((Ta*)e.out_act2)[o] = from_f32<Ta>(gelu_f<gelu_deg<Ta>()>(to_f32<Ta>(z)));   // of the stored z (recomputed bit for bit)
  } else if constexpr (EPI == EPI_DGELU) {
    const float z = to_f32<Ta>(((const Ta*)e.z_in)[o]);
    ((Ta*)e.out_act)[o] = from_f32<Ta>(v * gelu_grad_f<gelu_deg<Ta>()>(z));
  } else if constexpr (EPI == EPI_ACT) {
    ((Ta*)e.out_act)[o] = from_f32<Ta>(v);
  } else if constexpr (EPI == EPI_F32) {
    e.out_f32[o] = v;
  } else if constexpr (EPI == EPI_F32_ACC) {
    e.out_f32[o] += v;
  }
}

}  // namespace sr
