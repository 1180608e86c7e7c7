// EM and MVDR kernels for large arrays, 9 <= D <= 32 channels (e.g. multi-array set-ups with 24
// microphones).  Same algorithm, same fp64 arithmetic and the same pass / factor structure as the D <= 8
// kernels (arXiv 2212.05271, Section 2.2 and 2.3); what changes is the mapping:
// D is a run-time value and the contractions run on the fp64 matrix cores (gss_large_impl.h).
#include "gss_large_impl.h"

#define GSS_DECL_K(KK)                                                                                           \
  int gss_em_large_k##KK(gss_ctx* ctx, const gss_yview& Y, const uint8_t* activity, const int32_t* T_len, int S, int F, \
                         int Tmax, int D, int iters, int weight_mode, float* gamma, hipStream_t st);
GSS_DECL_K(1) GSS_DECL_K(2) GSS_DECL_K(3) GSS_DECL_K(4) GSS_DECL_K(5) GSS_DECL_K(6) GSS_DECL_K(7) GSS_DECL_K(8)
#undef GSS_DECL_K

int gss_em_large(gss_ctx* ctx, const gss_yview& Y, const uint8_t* activity, const int32_t* T_len, int S, int F, int Tmax,
                 int D, int K, int iters, int weight_mode, float* gamma, hipStream_t st) {
  switch (K) {
#define GSS_CASE_K(KK) \
  case KK: return gss_em_large_k##KK(ctx, Y, activity, T_len, S, F, Tmax, D, iters, weight_mode, gamma, st);
    GSS_CASE_K(1) GSS_CASE_K(2) GSS_CASE_K(3) GSS_CASE_K(4) GSS_CASE_K(5) GSS_CASE_K(6) GSS_CASE_K(7) GSS_CASE_K(8)
#undef GSS_CASE_K
    default: return GSS_EUNSUPPORTED;
  }
}

int gss_mvdr_large(gss_ctx* ctx, const gss_yview& Y, const float* gamma, const int32_t* T_len, int S, int F, int Tmax,
                   int D, int K, const int32_t* target, int32_t* ref, int ref_per_f, float* X, hipStream_t st) {
  float2* Xc = (float2*)X;
  // (19 and 20 channels: the last block in full; 4 x 4 x 4 products for it took 0.98 to 1.02 times as long)
  const int rest = D > 16 && D <= 24 && large_rest(D, K) == 2 ? 0 : large_rest(D, K);
  auto blocks = [&](auto NB) {
    constexpr int nb = decltype(NB)::value;
    if constexpr (nb != 3)
      if (rest == 2) return run_mvdr_large<nb, 2>(ctx, Y, gamma, T_len, S, F, Tmax, D, K, target, ref, ref_per_f, Xc, st);
    return rest == 1 ? run_mvdr_large<nb, 1>(ctx, Y, gamma, T_len, S, F, Tmax, D, K, target, ref, ref_per_f, Xc, st)
                     : run_mvdr_large<nb, 0>(ctx, Y, gamma, T_len, S, F, Tmax, D, K, target, ref, ref_per_f, Xc, st);
  };
  if (D <= 16) return blocks(std::integral_constant<int, 2>{});
  if (D <= 24) return blocks(std::integral_constant<int, 3>{});
  return blocks(std::integral_constant<int, 4>{});
}
