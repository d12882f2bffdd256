// Attention of the fp32 storage mode on v_mfma_f32_32x32x2_f32, fp32 throughout: forward, dK/dV and
// dQ at head dims 32, 64 and 128, on separate query and key/value buffers (self-attention passes the
// one token-major qkv buffer twice).  Formulas and layouts as in attention.hip.
//
// A workgroup of kW waves, four or eight, owns 32 rows of the resident dimension; its waves take the
// 32-row units of the streamed one in turn (unit u belongs to wave u mod kW) and their results are merged
// through LDS in wave order at the end, so a few hundred tokens already give every SIMD a wave, and results do not
// depend on scheduling.  A unit has HD MFMAs of 64 cycles per product pair (forward: 4096 cycles at
// head dim 64) for HD / 8 16-byte row loads and HD / 2 4-byte column loads per lane, so the operands
// come straight from global memory (each element once per workgroup, from L2) without LDS.
// Score register r of a lane (l32, h) holds the row srow(r) of the streamed unit and the resident row
// l32, which is the B operand layout of the next product: P and dS never leave their registers.
// Bound by the matrix rate (157 TFLOP/s) and, with one or two waves per SIMD, by the latency of the
// operand loads.  2 x 1013 tokens, four heads of 64: forward 847 -> 33, dK/dV 1626 -> 61, dQ 1240 -> 43
// us against one thread per row; 32 tokens, four heads of 32: 22 -> 4.4, 17 -> 8.0, 15 -> 4.7 us.
#include "common.h"
#include "sr_internal.h"

namespace sr {

namespace {

// workgroups per CU: two waves per SIMD, one at head dim 128 (its registers)
constexpr int f32_occ(int hd, int kw) { return kw == 8 || hd == 128 ? 1 : 2; }

SR_DEV f32x16 mfma32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
SR_DEV int srow(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }
SR_DEV void zero16(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
}

// One head of a row-major tensor: rows [0, n) of a sample, row stride ld (floats).  Rows at or past n
// read as zero, so neighbouring samples never enter a product.
struct Head {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t base, ld;
  int n;
};
SR_DEV Head head_of(const float* p, uint32_t elems, size_t first, int ld, int n) {
  return {make_rsrc(p, elems * 4u), (uint32_t)(first * 4), (uint32_t)ld, n};
}
// columns c .. c + 3 of a row
SR_DEV f32x4 row4(const Head& t, int row, int c) {
  const uint32_t off = row < t.n ? t.base + ((uint32_t)row * t.ld + (uint32_t)c) * 4u : 0x80000000u;
  return __builtin_bit_cast(f32x4, buf_load16(t.rs, off));
}
SR_DEV float elem(const Head& t, int row, int c) {
  const uint32_t off = row < t.n ? t.base + ((uint32_t)row * t.ld + (uint32_t)c) * 4u : 0x80000000u;
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(t.rs, off, 0, 0));
}

// Row fragment of rows r0 .. r0 + 31: element 4 j + t of lane (l32, h) is column 8 j + 4 h + t, the k
// order of every row-by-row product here.
template <int HD>
SR_DEV void rows32(const Head& t, int r0, int l32, int h, f32x4 (&f)[HD / 8]) {
#pragma unroll
  for (int j = 0; j < HD / 8; ++j) f[j] = row4(t, r0 + l32, 8 * j + 4 * h);
}
// acc[x][y] += sum_c a[x][c] b[y][c] (x: the unit's rows, y: the resident rows)
template <int HD>
SR_DEV void dot32(const f32x4 (&a)[HD / 8], const f32x4 (&b)[HD / 8], f32x16& acc) {
#pragma unroll
  for (int j = 0; j < HD / 8; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = mfma32(a[j][t], b[j][t], acc);
}
// acc[c][y] += sum over the unit's rows x of t[x][c] p[x][y], p in score layout
template <int HD>
SR_DEV void accumulate(const Head& t, int r0, int l32, int h, const float (&p)[16], f32x16 (&acc)[HD / 32]) {
#pragma unroll
  for (int db = 0; db < HD / 32; ++db) {
    float a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = elem(t, r0 + srow(r, h), 32 * db + l32);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db] = mfma32(a[r], p[r], acc[db]);
  }
}

// A wave's transposed result (acc[db][r] = X[column 32 db + srow(r)][row l32]) into its LDS plane.
template <int HD>
constexpr int plane_ld() { return HD + 4; }
template <int HD>
SR_DEV void to_plane(float* pl, const f32x16 (&acc)[HD / 32], int l32, int h) {
#pragma unroll
  for (int db = 0; db < HD / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 v = {acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]};
      *reinterpret_cast<f32x4*>(pl + l32 * plane_ld<HD>() + 32 * db + 8 * g + 4 * h) = v;
    }
}
// The waves' planes added in wave order, scaled, to rows r0 .. of dst.
template <int HD, int kW>
SR_DEV void merge(const float* planes, float* dst, size_t ld, int r0, int n, float scale) {
  for (int c = threadIdx.x; c < 32 * HD / 4; c += 64 * kW) {
    const int row = c / (HD / 4), col = c % (HD / 4) * 4;
    f32x4 v = *reinterpret_cast<const f32x4*>(planes + row * plane_ld<HD>() + col);
#pragma unroll
    for (int w = 1; w < kW; ++w)
      v += *reinterpret_cast<const f32x4*>(planes + (w * 32 + row) * plane_ld<HD>() + col);
    if (r0 + row < n) *reinterpret_cast<f32x4*>(dst + (size_t)(r0 + row) * ld + col) = v * scale;
  }
}

}  // namespace

// q: Sq rows (stride ldq), kv: Skv rows (stride ldkv, values D columns on), *_elems: elements
// addressable from each pointer.
template <int HD, int kW>
__global__ __launch_bounds__(64 * kW, f32_occ(HD, kW)) void attn_fwd_f32(const float* __restrict__ q, int ldq, uint32_t q_elems,
                                                       const float* __restrict__ kv, int ldkv, uint32_t kv_elems,
                                                       float* __restrict__ O, float* __restrict__ lse, int Sq, int Skv,
                                                       int H, int D, float sl2) {
  __shared__ __attribute__((aligned(16))) float planes[kW * 32 * plane_ld<HD>()];
  __shared__ float ms[kW][32], ls[kW][32];
  const int lane = threadIdx.x & 63, wid = wave_index(), l32 = lane & 31, h = lane >> 5;
  const int b = blockIdx.z, hh = blockIdx.y, q0 = blockIdx.x * 32;
  const Head hq = head_of(q, q_elems, (size_t)b * Sq * ldq + hh * HD, ldq, Sq);
  const Head hk = head_of(kv, kv_elems, (size_t)b * Skv * ldkv + hh * HD, ldkv, Skv);
  const Head hv = head_of(kv, kv_elems, (size_t)b * Skv * ldkv + D + hh * HD, ldkv, Skv);
  f32x4 qf[HD / 8];
  rows32<HD>(hq, q0, l32, h, qf);
  f32x16 o[HD / 32];
#pragma unroll
  for (int db = 0; db < HD / 32; ++db) zero16(o[db]);
  float m = -INFINITY, l = 0.f;
  for (int k0 = wid * 32; k0 < Skv; k0 += 32 * kW) {
    f32x4 kf[HD / 8];
    rows32<HD>(hk, k0, l32, h, kf);
    f32x16 s;
    zero16(s);
    dot32<HD>(kf, qf, s);   // S^T: key srow(r), query l32
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = k0 + srow(r, h) < Skv ? s[r] * sl2 : -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    const float mn = fmaxf(m, half_pair_max(mx));
    const float alpha = exp2f(m - mn);
    float p[16];
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = exp2f(s[r] - mn);
      l += p[r];
    }
#pragma unroll
    for (int db = 0; db < HD / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    m = mn;
    accumulate<HD>(hv, k0, l32, h, p, o);
  }
  l = half_pair_sum(l);
  if (h == 0) { ms[wid][l32] = m; ls[wid][l32] = l; }
  __syncthreads();
  // common reference max of the row; a wave without keys has m = -inf and weight 0
  float mx = ms[0][l32], tot = 0.f;
#pragma unroll
  for (int w = 1; w < kW; ++w) mx = fmaxf(mx, ms[w][l32]);
#pragma unroll
  for (int w = 0; w < kW; ++w) tot += ls[w][l32] * exp2f(ms[w][l32] - mx);
  const float f = exp2f(m - mx) / tot;
#pragma unroll
  for (int db = 0; db < HD / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] *= f;
  to_plane<HD>(planes + wid * 32 * plane_ld<HD>(), o, l32, h);
  if (wid == 0 && h == 0 && q0 + l32 < Sq) lse[((size_t)b * H + hh) * Sq + q0 + l32] = mx + log2f(tot);
  __syncthreads();
  merge<HD, kW>(planes, O + (size_t)b * Sq * D + hh * HD, D, q0, Sq, 1.0f);
}

// dK to dk_out (row stride ldo), dV D columns after it.
template <int HD, int kW>
__global__ __launch_bounds__(64 * kW, f32_occ(HD, kW)) void attn_dkv_f32(const float* __restrict__ q, int ldq, uint32_t q_elems,
                                                       const float* __restrict__ kv, int ldkv, uint32_t kv_elems,
                                                       const float* __restrict__ dO, const float* __restrict__ lse,
                                                       const float* __restrict__ delta, float* __restrict__ dk_out,
                                                       int ldo, int Sq, int Skv, int H, int D, float sl2, float scale) {
  __shared__ __attribute__((aligned(16))) float planes[kW * 32 * plane_ld<HD>()];
  const int lane = threadIdx.x & 63, wid = wave_index(), l32 = lane & 31, h = lane >> 5;
  const int b = blockIdx.z, hh = blockIdx.y, k0 = blockIdx.x * 32;
  const Head hq = head_of(q, q_elems, (size_t)b * Sq * ldq + hh * HD, ldq, Sq);
  const Head hk = head_of(kv, kv_elems, (size_t)b * Skv * ldkv + hh * HD, ldkv, Skv);
  const Head hv = head_of(kv, kv_elems, (size_t)b * Skv * ldkv + D + hh * HD, ldkv, Skv);
  const Head hd = head_of(dO, (uint32_t)((size_t)gridDim.z * Sq * D), (size_t)b * Sq * D + hh * HD, D, Sq);
  const float* lp = lse + ((size_t)b * H + hh) * Sq;
  const float* dp = delta + ((size_t)b * H + hh) * Sq;
  f32x4 kf[HD / 8], vf[HD / 8];
  rows32<HD>(hk, k0, l32, h, kf);
  rows32<HD>(hv, k0, l32, h, vf);
  f32x16 dk[HD / 32], dv[HD / 32];
#pragma unroll
  for (int db = 0; db < HD / 32; ++db) { zero16(dk[db]); zero16(dv[db]); }
  for (int q0 = wid * 32; q0 < Sq; q0 += 32 * kW) {
    f32x16 s, t;
    zero16(s);
    zero16(t);
    {
      f32x4 f[HD / 8];
      rows32<HD>(hq, q0, l32, h, f);
      dot32<HD>(f, kf, s);   // S: query srow(r), key l32
    }
    {
      f32x4 f[HD / 8];
      rows32<HD>(hd, q0, l32, h, f);
      dot32<HD>(f, vf, t);   // dP
    }
    float p[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = q0 + srow(r, h);
      const bool ok = i < Sq;
      const float lq = ok ? lp[i] : 0.f, dq = ok ? dp[i] : 0.f;
      p[r] = ok ? exp2f(s[r] * sl2 - lq) : 0.f;
      ds[r] = ok ? p[r] * (t[r] - dq) : 0.f;
    }
    accumulate<HD>(hd, q0, l32, h, p, dv);
    accumulate<HD>(hq, q0, l32, h, ds, dk);
  }
  float* out = dk_out + (size_t)b * Skv * ldo + hh * HD;
  to_plane<HD>(planes + wid * 32 * plane_ld<HD>(), dk, l32, h);
  __syncthreads();
  merge<HD, kW>(planes, out, ldo, k0, Skv, scale);
  __syncthreads();
  to_plane<HD>(planes + wid * 32 * plane_ld<HD>(), dv, l32, h);
  __syncthreads();
  merge<HD, kW>(planes, out + D, ldo, k0, Skv, 1.0f);
}

template <int HD, int kW>
__global__ __launch_bounds__(64 * kW, f32_occ(HD, kW)) void attn_dq_f32(const float* __restrict__ q, int ldq, uint32_t q_elems,
                                                      const float* __restrict__ kv, int ldkv, uint32_t kv_elems,
                                                      const float* __restrict__ dO, const float* __restrict__ lse,
                                                      const float* __restrict__ delta, float* __restrict__ dq_out,
                                                      int ldo, int Sq, int Skv, int H, int D, float sl2, float scale) {
  __shared__ __attribute__((aligned(16))) float planes[kW * 32 * plane_ld<HD>()];
  const int lane = threadIdx.x & 63, wid = wave_index(), l32 = lane & 31, h = lane >> 5;
  const int b = blockIdx.z, hh = blockIdx.y, q0 = blockIdx.x * 32;
  const Head hq = head_of(q, q_elems, (size_t)b * Sq * ldq + hh * HD, ldq, Sq);
  const Head hk = head_of(kv, kv_elems, (size_t)b * Skv * ldkv + hh * HD, ldkv, Skv);
  const Head hv = head_of(kv, kv_elems, (size_t)b * Skv * ldkv + D + hh * HD, ldkv, Skv);
  const Head hd = head_of(dO, (uint32_t)((size_t)gridDim.z * Sq * D), (size_t)b * Sq * D + hh * HD, D, Sq);
  f32x4 qf[HD / 8], df[HD / 8];
  rows32<HD>(hq, q0, l32, h, qf);
  rows32<HD>(hd, q0, l32, h, df);
  const bool mine = q0 + l32 < Sq;
  const size_t st = ((size_t)b * H + hh) * Sq + q0 + l32;
  const float lq = mine ? lse[st] : 0.f, dq_ = mine ? delta[st] : 0.f;
  f32x16 dq[HD / 32];
#pragma unroll
  for (int db = 0; db < HD / 32; ++db) zero16(dq[db]);
  for (int k0 = wid * 32; k0 < Skv; k0 += 32 * kW) {
    f32x16 s, t;
    zero16(s);
    zero16(t);
    {
      f32x4 f[HD / 8];
      rows32<HD>(hk, k0, l32, h, f);
      dot32<HD>(f, qf, s);   // S^T: key srow(r), query l32
    }
    {
      f32x4 f[HD / 8];
      rows32<HD>(hv, k0, l32, h, f);
      dot32<HD>(f, df, t);   // dP^T
    }
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      ds[r] = k0 + srow(r, h) < Skv ? exp2f(s[r] * sl2 - lq) * (t[r] - dq_) : 0.f;
    accumulate<HD>(hk, k0, l32, h, ds, dq);
  }
  to_plane<HD>(planes + wid * 32 * plane_ld<HD>(), dq, l32, h);
  __syncthreads();
  merge<HD, kW>(planes, dq_out + (size_t)b * Sq * ldo + hh * HD, ldo, q0, Sq, scale);
}

// ------------------------------------------------------------------------------ launchers

// Eight waves where four would leave the SIMDs one wave each (a round of workgroups at most, which then
// have no second one beside them) and every wave still has a unit: one wave's operand loads fly under the
// other's MFMAs.  2 x 1013 tokens, four heads of 64, 256 workgroups: forward 33.5 -> 29.5, dK/dV 64 ->
// 58, dQ 44 -> 39 us.
static bool eight_waves(int rows, int streamed, int H, int B) {
  return (long)((rows + 31) / 32) * H * B <= 256 && streamed > 32 * 7;
}

#define SR_F32_HD(KERNEL, ROWS, STREAMED, ...)                                                              \
  do {                                                                                                      \
    const dim3 g_((unsigned)(((ROWS) + 31) / 32), H, B);                                                    \
    const bool w8_ = eight_waves(ROWS, STREAMED, H, B);                                                     \
    if (hd == 32 && w8_) SR_LAUNCH((KERNEL<32, 8>), g_, dim3(512), 0, st, __VA_ARGS__);                     \
    else if (hd == 32) SR_LAUNCH((KERNEL<32, 4>), g_, dim3(256), 0, st, __VA_ARGS__);                       \
    else if (hd == 64 && w8_) SR_LAUNCH((KERNEL<64, 8>), g_, dim3(512), 0, st, __VA_ARGS__);                \
    else if (hd == 64) SR_LAUNCH((KERNEL<64, 4>), g_, dim3(256), 0, st, __VA_ARGS__);                       \
    else SR_LAUNCH((KERNEL<128, 4>), g_, dim3(256), 0, st, __VA_ARGS__);                                    \
    const hipError_t e_ = hipGetLastError();                                                                \
    if (e_ != hipSuccess) return e_;                                                                        \
  } while (0)

hipError_t launch_attn_fwd_f32(const float* q, int ldq, uint32_t q_elems, const float* kv, int ldkv, uint32_t kv_elems,
                               float* O, float* lse, int B, int Sq, int Skv, int H, int D, hipStream_t st) {
  const int hd = D / H;
  SR_F32_HD(attn_fwd_f32, Sq, Skv, q, ldq, q_elems, kv, ldkv, kv_elems, O, lse, Sq, Skv, H, D,
            1.4426950408889634f / sqrtf((float)hd));
  return hipSuccess;
}

hipError_t launch_attn_bwd_f32(const float* q, int ldq, uint32_t q_elems, const float* kv, int ldkv, uint32_t kv_elems,
                               const float* dO, const float* lse, const float* delta, float* dq, int ld_dq, float* dk,
                               int ld_dk, int B, int Sq, int Skv, int H, int D, hipStream_t st) {
  const int hd = D / H;
  const float scale = 1.0f / sqrtf((float)hd), sl2 = 1.4426950408889634f * scale;
  SR_F32_HD(attn_dkv_f32, Skv, Sq, q, ldq, q_elems, kv, ldkv, kv_elems, dO, lse, delta, dk, ld_dk,
            Sq, Skv, H, D, sl2, scale);
  SR_F32_HD(attn_dq_f32, Sq, Skv, q, ldq, q_elems, kv, ldkv, kv_elems, dO, lse, delta, dq, ld_dq,
            Sq, Skv, H, D, sl2, scale);
  return hipSuccess;
}

}  // namespace sr
