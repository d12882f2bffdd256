// GEMMs of the fp32 storage mode on the fp32 matrix instruction v_mfma_f32_32x32x2_f32 (fp32
// products, fp32 accumulation; 64 cycles each, 157 TFLOP/s on the chip).
//
//   C[m, n] = sum_k A(m, k) * B(n, k), operand layouts and epilogues as in gemm.hip.
//
// The k order inside a product is free as long as A and B agree: MFMA step (j, t) of a chunk of
// eight k takes k = 8 j + t (lanes 0..31) and 8 j + 4 + t (lanes 32..63), so that a k-major operand
// comes as one 16-byte read per lane and four steps.
//
// gemm_f32_tile: 128 x 128 or 64 x 64 outputs per workgroup (four waves in 2 x 2), operand tiles of
// 32 k staged in LDS (the next tile waits in registers).  Bound by the matrix rate.
// gemm_f32_split: 32 x 32 outputs per workgroup of eight waves, each of which sums the chunks of 16 k
// c = wave, wave + 8, ... straight from global memory; the eight partial tiles are added through LDS
// in wave order.  For outputs with too few 64 x 64 tiles to occupy the chip (small token counts,
// weight gradients of small models): bound by the latency of its loads and by the k loop, which the
// eight waves shorten eightfold.
// Against one workgroup per 64 x 64 tile of scalar FMAs with the whole k loop in series: M = 2026,
// D = 256, F = 1024: weight gradients 414 -> 16 us each, the forward and dX products 50 - 170 -> 14 - 25;
// M = 32, D = 128, F = 512: 10 - 62 -> 3.5 - 5.8 us.  The relative error against fp64 fell a little
// (1.1e-6 -> 9.2e-7 on the block's outputs), the split sums being shorter.
#include "common.h"
#include "epilogue.h"
#include "sr_internal.h"

namespace sr {

namespace {

SR_DEV f32x16 mfma32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

SR_DEV f32x4 buf_load4f(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(f32x4, buf_load16(r, off));
}
SR_DEV float buf_load1f(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// row of score-layout register r (lane half h) inside a 32 x 32 result
SR_DEV int crow(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

template <int EPI>
SR_DEV void finish(const EpiArgs& ep, int m, int n, float v) {
  if constexpr (EPI == EPI_DW) ep.out_f32[(size_t)m * ep.ldo + n] = v;
  else epilogue<EPI, float, float>(ep, m, n, v);
}

constexpr int FK = 32;   // k extent of an LDS tile

// Operand tile of R rows x FK k in LDS: k-major rows of FK + 4 floats (16-byte fragment reads of 16
// consecutive rows cover the 64 banks once), or k-rows of R + 8 floats (the two halves of a wave, four
// k-rows apart, read different banks).
template <int R, bool KM>
struct OpTile {
  static constexpr int LD = KM ? FK + 4 : R + 8;
  static constexpr int SIZE = KM ? R * LD : FK * LD;
  static constexpr int PER = R * FK / 4 / 256;   // 16-byte loads per thread
  f32x4 reg[PER];
  SR_DEV void load(__amdgpu_buffer_rsrc_t rs, int r0, int k0, int ld) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + 256 * i;
      const uint32_t off = KM ? (uint32_t)(r0 + c / (FK / 4)) * ld + k0 + c % (FK / 4) * 4
                              : (uint32_t)(k0 + c / (R / 4)) * ld + r0 + c % (R / 4) * 4;
      reg[i] = buf_load4f(rs, off * 4u);
    }
  }
  SR_DEV void store(float* t) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + 256 * i;
      float* p = KM ? t + c / (FK / 4) * LD + c % (FK / 4) * 4 : t + c / (R / 4) * LD + c % (R / 4) * 4;
      *reinterpret_cast<f32x4*>(p) = reg[i];
    }
  }
  // the four k of steps (j, 0..3) for row `row`
  static SR_DEV f32x4 frag(const float* t, int row, int j, int h) {
    if constexpr (KM) {
      return *reinterpret_cast<const f32x4*>(t + row * LD + 8 * j + 4 * h);
    } else {
      f32x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = t[(8 * j + 4 * h + q) * LD + row];
      return v;
    }
  }
};

}  // namespace

template <int BM, bool AK, bool BK, int EPI>
__global__ __launch_bounds__(256, 2) void gemm_f32_tile_kernel(const float* __restrict__ A, const float* __restrict__ Bm,
                                                               int M, int N, int Kd, int lda, int ldb, uint32_t a_bytes,
                                                               uint32_t b_bytes, EpiArgs ep) {
  constexpr int BN = BM, MI = BM / 64;
  using TA = OpTile<BM, AK>;
  using TB = OpTile<BN, BK>;
  __shared__ __attribute__((aligned(16))) float as[TA::SIZE];
  __shared__ __attribute__((aligned(16))) float bs[TB::SIZE];
  const int lane = threadIdx.x & 63, wid = wave_index(), l32 = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int wm = (wid >> 1) * (BM / 2), wn = (wid & 1) * (BN / 2);
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, a_bytes), rb = make_rsrc(Bm, b_bytes);
  f32x16 acc[MI][MI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const bool do_db = EPI == EPI_DW && ep.db_out != nullptr && blockIdx.x == 0 && threadIdx.x < BM;
  float db = 0.f;
  TA ta;
  TB tb;
  ta.load(ra, m0, 0, lda);
  tb.load(rb, n0, 0, ldb);
  for (int k0 = 0; k0 < Kd; k0 += FK) {
    ta.store(as);
    tb.store(bs);
    __syncthreads();
    if (k0 + FK < Kd) {
      ta.load(ra, m0, k0 + FK, lda);
      tb.load(rb, n0, k0 + FK, ldb);
    }
    if constexpr (EPI == EPI_DW) {   // bias gradient: row sums of A (m-major here)
      if (do_db)
        for (int k = 0; k < FK; ++k) db += as[k * TA::LD + threadIdx.x];
    }
#pragma unroll
    for (int j = 0; j < FK / 8; ++j) {
      f32x4 fa[MI], fb[MI];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        fa[i] = TA::frag(as, wm + 32 * i + l32, j, h);
        fb[i] = TB::frag(bs, wn + 32 * i + l32, j, h);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int jj = 0; jj < MI; ++jj) acc[i][jj] = mfma32(fa[i][t], fb[jj][t], acc[i][jj]);
    }
    __syncthreads();
  }
  if constexpr (EPI == EPI_DW)
    if (do_db && m0 + (int)threadIdx.x < M) ep.db_out[m0 + threadIdx.x] = db;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int jj = 0; jj < MI; ++jj)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm + 32 * i + crow(r, h), n = n0 + wn + 32 * jj + l32;
        if (m < M && n < N) finish<EPI>(ep, m, n, acc[i][jj][r]);
      }
}

constexpr int kSplitWaves = 8;

template <bool AK, bool BK, int EPI>
__global__ __launch_bounds__(64 * kSplitWaves, 2) void gemm_f32_split_kernel(const float* __restrict__ A,
                                                                             const float* __restrict__ Bm, int M, int N,
                                                                             int Kd, int lda, int ldb, uint32_t a_bytes,
                                                                             uint32_t b_bytes, EpiArgs ep) {
  __shared__ float red[kSplitWaves][32][33];
  __shared__ float dbr[kSplitWaves][32];
  const int lane = threadIdx.x & 63, wid = wave_index(), l32 = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, a_bytes), rb = make_rsrc(Bm, b_bytes);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float db = 0.f;
  // the lane's eight k of chunk k0 .. k0 + 15 (steps (0, 0..3), (1, 0..3)); an m-major row past K lies
  // past the operand and reads zero
  auto load = [&](__amdgpu_buffer_rsrc_t rs, auto km, int r, int ld, int k0, float (&v)[8]) {
    if constexpr (decltype(km)::value) {
      const uint32_t o = ((uint32_t)r * ld + k0 + 4 * h) * 4u;
      const f32x4 x = buf_load4f(rs, o), y = buf_load4f(rs, o + 32u);
#pragma unroll
      for (int t = 0; t < 4; ++t) { v[t] = x[t]; v[4 + t] = y[t]; }
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t)
        v[t] = buf_load1f(rs, ((uint32_t)(k0 + (t >> 2) * 8 + 4 * h + (t & 3)) * ld + r) * 4u);
    }
  };
  constexpr int STEP = 16 * kSplitWaves;
  const int chunks = (Kd + 15) / 16;
  const int mine = chunks > wid ? (chunks - wid + kSplitWaves - 1) / kSplitWaves : 0;
  float a[2][8], b[2][8];
  if (mine > 0) {
    load(ra, IC<AK>{}, m0 + l32, lda, wid * 16, a[0]);
    load(rb, IC<BK>{}, n0 + l32, ldb, wid * 16, b[0]);
  }
  auto step = [&](int c, auto cur) {   // loads chunk c + 1 while chunk c is multiplied
    constexpr int P = decltype(cur)::value;
    if (c + 1 < mine) {
      load(ra, IC<AK>{}, m0 + l32, lda, wid * 16 + (c + 1) * STEP, a[1 - P]);
      load(rb, IC<BK>{}, n0 + l32, ldb, wid * 16 + (c + 1) * STEP, b[1 - P]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      acc = mfma32(a[P][t], b[P][t], acc);
      if constexpr (EPI == EPI_DW) db += a[P][t];
    }
  };
  for (int c = 0; c < mine; c += 2) {
    step(c, IC<0>{});
    if (c + 1 < mine) step(c + 1, IC<1>{});
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wid][crow(r, h)][l32] = acc[r];
  if constexpr (EPI == EPI_DW) {
    db += __shfl_xor(db, 32, 64);
    if (h == 0) dbr[wid][l32] = db;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 1024 / (64 * kSplitWaves); ++q) {
    const int e = threadIdx.x + 64 * kSplitWaves * q, row = e >> 5, col = e & 31;
    float v = red[0][row][col];
#pragma unroll
    for (int w = 1; w < kSplitWaves; ++w) v += red[w][row][col];
    if (m0 + row < M && n0 + col < N) finish<EPI>(ep, m0 + row, n0 + col, v);
  }
  if constexpr (EPI == EPI_DW) {
    if (ep.db_out && blockIdx.x == 0 && threadIdx.x < 32 && m0 + (int)threadIdx.x < M) {
      float v = dbr[0][threadIdx.x];
#pragma unroll
      for (int w = 1; w < kSplitWaves; ++w) v += dbr[w][threadIdx.x];
      ep.db_out[m0 + threadIdx.x] = v;
    }
  }
}

// 128 x 128 tiles once they fill the chip twice, 64 x 64 while they fill it once; fewer outputs take
// the 32 x 32 tiles whose eight waves share the k loop.
template <bool AK, bool BK, int EPI>
static hipError_t run_f32(const GemmDesc& g, const EpiArgs& ep, hipStream_t st) {
  auto tiles = [&](int b) { return (long)((g.M + b - 1) / b) * ((g.N + b - 1) / b); };
  auto grid = [&](int b) { return dim3((unsigned)((g.N + b - 1) / b), (unsigned)((g.M + b - 1) / b)); };
#define SR_F32_ARGS                                                                                              \
  st, (const float*)g.A, (const float*)g.B, g.M, g.N, g.K, (int)g.lda, (int)g.ldb, (uint32_t)g.a_bytes,          \
      (uint32_t)g.b_bytes, ep
  if (tiles(128) >= 512) SR_LAUNCH((gemm_f32_tile_kernel<128, AK, BK, EPI>), grid(128), dim3(256), 0, SR_F32_ARGS);
  else if (tiles(64) >= 256) SR_LAUNCH((gemm_f32_tile_kernel<64, AK, BK, EPI>), grid(64), dim3(256), 0, SR_F32_ARGS);
  else SR_LAUNCH((gemm_f32_split_kernel<AK, BK, EPI>), grid(32), dim3(64 * kSplitWaves), 0, SR_F32_ARGS);
#undef SR_F32_ARGS
  return hipGetLastError();
}

// The block's products: forward (both operands k-major), dX (weight n-major) and dW (both token-major)
// on widths that are multiples of 64, which is every product of the fp32 mode: those of the adaLN and FiLM
// conditioning, over a handful of samples, are in gemv.hip.
bool gemm_f32_takes(const GemmDesc& g, int epi) {
  if (g.dtype != kF32 || g.N % 64) return false;
  switch (epi) {
    case EPI_BIAS_ACT: case EPI_RESID: case EPI_GELU: return g.a_kmajor && g.b_kmajor && g.K % 64 == 0;
    case EPI_DGELU: case EPI_ACT: case EPI_F32: case EPI_F32_ACC: return g.a_kmajor && !g.b_kmajor && g.K % 64 == 0;
    case EPI_DW: return !g.a_kmajor && !g.b_kmajor && g.M % 64 == 0;
    default: return false;
  }
}

hipError_t launch_gemm_f32(const GemmDesc& g, int epi, const EpiArgs& ep, hipStream_t st) {
  switch (epi) {
    case EPI_BIAS_ACT: return run_f32<true, true, EPI_BIAS_ACT>(g, ep, st);
    case EPI_RESID: return run_f32<true, true, EPI_RESID>(g, ep, st);
    case EPI_GELU: return run_f32<true, true, EPI_GELU>(g, ep, st);
    case EPI_DGELU: return run_f32<true, false, EPI_DGELU>(g, ep, st);
    case EPI_ACT: return run_f32<true, false, EPI_ACT>(g, ep, st);
    case EPI_F32: return run_f32<true, false, EPI_F32>(g, ep, st);
    case EPI_F32_ACC: return run_f32<true, false, EPI_F32_ACC>(g, ep, st);
    case EPI_DW: return run_f32<false, false, EPI_DW>(g, ep, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace sr
