// The pivot proposer's network on bf16 matrix cores: 28 -> 128 -> 128 -> 128
// -> 10 with ReLU, plus the row's 10 P_D amplitudes (inputs 18..27).
//
// v_mfma_f32_32x32x16_bf16 (wave64): A[i][k] at lane i + 32 (k / 8), element
// k % 8; B[k][j] at lane j + 32 (k / 8), element k % 8; D[i][j] at lane
// j + 32 ((i / 4) % 2), element 4 (i / 8) + i % 4.  Measured on gfx950 it
// gives the bits of v_mfma_f32_16x16x16_bf16 over the same 16 products at
// twice its rate (1374 against 723 TFLOP/s in a register loop), which
// v_mfma_f32_16x16x32_bf16 does not (it sums 32 products before it rounds).
#include "mlp.h"

#include <algorithm>

namespace bbl {
namespace {

constexpr int kIn = kMlpIn, kHid = kMlpHid, kOut = kMlpOut;
constexpr int oW1 = 0, oB1 = oW1 + kHid * kIn, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid,
              oW3 = oB2 + kHid, oB3 = oW3 + kHid * kHid, oW4 = oB3 + kHid,
              oB4 = oW4 + kOut * kHid;
static_assert(oB4 + kOut == kMlpParams, "parameter layout");

typedef uint16_t bf16;
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf2f(bf16 h) { return __uint_as_float((uint32_t)h << 16); }

// two floats rounded to bfloat16 (nearest even; NaN stays NaN)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const v2bf p = __builtin_convertvector((v2f){a, b}, v2bf);
  uint32_t u;
  __builtin_memcpy(&u, &p, 4);
  return u;
}

// ReLU that keeps NaN, so that broken weights reach the output: the IEEE
// maximum, one instruction
__device__ __forceinline__ float relu(float v) {
  float r;
  asm("v_maximum3_f32 %0, %1, 0, 0" : "=v"(r) : "v"(v));
  return r;
}

__device__ __forceinline__ v16f mma(v8bf a, v8bf b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ v16f zero16() {
  return v16f{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}

__device__ __forceinline__ v8bf as_v8bf(uint4 u) {
  v8bf v;
  __builtin_memcpy(&v, &u, 16);
  return v;
}

// eight consecutive floats (4-byte aligned) as eight bfloat16
__device__ __forceinline__ uint4 pack8(const float *__restrict__ p, int count) {
  float f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = 0.f;
  if (count == 8) __builtin_memcpy(f, p, 32);
  else if (count == 4) __builtin_memcpy(f, p, 16);
  return uint4{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]),
               pack_bf16(f[6], f[7])};
}

// The weights as A operands, one 16-byte piece per lane and 32 x 16 tile
// (tile (it, kt) of W2 at w2[(it * 8 + kt) * 64 + lane]), so that a wave reads
// a tile with one conflict-free ds_read_b128.  W4 has 16 of its 32 rows.
struct Frags {
  uint4 w1[8 * 64], w2[32 * 64], w3[32 * 64], w4[8 * 32];
  float b1[kHid], b2[kHid], b3[kHid], b4[16];
};

__device__ __forceinline__ void stage_square(const float *__restrict__ W, uint4 *dst) {
  for (int e = threadIdx.x; e < kHid * 16; e += blockDim.x) {
    const int i = e >> 4, kg = e & 15;
    dst[((i >> 5) * 8 + (kg >> 1)) * 64 + (i & 31) + 32 * (kg & 1)] = pack8(W + i * kHid + kg * 8, 8);
  }
}

__device__ void stage_weights(const float *__restrict__ p, Frags &w) {
  stage_square(p + oW2, w.w2);
  stage_square(p + oW3, w.w3);
  for (int e = threadIdx.x; e < kHid * 4; e += blockDim.x) {
    const int i = e >> 2, kg = e & 3;
    w.w1[((i >> 5) * 2 + (kg >> 1)) * 64 + (i & 31) + 32 * (kg & 1)] =
        pack8(p + oW1 + i * kIn + kg * 8, kg < 3 ? 8 : 4);
  }
  for (int e = threadIdx.x; e < 16 * 16; e += blockDim.x) {
    const int i = e >> 4, kg = e & 15;
    w.w4[(kg >> 1) * 32 + i + 16 * (kg & 1)] =
        pack8(p + oW4 + (i < kOut ? i : 0) * kHid + kg * 8, i < kOut ? 8 : 0);
  }
  for (int i = threadIdx.x; i < kHid; i += blockDim.x) {
    w.b1[i] = p[oB1 + i];
    w.b2[i] = p[oB2 + i];
    w.b3[i] = p[oB3 + i];
  }
  if (threadIdx.x < 16) w.b4[threadIdx.x] = threadIdx.x < kOut ? p[oB4 + threadIdx.x] : 0.f;
}

// Features 8 (2 kt + h) .. + 8 of a row as a B operand piece (features 28..31
// and rows past the end are zero).  Rows are 56 bytes, so the two loads need
// no more than the features' own alignment.
__device__ __forceinline__ v8bf load_x(const bf16 *__restrict__ X, int64_t row, int64_t rows,
                                       int kt, int h) {
  uint2 lo{0u, 0u}, hi{0u, 0u};
  if (row < rows) {
    const bf16 *p = X + row * kIn + 16 * kt + 8 * h;
    __builtin_memcpy(&lo, p, 8);
    if (kt == 0 || h == 0) __builtin_memcpy(&hi, p + 4, 8);
  }
  return as_v8bf(uint4{lo.x, lo.y, hi.x, hi.y});
}

// relu(acc + bias) of 32 features (lane = row) as the B operands of the next
// layer's k tiles 2 it and 2 it + 1.  The lane's 16 values are features
// 8 t + 4 h + 0..3, t = 0..3, of the 32; the operand wants 8 consecutive
// ones, so lanes l and l + 32 trade one pair of registers per k tile.
__device__ __forceinline__ void relu_operands(const v16f &acc, const float *bias, int h,
                                              v8bf &k0, v8bf &k1) {
  uint32_t p[8];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    v4f b;
    __builtin_memcpy(&b, bias + 8 * t + 4 * h, 16);
    p[2 * t] = pack_bf16(relu(acc[4 * t] + b[0]), relu(acc[4 * t + 1] + b[1]));
    p[2 * t + 1] = pack_bf16(relu(acc[4 * t + 2] + b[2]), relu(acc[4 * t + 3] + b[3]));
  }
#pragma unroll
  for (int t = 0; t < 4; t += 2) {
    const auto a = __builtin_amdgcn_permlane32_swap(p[2 * t], p[2 * t + 2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(p[2 * t + 1], p[2 * t + 3], false, false);
    const v8bf v = as_v8bf(uint4{a[0], b[0], a[1], b[1]});
    if (t == 0) k0 = v;
    else k1 = v;
  }
}

// One hidden layer for RT row tiles of 32 rows: KT k tiles in, 8 out.
template <int RT, int KT>
__device__ __forceinline__ void hidden(const uint4 *w, const float *bias, int lane,
                                       const v8bf (&in)[RT][KT], v8bf (&out)[RT][8]) {
  const int h = lane >> 5;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    v16f acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = zero16();
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const v8bf a = as_v8bf(w[(it * KT + kt) * 64 + lane]);
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[r] = mma(a, in[r][kt], acc[r]);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r)
      relu_operands(acc[r], bias + 32 * it, h, out[r][2 * it], out[r][2 * it + 1]);
  }
}

// Inference.  A wave carries RT tiles of 32 rows through all four layers in
// registers: with the weights as the A operand a layer's output has one row
// per lane, which (after a swap between the wave's halves) is the B operand of
// the next layer, so activations never leave the registers and the only
// traffic besides the rows is the weight tiles from LDS, each read once for
// RT tiles.  With one row tile the weight reads alone would take all of the
// LDS bandwidth (1 KB per 32-cycle MFMA on each of four SIMDs); two tiles
// halve them and fill the 256 registers a wave may have at two waves a SIMD.
// MFMA-bound: 5e6 rows are 0.41 TFLOP with padding, 0.30 ms at the rate above;
// the bytes (96 a row) take 0.10 ms.  Measured 0.370 ms (7.14 ms with the
// activations exchanged through LDS after every layer); 33,001 rows 10 us
// (137), 1000 rows 9.6 us (48), where staging the weights is most of it.
template <int RT>
__global__ __launch_bounds__(256, 2) void k_mlp_forward(const float *__restrict__ params,
                                                        const bf16 *__restrict__ X, int64_t rows,
                                                        float *__restrict__ out) {
  __shared__ Frags w;
  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int64_t stride = (int64_t)gridDim.x * 4 * 32 * RT;
  int64_t r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32 * RT;
  v8bf x[RT][2];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) x[r][kt] = load_x(X, r0 + 32 * r + lr, rows, kt, h);
  stage_weights(params, w);
  __syncthreads();
#pragma unroll 1
  for (; r0 < rows; r0 += stride) {
    v8bf u[RT][8], v[RT][8];
    hidden<RT, 2>(w.w1, w.b1, lane, x, u);
    // the next tile's rows and this tile's P_D amplitudes, used at the end
    v8bf xn[RT][2];
    uint2 s0[RT];
    uint32_t s1[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) xn[r][kt] = load_x(X, r0 + stride + 32 * r + lr, rows, kt, h);
      const int64_t row = r0 + 32 * r + lr;
      s0[r] = uint2{0u, 0u};
      s1[r] = 0u;
      if (row < rows) {
        __builtin_memcpy(&s0[r], X + row * kIn + kMlpSkip + 4 * h, 8);
        if (h == 0) __builtin_memcpy(&s1[r], X + row * kIn + kMlpSkip + 8, 4);
      }
    }
    hidden<RT, 8>(w.w2, w.b2, lane, u, v);
    hidden<RT, 8>(w.w3, w.b3, lane, v, u);
    v16f acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = zero16();
#pragma unroll
    for (int kt = 0; kt < 8; ++kt) {
      uint4 f = w.w4[kt * 32 + (lane & 15) + 16 * h];
      if (lr >= 16) f = uint4{0u, 0u, 0u, 0u};
      const v8bf a = as_v8bf(f);
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[r] = mma(a, u[r][kt], acc[r]);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int64_t row = r0 + 32 * r + lr;
      const float *b = w.b4 + 4 * h;
      float o[4];
      o[0] = (acc[r][0] + b[0]) + __uint_as_float(s0[r].x << 16);
      o[1] = (acc[r][1] + b[1]) + __uint_as_float(s0[r].x & 0xFFFF0000u);
      o[2] = (acc[r][2] + b[2]) + __uint_as_float(s0[r].y << 16);
      o[3] = (acc[r][3] + b[3]) + __uint_as_float(s0[r].y & 0xFFFF0000u);
      const float o2[2] = {(acc[r][4] + w.b4[8]) + __uint_as_float(s1[r] << 16),
                           (acc[r][5] + w.b4[9]) + __uint_as_float(s1[r] & 0xFFFF0000u)};
      if (row < rows) {
        __builtin_memcpy(out + row * kOut + 4 * h, o, 16);
        if (h == 0) __builtin_memcpy(out + row * kOut + 8, o2, 8);
      }
    }
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) x[r][kt] = xn[r][kt];
  }
}

}  // namespace

void mlp_forward(const float *params, const uint16_t *F, int64_t rows, float *out, hipStream_t s) {
  constexpr int RT = 2;
  const int64_t tiles = ceil_div(rows, 4 * 32 * RT);
  // two workgroups a CU fit by LDS
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(tiles, 512));
  hipLaunchKernelGGL(k_mlp_forward<RT>, dim3(grid), dim3(256), 0, s, params, F, rows, out);
  check_launch("k_mlp_forward");
}

}  // namespace bbl
