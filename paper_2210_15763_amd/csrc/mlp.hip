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
#include <cmath>

#include "philox.h"

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
typedef short v4s __attribute__((ext_vector_type(4)));
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

// ----------------------------------------------------------------- training
// 16 x 16 output tiles: v_mfma_f32_16x16x16_bf16 has A[i][k] at lane
// i + 16 (k / 4), element k % 4; B[k][j] at lane j + 16 (k / 4), element
// k % 4; D[i][j] at lane j + 16 (i / 4), element i % 4, so an output with one
// row per lane is the next layer's B operand as it stands.  Two such operands
// side by side are one of v_mfma_f32_16x16x32_bf16 (over 32 products in an
// order that both operands share).
//
// The weights as bf16 operands in one scratch array that every workgroup of
// the gradient reads, in 16-byte pieces: piece (it, kp, lane) of W holds
// W[16 it + lane % 16][32 kp + 4 (lane / 16) + 0..3] and the four 16 columns
// on, those of a transposed matrix W[32 kp + 4 (lane / 16) + 0..3]
// [16 it + lane % 16] and the four 16 rows on.  W4^T has 16 (10) rows to
// contract, so its pieces are 8 bytes.
constexpr int kSquarePieces = 8 * 4 * 64;
constexpr int oF2 = 8 * 64, oF3 = oF2 + kSquarePieces, oF4 = oF3 + kSquarePieces;
constexpr int kFwdPieces = oF4 + 4 * 64;
constexpr int oT3 = kSquarePieces, oT4 = oT3 + kSquarePieces;  // within the transposed pieces
constexpr int kBackPieces = oT4 + 8 * 32;
constexpr int kPieces = kFwdPieces + kBackPieces;
constexpr int kGradRows = 128;    // rows per workgroup and pass: eight waves of 16
constexpr int kGradSlots = 256;   // workgroups (partial gradients) at most

__device__ __forceinline__ uint2 pack4(const float (&f)[4]) {
  return uint2{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3])};
}

// W[i][k .. k + 4), zero from column kmax (a multiple of 4) on
__device__ __forceinline__ uint2 row_part(const float *__restrict__ W, int ld, int i, int k,
                                          int kmax) {
  float f[4] = {0.f, 0.f, 0.f, 0.f};
  if (k < kmax) __builtin_memcpy(f, W + i * ld + k, 16);
  return pack4(f);
}

// W[i .. i + 4)[j], zero from row imax on
__device__ __forceinline__ uint2 column_part(const float *__restrict__ W, int i, int imax, int j) {
  float f[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = i + e < imax ? W[(i + e) * kHid + j] : 0.f;
  return pack4(f);
}

__device__ __forceinline__ uint4 join(uint2 a, uint2 b) { return uint4{a.x, a.y, b.x, b.y}; }

__device__ uint4 forward_piece(const float *__restrict__ p, int e) {
  const int l = e & 63, i = l & 15, k = 4 * (l >> 4);
  if (e < oF2) {
    const int it = e >> 6;
    return join(row_part(p + oW1, kIn, 16 * it + i, k, kIn),
                row_part(p + oW1, kIn, 16 * it + i, k + 16, kIn));
  }
  const bool last = e >= oF4;
  const float *W = p + (last ? oW4 : e < oF3 ? oW2 : oW3);
  const int t = (last ? e - oF4 : e < oF3 ? e - oF2 : e - oF3) >> 6;
  const int row = last ? i : 16 * (t >> 2) + i, kp = t & 3;
  const int kmax = last && i >= kOut ? 0 : kHid;
  return join(row_part(W, kHid, row, 32 * kp + k, kmax),
              row_part(W, kHid, row, 32 * kp + k + 16, kmax));
}

__device__ uint4 transposed_piece(const float *__restrict__ p, int e) {
  if (e < oT4) {
    const float *W = p + (e < oT3 ? oW2 : oW3);
    const int t = (e < oT3 ? e : e - oT3) >> 6, l = e & 63;
    const int i = 32 * (t & 3) + 4 * (l >> 4), j = 16 * (t >> 2) + (l & 15);
    return join(column_part(W, i, kHid, j), column_part(W, i + 16, kHid, j));
  }
  uint2 u[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int f = 2 * (e - oT4) + h, l = f & 63;
    u[h] = column_part(p + oW4, 4 * (l >> 4), kOut, 16 * (f >> 6) + (l & 15));
  }
  return join(u[0], u[1]);
}

// The operand tiles, and (batch > 0) the uniform row sample with replacement:
// idx[r] from Philox counter (r, step, 0, 12), reduced modulo the dataset size.
__global__ __launch_bounds__(256) void k_mlp_prepare(const float *__restrict__ params,
                                                     uint4 *__restrict__ pieces, int64_t batch,
                                                     int64_t total, uint64_t key, uint32_t step,
                                                     int64_t *__restrict__ idx) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < kPieces)
    pieces[t] = t < kFwdPieces ? forward_piece(params, (int)t)
                               : transposed_piece(params, (int)t - kFwdPieces);
  for (int64_t r = t; r < batch; r += (int64_t)gridDim.x * blockDim.x) {
    U4 c;
    c.v[0] = (uint32_t)r;
    c.v[1] = (uint32_t)((uint64_t)r >> 32);
    c.v[2] = step;
    c.v[3] = 12;
    const U4 o = philox4x32_10(c, (uint32_t)key, (uint32_t)(key >> 32));
    const uint64_t x = ((uint64_t)o.v[0] << 32) | o.v[1];
    idx[r] = (int64_t)(x % (uint64_t)total);
  }
}

__device__ __forceinline__ v4s as_v4s(uint2 u) {
  v4s v;
  __builtin_memcpy(&v, &u, 8);
  return v;
}
// over 16 products, and over 32 (both halves of a piece)
__device__ __forceinline__ v4f mma16(uint2 a, uint2 b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_v4s(a), as_v4s(b), c, 0, 0, 0);
}
__device__ __forceinline__ v4f mma32(uint4 a, uint4 b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_v8bf(a), as_v8bf(b), c, 0, 0, 0);
}
__device__ __forceinline__ uint2 lo(uint4 u) { return uint2{u.x, u.y}; }
__device__ __forceinline__ uint2 hi(uint4 u) { return uint2{u.z, u.w}; }

// acc where the unit was active (h > 0), else 0
__device__ __forceinline__ uint2 masked(const v4f &acc, uint2 h) {
  const float m[4] = {__uint_as_float(h.x << 16), __uint_as_float(h.x & 0xFFFF0000u),
                      __uint_as_float(h.y << 16), __uint_as_float(h.y & 0xFFFF0000u)};
  float f[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) f[q] = m[q] > 0.f ? acc[q] : 0.f;
  return pack4(f);
}

// Keeps the scheduler from raising the weight reads of all eight tiles of a
// layer above the first: they run one tile ahead (38 against 40 us at batch
// 16384).
__device__ __forceinline__ void one_tile_ahead() { __builtin_amdgcn_sched_barrier(0); }

// One hidden layer of 16 rows in both orientations: `out` (lane = row) is the
// next layer's operand, `outr` (lane = feature, rows in the registers) the
// operand of a product over the rows.  The same registers in the other order
// give the transposed output, bit for bit (both sum 16 products at a time, in
// order, as inference does).
template <int KP>
__device__ __forceinline__ void hidden_both(const uint4 *w, const float *bias, int lane,
                                            const uint4 (&in)[KP], uint4 (&out)[4],
                                            uint2 (&outr)[8]) {
  const int g = lane >> 4;
  uint4 next[KP];
#pragma unroll
  for (int kp = 0; kp < KP; ++kp) next[kp] = w[kp * 64 + lane];
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    v4f af{0.f, 0.f, 0.f, 0.f}, ar{0.f, 0.f, 0.f, 0.f};
    uint4 cur[KP];
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) {
      cur[kp] = next[kp];
      if (it < 7) next[kp] = w[((it + 1) * KP + kp) * 64 + lane];
    }
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) {
      const uint4 a = cur[kp];
      af = mma16(lo(a), lo(in[kp]), af);
      af = mma16(hi(a), hi(in[kp]), af);
      ar = mma16(lo(in[kp]), lo(a), ar);
      ar = mma16(hi(in[kp]), hi(a), ar);
    }
    v4f b;
    __builtin_memcpy(&b, bias + 16 * it + 4 * g, 16);
    const float br = bias[16 * it + (lane & 15)];
    float f[4], r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f[q] = relu(af[q] + b[q]);
      r[q] = relu(ar[q] + br);
    }
    const uint2 u = pack4(f);
    if (it & 1) out[it >> 1] = join(lo(out[it >> 1]), u);
    else out[it >> 1] = join(u, u);
    outr[it] = pack4(r);
    one_tile_ahead();
  }
}

// The error one layer back, masked by that layer's activations, in both
// orientations (F: the lane = row one is wanted).
template <bool F>
__device__ __forceinline__ void back_both(const uint4 *wt, int lane, const uint4 (&in)[4],
                                          const uint4 (&hf)[4], const uint2 (&hr)[8],
                                          uint4 (&out)[4], uint2 (&outr)[8]) {
  uint4 next[4];
#pragma unroll
  for (int kp = 0; kp < 4; ++kp) next[kp] = wt[kp * 64 + lane];
#pragma unroll
  for (int jt = 0; jt < 8; ++jt) {
    v4f af{0.f, 0.f, 0.f, 0.f}, ar{0.f, 0.f, 0.f, 0.f};
    uint4 cur[4];
#pragma unroll
    for (int kp = 0; kp < 4; ++kp) {
      cur[kp] = next[kp];
      if (jt < 7) next[kp] = wt[((jt + 1) * 4 + kp) * 64 + lane];
    }
#pragma unroll
    for (int kp = 0; kp < 4; ++kp) {
      const uint4 a = cur[kp];
      if constexpr (F) {
        af = mma16(lo(a), lo(in[kp]), af);
        af = mma16(hi(a), hi(in[kp]), af);
      }
      ar = mma16(lo(in[kp]), lo(a), ar);
      ar = mma16(hi(in[kp]), hi(a), ar);
    }
    if constexpr (F) {
      if (jt & 1) out[jt >> 1] = join(lo(out[jt >> 1]), masked(af, hi(hf[jt >> 1])));
      else out[jt >> 1] = join(masked(af, lo(hf[jt >> 1])), uint2{0u, 0u});
    }
    outr[jt] = masked(ar, hr[jt]);
    one_tile_ahead();
  }
}

// Tiles with the rows in the registers, as pieces of 32 rows: wave w holds
// rows 16 w .. 16 w + 16, half of piece [tile][w / 2][lane].
template <int NT>
__device__ __forceinline__ void put(uint4 *buf, int wave, int lane, const uint2 (&t)[NT]) {
#pragma unroll
  for (int i = 0; i < NT; ++i)
    reinterpret_cast<uint2 *>(buf + (i * 4 + (wave >> 1)) * 64 + lane)[wave & 1] = t[i];
}

// A workgroup's partial gradient, in the order the tiles leave the matrix
// cores: [tile][lane][4] for W3, W2 (tile 8 it + jt), W1 (2 it + jt), W4 (jt),
// element row 16 it + 4 (lane / 16) + e, column 16 jt + lane % 16, then the
// biases of layers 3, 2, 1, 4.  One 16-byte store a lane and tile.
constexpr int pW3 = 0, pW2 = pW3 + 64 * 256, pW1 = pW2 + 64 * 256, pW4 = pW1 + 16 * 256,
              pB3 = pW4 + 8 * 256, pB2 = pB3 + kHid, pB1 = pB2 + kHid, pB4 = pB1 + kHid,
              kSlot = pB4 + 16;

// Parameter index of an element of a partial, -1 for padding.
__device__ __forceinline__ int param_of(int e) {
  if (e >= pB3) {
    if (e >= pB4) return e - pB4 < kOut ? oB4 + e - pB4 : -1;
    return e < pB2 ? oB3 + e - pB3 : e < pB1 ? oB2 + e - pB2 : oB1 + e - pB1;
  }
  const int i = 4 * ((e >> 6) & 3) + (e & 3), j = (e >> 2) & 15;
  if (e < pW1) {
    const int t = (e < pW2 ? e : e - pW2) >> 8;
    return (e < pW2 ? oW3 : oW2) + (16 * (t >> 3) + i) * kHid + 16 * (t & 7) + j;
  }
  if (e < pW4) {
    const int t = (e - pW1) >> 8, c = 16 * (t & 1) + j;
    return c < kIn ? oW1 + (16 * (t >> 1) + i) * kIn + c : -1;
  }
  return i < kOut ? oW4 + i * kHid + 16 * ((e - pW4) >> 8) + j : -1;
}

// Adds (tile `it` of D)^T (tiles j0 .. j0 + NJ of H) over the 128 rows to NJ
// tiles at g, and the tile's row sums to 16 biases at gb.  first: the partial
// holds nothing yet.
template <int NJ>
__device__ __forceinline__ void weight_grad(const uint4 *D, int it, const uint4 *H, int j0,
                                            int lane, bool first, float *__restrict__ g,
                                            float *__restrict__ gb) {
  const uint32_t one = 0x3F803F80u;
  v4f G[NJ], Gb{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NJ; ++j) G[j] = v4f{0.f, 0.f, 0.f, 0.f};
  if (!first) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) G[j] = *reinterpret_cast<const v4f *>(g + j * 256 + 4 * lane);
    if (gb) Gb = *reinterpret_cast<const v4f *>(gb + 4 * (lane >> 4));
  }
#pragma unroll
  for (int kp = 0; kp < 4; ++kp) {
    const uint4 a = D[(it * 4 + kp) * 64 + lane];
    Gb = mma32(a, uint4{one, one, one, one}, Gb);
#pragma unroll
    for (int j = 0; j < NJ; ++j) G[j] = mma32(a, H[((j0 + j) * 4 + kp) * 64 + lane], G[j]);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) *reinterpret_cast<v4f *>(g + j * 256 + 4 * lane) = G[j];
  if (gb && (lane & 15) == 0) *reinterpret_cast<v4f *>(gb + 4 * (lane >> 4)) = Gb;
}

// N pieces from global memory to LDS by 512 threads, all loads in flight
// before the first is stored.
template <int N>
__device__ __forceinline__ void stage(const uint4 *__restrict__ src, uint4 *dst) {
  constexpr int U = (N + 511) / 512;
  uint4 t[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = u * 512 + (int)threadIdx.x;
    t[u] = src[e < N ? e : N - 1];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = u * 512 + (int)threadIdx.x;
    if (e < N) dst[e] = t[u];
  }
}

// Gradient of the mean squared error over `rows` rows (rows idx[] of X and T
// when idx is given) into one partial per workgroup.
//
// A wave takes 16 rows through the network and back with activations and
// errors in registers, each layer computed in both orientations: lane = row
// feeds the next layer, lane = feature is the operand of the weight gradients,
// which contract over the rows.  That is more matrix work than one orientation
// needs and saves every transposition.  The eight waves then pool their 128
// rows through LDS, one layer at a time, and each adds an eighth of the
// weight-gradient tiles to the workgroup's partial (19 tiles; held in
// registers over all passes they made the rest spill).  The forward pieces
// share their LDS with that exchange and are staged anew for each pass (76 KB
// from L2).  One workgroup of two waves a SIMD a CU; the chain of layers and
// the partials' traffic bound it at training batches.
struct GradShared {
  uint4 fwd[kFwdPieces];     // forward pieces, then the exchange of two 128 x 128 blocks
  uint4 back[kBackPieces];
  float b1[kHid], b2[kHid], b3[kHid], b4[16];
  bf16 x[kGradRows * kIn];   // the pass's rows and targets (zero past the end)
  float t[kGradRows * kOut];
  double loss[8];
};
static_assert(2 * kSquarePieces <= kFwdPieces, "the exchange fits over the forward pieces");
static_assert(sizeof(GradShared) <= 160 * 1024, "LDS of a compute unit");

__global__ __launch_bounds__(512, 2) void k_mlp_grad(const float *__restrict__ params,
                                                     const uint4 *__restrict__ pieces,
                                                     const bf16 *__restrict__ X,
                                                     const float *__restrict__ T, int64_t rows,
                                                     const int64_t *__restrict__ idx, float scale,
                                                     float *__restrict__ partial,
                                                     double *__restrict__ loss_part) {
  __shared__ GradShared w;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, lr = lane & 15;
  stage<kBackPieces>(pieces + kFwdPieces, w.back);
  if (threadIdx.x < kHid) {
    w.b1[threadIdx.x] = params[oB1 + threadIdx.x];
    w.b2[threadIdx.x] = params[oB2 + threadIdx.x];
    w.b3[threadIdx.x] = params[oB3 + threadIdx.x];
    if (threadIdx.x < 16) w.b4[threadIdx.x] = threadIdx.x < kOut ? params[oB4 + threadIdx.x] : 0.f;
  }
  const v4f zero{0.f, 0.f, 0.f, 0.f};
  float *gp = partial + (int64_t)blockIdx.x * kSlot;
  double lsum = 0.0;
  uint4 *exD = w.fwd, *exH = w.fwd + kSquarePieces;
  const int row = 16 * wave + lr;       // lane = row
  const int rowr = 16 * wave + 4 * g;   // lane = feature: rows rowr + 0..3
#pragma unroll 1
  for (int64_t r0 = (int64_t)blockIdx.x * kGradRows; r0 < rows;
       r0 += (int64_t)gridDim.x * kGradRows) {
    const bool first = r0 == (int64_t)blockIdx.x * kGradRows;
    __syncthreads();  // the last pass's exchange has been read
    {  // 7 + 5 pieces of 8 bytes a row, three a thread
      uint2 u[3];
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const int e = s * 512 + (int)threadIdx.x, r = e / 12, c = e % 12;
        u[s] = uint2{0u, 0u};
        if (r0 + r < rows) {
          const int64_t src = idx ? idx[r0 + r] : r0 + r;
          if (c < 7) __builtin_memcpy(&u[s], X + src * kIn + 4 * c, 8);
          else __builtin_memcpy(&u[s], T + src * kOut + 2 * (c - 7), 8);
        }
      }
      stage<kFwdPieces>(pieces, w.fwd);
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const int e = s * 512 + (int)threadIdx.x, r = e / 12, c = e % 12;
        if (c < 7) __builtin_memcpy(w.x + r * kIn + 4 * c, &u[s], 8);
        else __builtin_memcpy(w.t + r * kOut + 2 * (c - 7), &u[s], 8);
      }
    }
    __syncthreads();
    uint4 h1[4], h2[4], h3[4];
    uint2 h1r[8], h2r[8], h3r[8];
    {
      uint2 x0, x1{0u, 0u};
      __builtin_memcpy(&x0, w.x + row * kIn + 4 * g, 8);
      if (g < 3) __builtin_memcpy(&x1, w.x + row * kIn + 16 + 4 * g, 8);
      const uint4 x[1] = {join(x0, x1)};
      hidden_both<1>(w.fwd, w.b1, lane, x, h1, h1r);
    }
    hidden_both<4>(w.fwd + oF2, w.b2, lane, h1, h2, h2r);
    hidden_both<4>(w.fwd + oF3, w.b3, lane, h2, h3, h3r);
    // output layer and d loss / d out = scale * (out - target)
    uint2 d, dr[1];
    {
      v4f af = zero, ar = zero;
#pragma unroll
      for (int kp = 0; kp < 4; ++kp) {
        const uint4 a = w.fwd[oF4 + kp * 64 + lane];
        af = mma16(lo(a), lo(h3[kp]), af);
        af = mma16(hi(a), hi(h3[kp]), af);
        ar = mma16(lo(h3[kp]), lo(a), ar);
        ar = mma16(hi(h3[kp]), hi(a), ar);
      }
      float f[4], r[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 4 * g + q, cc = c < kOut ? c : 0;
        float o = ((af[q] + w.b4[cc]) + bf2f(w.x[row * kIn + kMlpSkip + cc])) - w.t[row * kOut + cc];
        o = c < kOut && r0 + row < rows ? o : 0.f;
        lsum += (double)o * o;
        f[q] = scale * o;
        const int cr = lr < kOut ? lr : 0;
        o = ((ar[q] + w.b4[cr]) + bf2f(w.x[(rowr + q) * kIn + kMlpSkip + cr])) -
            w.t[(rowr + q) * kOut + cr];
        r[q] = lr < kOut && r0 + rowr + q < rows ? scale * o : 0.f;
      }
      d = pack4(f);
      dr[0] = pack4(r);
    }
    __syncthreads();  // the forward pieces are read
    put(exD, wave, lane, dr);
    put(exH, wave, lane, h3r);
    __syncthreads();
    weight_grad<1>(exD, 0, exH, wave, lane, first, gp + pW4 + wave * 256,
                   wave == 0 ? gp + pB4 : nullptr);
    uint4 e3[4], e2[4];
    uint2 er[8];
#pragma unroll
    for (int jt = 0; jt < 8; ++jt) {
      const uint2 a = reinterpret_cast<const uint2 *>(w.back + oT4)[jt * 64 + lane];
      const v4f af = mma16(a, d, zero), ar = mma16(d, a, zero);
      if (jt & 1) e3[jt >> 1] = join(lo(e3[jt >> 1]), masked(af, hi(h3[jt >> 1])));
      else e3[jt >> 1] = join(masked(af, lo(h3[jt >> 1])), uint2{0u, 0u});
      er[jt] = masked(ar, h3r[jt]);
    }
    __syncthreads();
    put(exD, wave, lane, er);
    put(exH, wave, lane, h2r);
    __syncthreads();
    weight_grad<8>(exD, wave, exH, 0, lane, first, gp + pW3 + wave * 2048, gp + pB3 + 16 * wave);
    back_both<true>(w.back + oT3, lane, e3, h2, h2r, e2, er);
    __syncthreads();
    put(exD, wave, lane, er);
    put(exH, wave, lane, h1r);
    __syncthreads();
    weight_grad<8>(exD, wave, exH, 0, lane, first, gp + pW2 + wave * 2048, gp + pB2 + 16 * wave);
    back_both<false>(w.back, lane, e2, h1, h1r, e3, er);
    __syncthreads();
    put(exD, wave, lane, er);
    uint2 xr[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int c = 16 * t + lr;
      const bf16 *p = w.x + rowr * kIn + (c < kIn ? c : 0);
      const uint32_t x0 = p[0], x1 = p[kIn], x2 = p[2 * kIn], x3 = p[3 * kIn];
      xr[t] = c < kIn ? uint2{x0 | (x1 << 16), x2 | (x3 << 16)} : uint2{0u, 0u};
    }
    put(exH, wave, lane, xr);
    __syncthreads();
    weight_grad<2>(exD, wave, exH, 0, lane, first, gp + pW1 + wave * 512, gp + pB1 + 16 * wave);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
  if (lane == 0) w.loss[wave] = lsum;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < 8; ++i) s += w.loss[i];
    loss_part[blockIdx.x] = s;
  }
}

__device__ __forceinline__ float adam_one(float *p, float *m, float *v, int64_t i, float gi,
                                          float lr, float b1, float b2, float eps, float c1,
                                          float c2) {
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  return p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// grad[p] = sum over slots, or (grad null) one Adam step with that sum; loss =
// sum of loss partials / count.  A workgroup takes 64 elements, each wave
// every fourth slot with 16 loads in flight; fixed order.
__global__ __launch_bounds__(256) void k_mlp_grad_reduce(
    const float *__restrict__ partial, int slots, const double *__restrict__ loss_part,
    double inv_count, float *__restrict__ grad, float *__restrict__ loss, float *__restrict__ pw,
    float *__restrict__ m, float *__restrict__ v, float lr, float b1, float b2, float eps,
    float c1, float c2) {
  __shared__ float sum[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane, ec = e < kSlot ? e : kSlot - 1;
  float s = 0.f;
  int k = wave;
  for (; k + 60 < slots; k += 64) {
    float t[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) t[u] = partial[(int64_t)(k + 4 * u) * kSlot + ec];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += t[u];
  }
  for (; k < slots; k += 4) s += partial[(int64_t)k * kSlot + ec];
  sum[wave][lane] = s;
  __syncthreads();
  const int p = e < kSlot ? param_of(e) : -1;
  if (wave == 0 && p >= 0) {
    const float g = (sum[0][lane] + sum[1][lane]) + (sum[2][lane] + sum[3][lane]);
    if (grad) grad[p] = g;
    else pw[p] = adam_one(pw, m, v, p, g, lr, b1, b2, eps, c1, c2);
  }
  if (blockIdx.x == 0 && wave == 1 && loss) {
    double l = 0.0;
    for (int q = lane; q < slots; q += 64) l += loss_part[q];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) *loss = (float)(l * inv_count);
  }
}

__global__ void k_adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, int64_t count, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = adam_one(p, m, v, i, g[i], lr, b1, b2, eps, c1, c2);
}

// He-uniform weights (bound sqrt(6 / fan_in)), zero biases; Philox counter
// (index, 0, 0, 11) under the caller's key.
__global__ void k_mlp_init(float *__restrict__ p, uint64_t key) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kMlpParams) return;
  // hidden layers He-uniform; the output layer (and every bias) zero, so an
  // untrained network returns the P_D amplitudes unchanged
  int fan = 0;
  if (i < oB1) fan = kIn;
  else if (i >= oW2 && i < oB2) fan = kHid;
  else if (i >= oW3 && i < oB3) fan = kHid;
  if (fan == 0) {
    p[i] = 0.f;
    return;
  }
  U4 c;
  c.v[0] = (uint32_t)i;
  c.v[1] = 0;
  c.v[2] = 0;
  c.v[3] = 11;
  const U4 r = philox4x32_10(c, (uint32_t)key, (uint32_t)(key >> 32));
  const double u = u53(r.v[0], r.v[1]);
  p[i] = (float)((2.0 * u - 1.0) * sqrt(6.0 / fan));
}

int grad_slots(int64_t rows) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(rows, kGradRows), kGradSlots));
}

// Scratch of one gradient: operand tiles, partial gradients, loss partials.
struct GradScratch {
  uint4 *pieces;
  float *partial;
  double *loss;
  char *end;
};
GradScratch grad_scratch(char *base, int slots) {
  GradScratch g;
  g.pieces = reinterpret_cast<uint4 *>(base);
  base += align_up((size_t)kPieces * 16);
  g.partial = reinterpret_cast<float *>(base);
  base += align_up((size_t)slots * kSlot * 4);
  g.loss = reinterpret_cast<double *>(base);
  g.end = base + align_up((size_t)slots * 8);
  return g;
}

struct AdamArgs {
  float *p, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};
AdamArgs adam_args(float *p, float *m, float *v, int step, float lr, float b1, float b2,
                   float eps) {
  return AdamArgs{p, m, v, lr, b1, b2, eps, 1.f - std::pow(b1, (float)step),
                  1.f - std::pow(b2, (float)step)};
}

// Operand tiles (and the sample, batch > 0), gradient partials, their sum.
void grad_step(const float *params, const bf16 *F, const float *T, int64_t rows,
               const GradScratch &g, int64_t *idx, int64_t total, uint64_t key, int step,
               float *grad, float *loss, const AdamArgs &a, hipStream_t s) {
  const int slots = grad_slots(rows);
  const int64_t sample = idx ? rows : 0;
  const int64_t blocks = std::max<int64_t>(ceil_div(kPieces, 256),
                                           std::min<int64_t>(ceil_div(sample, 256), 1024));
  hipLaunchKernelGGL(k_mlp_prepare, dim3((unsigned)blocks), dim3(256), 0, s, params, g.pieces,
                     sample, total, key, (uint32_t)step, idx);
  check_launch("k_mlp_prepare");
  const float scale = (float)(2.0 / ((double)rows * kOut));
  hipLaunchKernelGGL(k_mlp_grad, dim3(slots), dim3(512), 0, s, params, g.pieces, F, T, rows, idx,
                     scale, g.partial, g.loss);
  check_launch("k_mlp_grad");
  hipLaunchKernelGGL(k_mlp_grad_reduce, dim3((unsigned)ceil_div(kSlot, 64)), dim3(256), 0, s,
                     g.partial, slots, g.loss, 1.0 / ((double)rows * kOut), grad, loss, a.p, a.m,
                     a.v, a.lr, a.b1, a.b2, a.eps, a.c1, a.c2);
  check_launch("k_mlp_grad_reduce");
}

char *scratch_base(void *ws) {
  return reinterpret_cast<char *>(align_up(reinterpret_cast<uintptr_t>(ws), 256));
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

void mlp_init(float *params, uint64_t key, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_init, dim3((unsigned)ceil_div(kMlpParams, 256)), dim3(256), 0, s,
                     params, key);
  check_launch("k_mlp_init");
}

size_t mlp_grad_bytes(int64_t rows) {
  return (size_t)(grad_scratch(nullptr, grad_slots(rows)).end - (char *)nullptr) + 256;
}

void mlp_grad(const float *params, const uint16_t *F, const float *T, int64_t rows, void *ws,
              float *grad, float *loss, hipStream_t s) {
  grad_step(params, F, T, rows, grad_scratch(scratch_base(ws), grad_slots(rows)), nullptr, 0, 0, 0,
            grad, loss, AdamArgs{}, s);
}

void mlp_adam(float *p, float *m, float *v, const float *g, int64_t count, int step, float lr,
              float b1, float b2, float eps, hipStream_t s) {
  const AdamArgs a = adam_args(p, m, v, step, lr, b1, b2, eps);
  hipLaunchKernelGGL(k_adam, dim3(capped_grid(ceil_div(count, 256), 256)), dim3(256), 0, s, p, m,
                     v, g, count, lr, b1, b2, eps, a.c1, a.c2);
  check_launch("k_adam");
}

size_t mlp_train_bytes(int64_t batch) { return mlp_grad_bytes(batch) + align_up((size_t)batch * 8); }

void mlp_train_step(float *params, float *m, float *v, int step, float lr, const uint16_t *F,
                    const float *T, int64_t total, int64_t batch, uint64_t key, void *ws,
                    float *loss, hipStream_t s) {
  const GradScratch g = grad_scratch(scratch_base(ws), grad_slots(batch));
  grad_step(params, F, T, batch, g, reinterpret_cast<int64_t *>(g.end), total, key, step, nullptr,
            loss, adam_args(params, m, v, step, lr, 0.9f, 0.999f, 1e-8f), s);
}

}  // namespace bbl
