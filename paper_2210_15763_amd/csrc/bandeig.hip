// Lowest eigenpairs of the block-tridiagonal band matrix T_j built from the
// A's and B's (Methods, block Lanczos: the paper hands this small band matrix
// to standard dense LAPACK eigensolvers).  On the GPU it is solved by
//   1. Sturm-count multisection: the number of negative pivots of the band
//      LDL^T factorisation of (T - sigma I) equals the number of eigenvalues
//      below sigma (Sylvester's law of inertia); many shifts are counted at
//      once, one lane per shift with the factorisation window in registers
//      (bandwidths 1, 2, 4, 8, 10, 16) or one 64-lane workgroup per shift;
//   2. inverse iteration on each wanted eigenvalue with the same band LDL^T;
//      in both, the register path factors from the two ends of the matrix
//      towards a middle block, two lanes a shift, which halves the chain of
//      dependent rows that bounds them;
//   3. a Rayleigh-Ritz step on the span of the inverse-iteration vectors, which
//      orthonormalises them and refines the Ritz values.
// Only the k lowest eigenpairs (and the largest eigenvalue, for ||H||_est) are
// computed, in FP64.  Band storage: band[i*(kd+1) + d] = T[i][i-d], d = 0..kd.
#include "bandeig.h"
#include "common.h"
#include "small.h"

namespace bbl {
namespace {

constexpr int kChunk = 64;               // band rows staged in LDS at a time
constexpr int kMaxW = kMaxBlock + 1;     // window width (kd + 1)
constexpr int kMaxPairs = kMaxBlock * (kMaxBlock + 1) / 2;
constexpr int kMaxPPT = (kMaxPairs + 63) / 64;   // pairs per thread

// One band LDL^T sweep of (T - sigma I) by a 64-lane workgroup.  The active
// trailing window (rows/cols k..k+kd) lives in LDS with circular slots
// (absolute index i -> slot i % W).  Returns the number of negative pivots.
// With store = true, the unit-lower multipliers L[k][r-1] = l_{k+r,k} and the
// pivots D[k] are written out.
__device__ int ldl_sweep(const double *__restrict__ Tb, int N, int kd, double sigma,
                         double pivmin, bool store, double *win, double *chunk, double *L,
                         double *D) {
  const int W = kd + 1;
  const int NP = kd * (kd + 1) / 2;
  const int t = threadIdx.x;
  // this thread's (r, c) pairs, 1 <= c <= r <= kd, and their current slots
  int pr[kMaxPPT], rs[kMaxPPT], cs[kMaxPPT];
#pragma unroll
  for (int q = 0; q < kMaxPPT; ++q) {
    const int e = t + 64 * q;
    int r = 1, base = 0;
    while (e < NP && base + r <= e) {
      base += r;
      ++r;
    }
    const int c = (e < NP) ? e - base + 1 : 1;
    pr[q] = (e < NP) ? r : 1 << 20;  // out-of-range pairs never update
    rs[q] = r % W;
    cs[q] = c % W;
  }
  // rows 0..W-1 of the band into the window; then stream chunks
  for (int i = t; i < min(kChunk, N) * W; i += blockDim.x) chunk[i] = Tb[i];
  __syncthreads();
  for (int e = t; e < W * W; e += blockDim.x) {
    const int r = e / W, c = e % W;
    double v = 0.0;
    if (r < N && c <= r) {
      v = chunk[r * W + (r - c)];
      if (r == c) v -= sigma;
    }
    win[e] = v;
  }
  __syncthreads();
  int cnt = 0;
  int ks = 0;
  for (int k = 0; k < N; ++k) {
    double d = win[ks * W + ks];
    if (fabs(d) < pivmin) d = (store && d > 0.0) ? pivmin : -pivmin;
    cnt += (d < 0.0) ? 1 : 0;
    const double inv = 1.0 / d;
    if (store) {
      if (t == 0) D[k] = d;
      if (t < kd) {
        int sl = ks + 1 + t;
        if (sl >= W) sl -= W;
        L[(int64_t)k * kd + t] = (k + 1 + t < N) ? win[sl * W + ks] * inv : 0.0;
      }
    }
#pragma unroll
    for (int q = 0; q < kMaxPPT; ++q) {
      if (k + pr[q] < N) {
        const double wr = win[rs[q] * W + ks] * inv;  // multiplier l_{r,k}
        const double lc = win[cs[q] * W + ks];
        win[rs[q] * W + cs[q]] = fma(-wr, lc, win[rs[q] * W + cs[q]]);
      }
      rs[q] = (rs[q] + 1 == W) ? 0 : rs[q] + 1;
      cs[q] = (cs[q] + 1 == W) ? 0 : cs[q] + 1;
    }
    __syncthreads();
    const int nr = k + W;  // row entering the window, into slot ks
    if (nr < N) {
      if (nr % kChunk == 0) {
        const int rows = min(kChunk, N - nr);
        for (int i = t; i < rows * W; i += blockDim.x) chunk[i] = Tb[(int64_t)nr * W + i];
        __syncthreads();
      }
      if (t < W) {
        double v = chunk[(nr % kChunk) * W + t];  // T[nr][nr - t]
        if (t == 0) v -= sigma;
        int sl = ks - t;  // slot of column nr - t  (nr = ks mod W)
        if (sl < 0) sl += W;
        win[ks * W + sl] = v;
      }
    }
    ks = (ks + 1 == W) ? 0 : ks + 1;
    __syncthreads();
  }
  return cnt;
}

__global__ __launch_bounds__(64) void k_sturm(const double *__restrict__ Tb, int N, int kd,
                                              const double *__restrict__ shifts,
                                              int *__restrict__ counts, double pivmin) {
  extern __shared__ double smem[];
  double *win = smem;
  double *chunk = smem + (kd + 1) * (kd + 1);
  const int c = ldl_sweep(Tb, N, kd, shifts[blockIdx.x], pivmin, false, win, chunk, nullptr,
                          nullptr);
  if (threadIdx.x == 0) counts[blockIdx.x] = c;
}

// Register-window band LDL^T for a compile-time bandwidth KD: one shift per
// lane.  The (KD+1) x (KD+1) trailing window of the partially factored
// T - sigma I is held as its lower triangle in registers, indexed by circular
// slots; the row loop is unrolled by KD + 1 so that every slot index is a
// compile-time constant.  Band rows are the same for all lanes (uniform
// loads).  Step k: pivot d = R[k][k], multipliers w_i = R[k+i][k] / d, update
// R[k+i][k+j] -= w_i R[k+j][k]; the same arithmetic as ldl_sweep.
constexpr int tri(int a, int b) { return a >= b ? a * (a + 1) / 2 + b : b * (b + 1) / 2 + a; }

// Steps M..KD of one unrolled group of W = KD + 1 rows, slot indices static.
// STORE: multipliers l_{k+i,k} to L[(k*KD + i-1) * ls] and 1/d to
// Dinv[k * ls] (a tiny pivot keeps its sign there); otherwise a tiny pivot
// counts as negative.  ls interleaves the factors of ls lanes.
// FULL: every row of the group and every row entering the window lies inside
// the matrix, so the group is straight-line code whose band loads can be
// issued ahead of the pivot's division; otherwise rows are checked and the
// entering row's loads are clamped to the last row (and zeroed after).
template <int KD, int M, bool STORE, bool FULL>
__device__ __forceinline__ void ldl_steps(const double *__restrict__ Tb, int N, int k0,
                                          double sigma, double pivmin,
                                          double (&R)[(KD + 1) * (KD + 2) / 2], int &cnt,
                                          double *__restrict__ L, double *__restrict__ Dinv,
                                          int ls) {
  if constexpr (M <= KD) {
    constexpr int W = KD + 1;
    const int k = k0 + M;
    if (FULL || k < N) {
      // row k + W enters in the slot freed by this step: T[k+W][k+W-t]
      const int nr = k + W;
      const bool nin = FULL || nr < N;
      const double *rowp = Tb + (int64_t)(FULL ? nr : min(nr, N - 1)) * W;
      double nv[W];
#pragma unroll
      for (int t = 0; t <= KD; ++t) nv[t] = rowp[t];
      // relative row i of the window lives in slot (M + i) % W
      double d = R[tri(M, M)];
      if (fabs(d) < pivmin) d = (STORE && d > 0.0) ? pivmin : -pivmin;
      cnt += d < 0.0 ? 1 : 0;
      const double inv = newton_inv(d);
      double w[KD + 1];
#pragma unroll
      for (int i = 1; i <= KD; ++i) w[i] = R[tri((M + i) % W, M)] * inv;
      if constexpr (STORE) {
        Dinv[(int64_t)k * ls] = inv;
#pragma unroll
        for (int i = 1; i <= KD; ++i)
          L[((int64_t)k * KD + i - 1) * ls] = (FULL || k + i < N) ? w[i] : 0.0;
      }
#pragma unroll
      for (int i = 1; i <= KD; ++i) {
        const int si = (M + i) % W;
#pragma unroll
        for (int j = 1; j <= i; ++j) {
          const int sj = (M + j) % W;
          R[tri(si, sj)] = fma(-w[i], R[tri(sj, M)], R[tri(si, sj)]);
        }
      }
#pragma unroll
      for (int t = 0; t <= KD; ++t) {
        const double v = t == 0 ? nv[0] - sigma : nv[t];
        R[tri(M, (M + W - t) % W)] = nin ? v : 0.0;
      }
      ldl_steps<KD, M + 1, STORE, FULL>(Tb, N, k0, sigma, pivmin, R, cnt, L, Dinv, ls);
    }
  }
}

// The whole band LDL^T sweep: full groups first, then the tail.
template <int KD, bool STORE>
__device__ __forceinline__ void ldl_sweep_reg(const double *__restrict__ Tb, int N, double sigma,
                                              double pivmin, double (&R)[(KD + 1) * (KD + 2) / 2],
                                              int &cnt, double *__restrict__ L,
                                              double *__restrict__ Dinv, int ls) {
  constexpr int W = KD + 1;
  int k0 = 0;
  // one group of W rows per trip; unrolling this loop further would only
  // multiply the code (the group is already W steps of straight-line code)
#pragma unroll 1
  for (; k0 + 2 * W <= N; k0 += W)
    ldl_steps<KD, 0, STORE, true>(Tb, N, k0, sigma, pivmin, R, cnt, L, Dinv, ls);
#pragma unroll 1
  for (; k0 < N; k0 += W)
    ldl_steps<KD, 0, STORE, false>(Tb, N, k0, sigma, pivmin, R, cnt, L, Dinv, ls);
}

// Window of rows 0..KD of T - sigma I.
template <int KD>
__device__ __forceinline__ void ldl_window_init(const double *__restrict__ Tb, int N, double sigma,
                                                double (&R)[(KD + 1) * (KD + 2) / 2]) {
  constexpr int W = KD + 1;
#pragma unroll
  for (int r = 0; r < W; ++r)
#pragma unroll
    for (int c = 0; c <= r; ++c) {
      double v = 0.0;
      if (r < N) {
        v = Tb[(int64_t)r * W + (r - c)];
        if (r == c) v -= sigma;
      }
      R[tri(r, c)] = v;
    }
}

// ------------------------------------------------- two-sided factorisation
// Rows 0 .. m1 are eliminated from the top and, at the same time by another
// wave, rows N - 1 .. N - m2 from the bottom (the same sweep on the matrix with
// its rows and columns reversed); the middle block of KD rows couples to both,
// collects both Schur updates and is factored last.  Both sweeps run whole
// groups of W = KD + 1 rows, so that a row's window slot is a compile-time
// index: m2 is a multiple of W, and the top sweep starts `pad` rows before row
// 0, identity rows that couple to nothing.
struct Split {
  int m1, m2, pad;
};
__host__ __device__ inline Split split_rows(int N, int kd) {
  const int W = kd + 1;
  Split s;
  s.m2 = N > kd ? (N - kd) / 2 / W * W : 0;
  s.m1 = N - kd - s.m2;
  s.pad = (W - s.m1 % W) % W;
  return s;
}

// The band rows that enter a sweep's window, staged in LDS by the sweep's own
// wave a chunk of groups at a time, the next chunk's loads in flight meanwhile.
// (Read straight from memory, by scalar loads, a step took 0.21 us at kd = 8:
// scalar loads return out of order, so a wave can only wait for all of them;
// with the stage it takes 0.13.)
template <int KD>
struct BandStage {
  static constexpr int W = KD + 1;
  // groups of W rows: about 72 rows, at most 11 doubles a lane
  static constexpr int G = 72 / W < 704 / (W * W) ? 72 / W : 704 / (W * W);
  static constexpr int E = G * W * W;              // doubles of a chunk
  static constexpr int PER = (E + 63) / 64;
  const double *Tb;
  double *buf;
  int64_t next, last;
  int lane;
  double pre[PER];
  __device__ __forceinline__ BandStage(const double *Tb_, int N, int pad, double *buf_, int lane_)
      : Tb(Tb_), buf(buf_), next((int64_t)(W - pad) * W), last((int64_t)N * W - 1), lane(lane_) {
    load();
    // slots d > i of row i hold no entry of the matrix, whatever is in them; of
    // the entering rows only those of the first chunk (of at least W) have any
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = (W - pad) * W + lane + 64 * u;
      if (i % W > i / W) pre[u] = 0.0;
    }
  }
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int64_t i = next + lane + 64 * u;
      pre[u] = Tb[i < last ? i : last];  // past the end only rows that are never used
    }
    next += E;
  }
  // the loaded chunk to LDS, the next one on its way
  __device__ __forceinline__ const double *turn() {
    wave_fence();
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (lane + 64 * u < E) buf[lane + 64 * u] = pre[u];
    wave_fence();
    load();
    return buf;
  }
};

// Window of rows -pad .. KD - pad of T - sigma I.
template <int KD>
__device__ __forceinline__ void window_init(const double *__restrict__ Tb, int pad, double sigma,
                                            double (&R)[(KD + 1) * (KD + 2) / 2]) {
  constexpr int W = KD + 1;
#pragma unroll
  for (int r = 0; r < W; ++r)
#pragma unroll
    for (int c = 0; c <= r; ++c) {
      double v = r == c ? 1.0 : 0.0;
      if (r >= pad) {
        v = 0.0;
        if (c >= pad) v = Tb[(int64_t)(r - pad) * W + (r - c)] - (r == c ? sigma : 0.0);
      }
      R[tri(r, c)] = v;
    }
}

// Steps M .. KD of a group of W rows; rows: the W band rows that enter.  A tiny
// pivot counts as negative.
template <int KD, int M>
__device__ __forceinline__ void group_steps(const double *rows, double sigma, double pivmin,
                                            double (&R)[(KD + 1) * (KD + 2) / 2], int &cnt) {
  if constexpr (M <= KD) {
    constexpr int W = KD + 1;
    double nv[W];
#pragma unroll
    for (int t = 0; t <= KD; ++t) nv[t] = rows[M * W + t];
    double d = R[tri(M, M)];
    if (fabs(d) < pivmin) d = -pivmin;
    cnt += d < 0.0 ? 1 : 0;
    const double inv = newton_inv(d);
    double w[KD + 1];
#pragma unroll
    for (int i = 1; i <= KD; ++i) w[i] = R[tri((M + i) % W, M)] * inv;
#pragma unroll
    for (int i = 1; i <= KD; ++i) {
      const int si = (M + i) % W;
#pragma unroll
      for (int j = 1; j <= i; ++j) {
        const int sj = (M + j) % W;
        R[tri(si, sj)] = fma(-w[i], R[tri(sj, M)], R[tri(si, sj)]);
      }
    }
#pragma unroll
    for (int t = 0; t <= KD; ++t) R[tri(M, (M + W - t) % W)] = t == 0 ? nv[0] - sigma : nv[t];
    group_steps<KD, M + 1>(rows, sigma, pivmin, R, cnt);
  }
}

// The sweep over rows -pad .. m of one end; leaves the window of rows m .. m + KD.
template <int KD>
__device__ __forceinline__ void end_sweep(const double *__restrict__ Tb, int N, int m, int pad,
                                          double sigma, double pivmin,
                                          double (&R)[(KD + 1) * (KD + 2) / 2], int &cnt,
                                          double *buf, int lane) {
  constexpr int W = KD + 1;
  window_init<KD>(Tb, pad, sigma, R);
  BandStage<KD> st(Tb, N, pad, buf, lane);
#pragma unroll 1
  for (int k0 = -pad; k0 < m;) {
    const double *rows = st.turn();
#pragma unroll 1
    for (int g = 0; g < BandStage<KD>::G && k0 < m; ++g, k0 += W)
      group_steps<KD, 0>(rows + g * W * W, sigma, pivmin, R, cnt);
  }
}

// Adds the bottom sweep's window (entry (a, c), a >= c, at ex[tri(a, c) * es])
// to the top one's: T - sigma I is in both, so it is taken out once.
template <int KD>
__device__ __forceinline__ void merge_middle(const double *__restrict__ Tb, int m1, double sigma,
                                             const double *ex, int es,
                                             double (&R)[(KD + 1) * (KD + 2) / 2]) {
#pragma unroll
  for (int r = 0; r < KD; ++r)
#pragma unroll
    for (int c = 0; c <= r; ++c) {
      const double t = Tb[(int64_t)(m1 + r) * (KD + 1) + (r - c)] - (r == c ? sigma : 0.0);
      R[tri(r, c)] += ex[tri(KD - 1 - c, KD - 1 - r) * es] - t;
    }
}

// LDL^T of the middle block.
template <int KD>
__device__ __forceinline__ void middle_steps(double pivmin, double (&R)[(KD + 1) * (KD + 2) / 2],
                                             int &cnt) {
#pragma unroll
  for (int s = 0; s < KD; ++s) {
    double d = R[tri(s, s)];
    if (fabs(d) < pivmin) d = -pivmin;
    cnt += d < 0.0 ? 1 : 0;
    const double inv = newton_inv(d);
#pragma unroll
    for (int i = s + 1; i < KD; ++i) {
      const double w = R[tri(i, s)] * inv;
#pragma unroll
      for (int j = s + 1; j <= i; ++j) R[tri(i, j)] = fma(-w, R[tri(j, s)], R[tri(i, j)]);
    }
  }
}

// Multisection.  Round 0 spreads nsh shifts evenly over the Gershgorin
// interval, shared by all targets; later rounds give each target SP shifts
// inside its bracket.  Target t < k is eigenvalue index t; target k is index
// N - 1 (the largest).  count(sigma) = number of eigenvalues below sigma, so
// lambda_idx lies in [max{sigma: count <= idx}, min{sigma: count > idx}].  A
// round's shifts follow from its brackets, so only the counts are stored; the
// next kernel narrows the brackets itself (every workgroup the one it needs,
// from the 4 SP or 4 nsh bytes of counts) instead of a launch in between.
constexpr int kGershMax = 64;  // workgroups of k_gersh: one bound a lane
__device__ __forceinline__ double gersh_pad(double lo, double hi) {
  return 1e-12 * fmax(fabs(lo), fabs(hi)) + 1e-300;
}

struct Bisect {
  const double *gersh;  // (lower, upper) bounds of ng parts
  int ng;
  double *brk;          // [round][target][2]: bracket at the start of round >= 1
  int *counts[2];       // counts of even and odd rounds
  int nsh, SP, k, N;
};

// The padded Gershgorin interval, by every wave for itself.
__device__ __forceinline__ void gersh_interval(const Bisect &B, double &lo, double &hi) {
  const int g = min((int)threadIdx.x & 63, B.ng - 1);
  lo = B.gersh[2 * g];
  hi = B.gersh[2 * g + 1];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  if (B.ng > 1) {
    const double pad = gersh_pad(lo, hi);
    lo -= pad;
    hi += pad;
  }
}

__device__ __forceinline__ double shift_at(double lo, double hi, int s, int S) {
  return lo + (hi - lo) * (double)(s + 1) / (double)(S + 1);
}

// Target tg's bracket at the start of `round` (>= 1), by all THREADS threads;
// red: 2 * THREADS doubles of LDS.
template <int THREADS>
__device__ __forceinline__ void bracket(const Bisect &B, int round, int tg, double *red,
                                        double &lo, double &hi) {
  const int NT = B.k + 1, idx = tg < B.k ? tg : B.N - 1;
  const bool shared = round == 1;
  double lo0, hi0;
  if (shared) {
    gersh_interval(B, lo0, hi0);
  } else {
    const double *b0 = B.brk + (round - 1) * 2 * NT + 2 * tg;
    lo0 = b0[0];
    hi0 = b0[1];
  }
  const int S = shared ? B.nsh : B.SP;
  const int *c = B.counts[(round - 1) & 1] + (shared ? 0 : tg * B.SP);
  double l = lo0, h = hi0;
  for (int s0 = 4 * (int)threadIdx.x; s0 < S; s0 += 4 * THREADS) {  // S: a multiple of 4
    const int4 v = *reinterpret_cast<const int4 *>(c + s0);
    const int cv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double sg = shift_at(lo0, hi0, s0 + e, S);
      if (cv[e] <= idx) l = fmax(l, sg);
      else h = fmin(h, sg);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    l = fmax(l, __shfl_xor(l, off, 64));
    h = fmin(h, __shfl_xor(h, off, 64));
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = l;
    red[2 * (threadIdx.x >> 6) + 1] = h;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    l = fmax(l, red[2 * w]);
    h = fmin(h, red[2 * w + 1]);
  }
  if (l > h) {  // rounding made the counts non-monotone: keep the crossing
    const double m = 0.5 * (l + h);
    l = m;
    h = m;
  }
  lo = l;
  hi = h;
}

// Sturm counts of one round, 64 shifts a workgroup: wave 0 from the top, wave
// 1 from the bottom.  Tr: the reversed band.  Bound by the issue of a row's KD
// (KD + 1) / 2 FP64 multiply-adds (0.13 us a row at kd = 8).  Measured a round at
// N = 1448, kd = 8: 98 us (216 from one end, plus 7 for a launch that narrowed
// the brackets); N = 352, kd = 4 19 (35 + 7); N = 640, kd = 16, whose window
// overflows into accumulation registers, 259 (548 by a workgroup per shift).
template <int KD>
__global__ __launch_bounds__(128) void k_sturm_reg(const double *__restrict__ T,
                                                   const double *__restrict__ Tr, int N, Bisect B,
                                                   int round, double pivmin) {
  constexpr int NP = KD * (KD + 1) / 2;
  __shared__ double ex[NP * 64];
  __shared__ int exc[64];
  __shared__ double red[4], buf[2][BandStage<KD>::E];
  const int lane = threadIdx.x & 63, up = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double lo, hi;
  int s = (int)blockIdx.x * 64 + lane, S = B.nsh;
  if (round == 0) {
    gersh_interval(B, lo, hi);
  } else {
    const int per = B.SP / 64, tg = (int)blockIdx.x / per;
    bracket<128>(B, round, tg, red, lo, hi);
    s -= tg * B.SP;
    S = B.SP;
    if ((int)blockIdx.x % per == 0 && threadIdx.x == 0) {
      double *b = B.brk + round * 2 * (B.k + 1) + 2 * tg;
      b[0] = lo;
      b[1] = hi;
    }
  }
  const double sigma = shift_at(lo, hi, s, S);
  int *counts = B.counts[round & 1] + (int)blockIdx.x * 64;
  double R[(KD + 1) * (KD + 2) / 2];
  int cnt = 0;
  const Split sp = split_rows(N, KD);
  if (sp.m2 == 0) {  // too short to split
    if (up) return;
    ldl_window_init<KD>(T, N, sigma, R);
    ldl_sweep_reg<KD, false>(T, N, sigma, pivmin, R, cnt, nullptr, nullptr, 0);
    counts[lane] = cnt;
    return;
  }
  end_sweep<KD>(up ? Tr : T, N, up ? sp.m2 : sp.m1, up ? 0 : sp.pad, sigma, pivmin, R, cnt,
                buf[up], lane);
  if (up) {
#pragma unroll
    for (int r = 0; r < KD; ++r)
#pragma unroll
      for (int c = 0; c <= r; ++c) ex[tri(r, c) * 64 + lane] = R[tri(r, c)];
    exc[lane] = cnt;
  }
  __syncthreads();
  if (up) return;
  merge_middle<KD>(T, sp.m1, sigma, ex + lane, 64, R);
  middle_steps<KD>(pivmin, R, cnt);
  counts[lane] = cnt + exc[lane];
}

void sturm_reg(const double *T, const double *Tr, int N, int kd, const Bisect &B, int round,
               double pivmin, hipStream_t s) {
  const unsigned g = (unsigned)((round == 0 ? B.nsh : (B.k + 1) * B.SP) / 64);
#define BBL_STURM(K)                                                                            \
  case K:                                                                                       \
    hipLaunchKernelGGL(k_sturm_reg<K>, dim3(g), dim3(128), 0, s, T, Tr, N, B, round, pivmin);   \
    break;
  switch (kd) {
    BBL_STURM(1)
    BBL_STURM(2)
    BBL_STURM(4)
    BBL_STURM(8)
    BBL_STURM(10)
    BBL_STURM(16)
  }
#undef BBL_STURM
  check_launch("k_sturm_reg");
}

// Final brackets, for the kernels that read them from memory.
__global__ __launch_bounds__(128) void k_final_brackets(Bisect B, int rounds, double *brk) {
  __shared__ double red[4];
  double lo, hi;
  bracket<128>(B, rounds, blockIdx.x, red, lo, hi);
  if (threadIdx.x == 0) {
    brk[2 * blockIdx.x] = lo;
    brk[2 * blockIdx.x + 1] = hi;
  }
}

// Gershgorin bounds of each workgroup's rows, (lower, upper) pairs in out (one
// workgroup: the padded interval itself); and (Tr not null) the band with rows
// and columns reversed, Tr[i][d] = T[N-1-i+d][N-1-i].
__global__ __launch_bounds__(128) void k_gersh(const double *__restrict__ Tb, int N, int kd,
                                               double *out, double *__restrict__ Tr) {
  __shared__ double slo[2], shi[2];
  const int W = kd + 1;
  double lo = 1e300, hi = -1e300;
  for (int i = blockIdx.x * 128 + threadIdx.x; i < N; i += gridDim.x * 128) {
    double s = 0.0;
    const double a = Tb[(int64_t)i * W];
    if (Tr) Tr[(int64_t)(N - 1 - i) * W] = a;
#pragma unroll 8
    for (int d = 1; d <= kd; ++d) {
      const double l = i - d >= 0 ? Tb[(int64_t)i * W + d] : 0.0;
      const double v = i + d < N ? Tb[(int64_t)(i + d) * W + d] : 0.0;
      s += fabs(l) + fabs(v);
      if (Tr) Tr[(int64_t)(N - 1 - i) * W + d] = v;
    }
    lo = fmin(lo, a - s);
    hi = fmax(hi, a + s);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    slo[threadIdx.x >> 6] = lo;
    shi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    lo = fmin(slo[0], slo[1]);
    hi = fmax(shi[0], shi[1]);
    const double pad = gridDim.x == 1 ? gersh_pad(lo, hi) : 0.0;
    out[2 * blockIdx.x] = lo - pad;
    out[2 * blockIdx.x + 1] = hi + pad;
  }
}

// Round 1: shared shifts evenly spaced strictly inside [lo, hi].
__global__ void k_bisect_init(const double *gersh, int S, double *shifts, double *brk, int NT) {
  const double lo = gersh[0], hi = gersh[1];
  for (int s = threadIdx.x + blockIdx.x * blockDim.x; s < S; s += blockDim.x * gridDim.x)
    shifts[s] = lo + (hi - lo) * (double)(s + 1) / (double)(S + 1);
  if (blockIdx.x == 0)
    for (int t = threadIdx.x; t < NT; t += blockDim.x) {
      brk[2 * t] = lo;
      brk[2 * t + 1] = hi;
    }
}

// Narrow one target's bracket (workgroup tg) from the counts of the last
// round, then lay out S_next shifts inside it.  Target t < k is eigenvalue
// index t; target k is index N - 1 (the largest).  count(sigma) = number of
// eigenvalues below sigma, so lambda_idx lies in
// [max{sigma: count <= idx}, min{sigma: count > idx}].  In the shared round
// every target scans all S_per shifts; afterwards target tg owns shifts
// [tg S_per, (tg + 1) S_per).
__global__ __launch_bounds__(256) void k_bisect_update(int shared_round, const double *shifts,
                                                       const int *counts, int S_per, int N,
                                                       int k, double *brk, int S_next,
                                                       double *next_shifts) {
  __shared__ double slo[256], shi[256];
  const int tg = blockIdx.x;
  const int idx = (tg < k) ? tg : N - 1;
  const int s0 = shared_round ? 0 : tg * S_per;
  double lo = brk[2 * tg], hi = brk[2 * tg + 1];
  for (int s = threadIdx.x; s < S_per; s += blockDim.x) {
    const double sg = shifts[s0 + s];
    const int c = counts[s0 + s];
    if (c <= idx) lo = fmax(lo, sg);
    else hi = fmin(hi, sg);
  }
  slo[threadIdx.x] = lo;
  shi[threadIdx.x] = hi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      slo[threadIdx.x] = fmax(slo[threadIdx.x], slo[threadIdx.x + w]);
      shi[threadIdx.x] = fmin(shi[threadIdx.x], shi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  double l = slo[0], h = shi[0];
  if (l > h) {  // rounding made the counts non-monotone: keep the crossing
    const double m = 0.5 * (l + h);
    l = m;
    h = m;
  }
  if (threadIdx.x == 0) {
    brk[2 * tg] = l;
    brk[2 * tg + 1] = h;
  }
  if (next_shifts)
    for (int s = threadIdx.x; s < S_next; s += blockDim.x)
      next_shifts[tg * S_next + s] = l + (h - l) * (double)(s + 1) / (double)(S_next + 1);
}

__device__ __forceinline__ double hash_unit(uint32_t x) {
  // integer hash (Wang-style mixing) to a value in (-1, 1)
  x = (x ^ 61u) ^ (x >> 16);
  x *= 9u;
  x = x ^ (x >> 4);
  x *= 0x27d4eb2du;
  x = x ^ (x >> 15);
  return ((double)x + 0.5) * (2.0 / 4294967296.0) - 1.0;
}

// Inverse iteration for target tg = blockIdx.x < k at the bracket midpoint.
__global__ __launch_bounds__(64) void k_invit(const double *__restrict__ Tb, int N, int kd,
                                              const double *__restrict__ brk, int k,
                                              double pivmin, double *Lscr, double *Dscr,
                                              double *X, int niter) {
  extern __shared__ double smem[];
  double *win = smem;
  double *chunk = win + (kd + 1) * (kd + 1);
  double *x = chunk + kChunk * (kd + 1);
  __shared__ double red[64];
  const int tg = blockIdx.x;
  const int t = threadIdx.x;
  const double theta = 0.5 * (brk[2 * tg] + brk[2 * tg + 1]);
  double *L = Lscr + (int64_t)tg * N * kd;
  double *D = Dscr + (int64_t)tg * N;
  ldl_sweep(Tb, N, kd, theta, pivmin, true, win, chunk, L, D);
  __threadfence();
  __syncthreads();
  for (int i = t; i < N; i += 64) x[i] = hash_unit((uint32_t)(i * 40503u + tg * 2654435761u + 7u));
  __syncthreads();
  for (int it = 0; it < niter; ++it) {
    // forward: unit lower L
    for (int kk = 0; kk < N; ++kk) {
      const double xk = x[kk];
      if (t < kd && kk + 1 + t < N) x[kk + 1 + t] -= L[(int64_t)kk * kd + t] * xk;
      __syncthreads();
    }
    for (int i = t; i < N; i += 64) x[i] /= D[i];
    __syncthreads();
    // backward: L^T
    for (int kk = N - 1; kk >= 0; --kk) {
      double p = (t < kd && kk + 1 + t < N) ? L[(int64_t)kk * kd + t] * x[kk + 1 + t] : 0.0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off, 64);
      if (t == 0) x[kk] -= p;
      __syncthreads();
    }
    // normalise
    double s = 0.0;
    for (int i = t; i < N; i += 64) s += x[i] * x[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (t == 0) red[0] = s;
    __syncthreads();
    const double inv = red[0] > 0.0 ? 1.0 / sqrt(red[0]) : 1.0;
    for (int i = t; i < N; i += 64) x[i] *= inv;
    __syncthreads();
  }
  for (int i = t; i < N; i += 64) X[(int64_t)i * k + tg] = x[i];
}

// Forward substitution L y = x (L unit lower, bandwidth KD, multipliers
// L[j*KD + r-1] = l_{j+r,j}), right-looking: once y_j is final it is removed
// from x_{j+1..j+KD}.  q holds x_j..x_{j+KD-1} in circular slots; the slot of
// x_{j0+s} is s % KD for the group of KD rows starting at j0.  All loads of a
// group (its multipliers, inverse pivots and entering x values) are issued
// before its arithmetic, so that one memory latency is exposed per group
// rather than per row.  Stores z_j = y_j / d_j in place of x_j.
// FULL: rows j0 .. j0 + 2 KD - 1 all exist, so no clamping or selects.
template <int KD, bool FULL>
__device__ __forceinline__ void fwd_group(const double *__restrict__ L,
                                          const double *__restrict__ Dinv, int ls, double *X,
                                          int ldx, int N, int j0, double (&q)[KD]) {
  // loads clamped to the last row (and zeroed after) so that they carry no
  // branch and can all be issued at once
  double Lg[KD][KD], dv[KD], xn[KD];
#pragma unroll
  for (int m = 0; m < KD; ++m) {
    const int j = j0 + m;
    const bool in = FULL || j < N, nin = FULL || j + KD < N;
    const int jc = FULL ? j : min(j, N - 1), jnc = FULL ? j + KD : min(j + KD, N - 1);
#pragma unroll
    for (int r = 0; r < KD; ++r) {
      const double v = L[((int64_t)jc * KD + r) * ls];
      Lg[m][r] = in ? v : 0.0;
    }
    const double dvv = Dinv[(int64_t)jc * ls];
    const double xv = X[(int64_t)jnc * ldx];
    dv[m] = in ? dvv : 0.0;
    xn[m] = nin ? xv : 0.0;
  }
#pragma unroll
  for (int m = 0; m < KD; ++m) {
    const double y = q[m];
#pragma unroll
    for (int r = 1; r < KD; ++r) q[(m + r) % KD] = fma(-Lg[m][r - 1], y, q[(m + r) % KD]);
    q[m] = fma(-Lg[m][KD - 1], y, xn[m]);
    if (FULL || j0 + m < N) X[(int64_t)(j0 + m) * ldx] = y * dv[m];
  }
}

// Back substitution L^T x = z, rows i = i0, i0 - 1, ..., i0 - KD + 1:
// x_i = z_i - sum_r l_{i+r,i} x_{i+r}.  wv holds x_{i+1..i+KD}; the slot of
// x_m is (m - i0 - 1) mod KD.  Loads of the group first, as above.
// Accumulates ||x||^2 in row order.
// FULL: rows i0 - KD + 1 .. i0 all exist.
template <int KD, bool FULL>
__device__ __forceinline__ void bwd_group(const double *__restrict__ L, int ls, double *X,
                                          int ldx, int i0, double (&wv)[KD], double &nrm2) {
  double Lg[KD][KD], zg[KD];
#pragma unroll
  for (int m = 0; m < KD; ++m) {
    const int i = i0 - m;
    const bool in = FULL || i >= 0;
    const int ic = FULL ? i : max(i, 0);
#pragma unroll
    for (int r = 0; r < KD; ++r) {
      const double v = L[((int64_t)ic * KD + r) * ls];
      Lg[m][r] = in ? v : 0.0;
    }
    const double zv = X[(int64_t)ic * ldx];
    zg[m] = in ? zv : 0.0;
  }
#pragma unroll
  for (int m = 0; m < KD; ++m) {
    if (!FULL && i0 - m < 0) break;
    double a0 = 0.0, a1 = 0.0;
#pragma unroll
    for (int r = 1; r <= KD; ++r) {
      const double v = wv[((r - m - 1) % KD + KD) % KD];
      if (r & 1) a0 = fma(Lg[m][r - 1], v, a0);
      else a1 = fma(Lg[m][r - 1], v, a1);
    }
    const double xi = zg[m] - (a0 + a1);
    wv[KD - 1 - m] = xi;
    X[(int64_t)(i0 - m) * ldx] = xi;
    nrm2 = fma(xi, xi, nrm2);
  }
}

// Inverse iteration for a compile-time bandwidth at the bracket midpoint
// theta of target tg < k: factor T - theta I with the register window,
// keeping the multipliers and inverse pivots, then run niter solves
// L D L^T x <- x from a hashed start, normalising after each.  Column tg of
// X (row-major N x k) receives the vector.  One lane per target, factors in
// global scratch (interleaved over the k lanes, so every load and store of the
// wave is contiguous), vectors in X or (XLDS) in dynamic LDS (N k doubles),
// copied to X at the end.  For matrices whose factors do not fit in LDS
// (k_invit_two).
template <int KD, bool XLDS>
__global__ __launch_bounds__(64) void k_invit_reg(const double *__restrict__ Tb, int N,
                                                  const double *__restrict__ brk, int k,
                                                  double pivmin, double *Lscr, double *Dscr,
                                                  double *X, int niter) {
  constexpr int W = KD + 1;
  extern __shared__ double smem_inv[];
  const int tg = (int)(blockIdx.x * 64 + threadIdx.x);
  if (tg >= k) return;
  const double theta = 0.5 * (brk[2 * tg] + brk[2 * tg + 1]);
  // l_{j+r,j} at L[(j*KD + r-1) * ls], 1/d_j at Dinv[j * ls], x_j at x[j * lx]
  double *L = Lscr + tg, *Dinv = Dscr + tg, *x = (XLDS ? smem_inv : X) + tg;
  const int ls = k, lx = k;
  double R[W * (W + 1) / 2];
  ldl_window_init<KD>(Tb, N, theta, R);
  int cnt = 0;
  ldl_sweep_reg<KD, true>(Tb, N, theta, pivmin, R, cnt, L, Dinv, ls);
  for (int i = 0; i < N; ++i)
    x[(int64_t)i * lx] = hash_unit((uint32_t)(i * 40503u + tg * 2654435761u + 7u));
  for (int it = 0; it < niter; ++it) {
    double q[KD];
#pragma unroll
    for (int r = 0; r < KD; ++r) q[r] = r < N ? x[(int64_t)r * lx] : 0.0;
    int j0 = 0;
#pragma unroll 1
    for (; j0 + 2 * KD <= N; j0 += KD) fwd_group<KD, true>(L, Dinv, ls, x, lx, N, j0, q);
#pragma unroll 1
    for (; j0 < N; j0 += KD) fwd_group<KD, false>(L, Dinv, ls, x, lx, N, j0, q);
    double wv[KD];
#pragma unroll
    for (int r = 0; r < KD; ++r) wv[r] = 0.0;
    double nrm2 = 0.0;
    int i0 = N - 1;
#pragma unroll 1
    for (; i0 - KD + 1 >= 0; i0 -= KD) bwd_group<KD, true>(L, ls, x, lx, i0, wv, nrm2);
#pragma unroll 1
    for (; i0 >= 0; i0 -= KD) bwd_group<KD, false>(L, ls, x, lx, i0, wv, nrm2);
    const double sc = nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 1.0;
    for (int i = 0; i < N; ++i) x[(int64_t)i * lx] *= sc;
  }
  if (XLDS)
    for (int i = 0; i < N; ++i) X[(int64_t)i * k + tg] = x[(int64_t)i * lx];
}

// Wave-wide sum by an xor butterfly; both partners of every step add the
// same two operands, so all 64 lanes end with identical bits.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The factorisation sweep of one end by one wave: lane l holds row l (window
// slot) of the symmetric (KD + 1) x (KD + 1) window, so a row's step is KD fused
// multiply-adds a lane instead of KD (KD + 1) / 2, with the pivot column's
// entries broadcast by v_readlane.  Multipliers l_{k+i,k} go to
// L[dir k KD + i - 1], 1/d to Dinv[dir k]; a tiny pivot keeps its sign.
template <int KD, int M>
__device__ __forceinline__ void lane_steps(const double *rows, int k0, double sigma,
                                           double pivmin, double (&R)[KD + 1], double *L,
                                           double *Dinv, int dir, int lane) {
  if constexpr (M <= KD) {
    constexpr int W = KD + 1;
    const int k = k0 + M;
    const double *rowp = rows + M * W;  // the band row that enters slot M
    double nv[W];
#pragma unroll
    for (int t = 1; t <= KD; ++t) nv[t] = rowp[t];
    const int rel = lane >= M ? lane - M : lane - M + W;  // row k + rel is in this lane
    const double mine = rowp[lane < W ? (rel == 0 ? 0 : W - rel) : 0];
    double d = lane_value(R[M], M);
    if (fabs(d) < pivmin) d = d > 0.0 ? pivmin : -pivmin;
    const double inv = newton_inv(d);
    const double w = R[M] * inv;
    if (k >= 0) {
      if (lane == M) Dinv[dir * k] = inv;
      else if (lane < W) L[dir * k * KD + rel - 1] = w;
    }
#pragma unroll
    for (int j = 0; j < W; ++j)
      if (j != M) R[j] = fma(-w, lane_value(R[M], j), R[j]);
    R[M] = mine - (lane == M ? sigma : 0.0);
    if (lane == M) {
#pragma unroll
      for (int j = 0; j < W; ++j)
        if (j != M) R[j] = nv[(M + W - j) % W];
    }
    lane_steps<KD, M + 1>(rows, k0, sigma, pivmin, R, L, Dinv, dir, lane);
  }
}

template <int KD>
__device__ __forceinline__ void lane_sweep(const double *__restrict__ Tb, int N, int m, int pad,
                                           double sigma, double pivmin, double (&R)[KD + 1],
                                           double *L, double *Dinv, int dir, double *buf,
                                           int lane) {
  constexpr int W = KD + 1;
#pragma unroll
  for (int j = 0; j < W; ++j) {
    const int a = max(lane, j) - pad, c = min(lane, j) - pad;
    R[j] = lane == j ? 1.0 : 0.0;  // rows before 0 couple to nothing
    if (lane < W && a >= 0 && a < N)
      R[j] = c >= 0 ? Tb[(int64_t)a * W + (a - c)] - (lane == j ? sigma : 0.0) : 0.0;
  }
  BandStage<KD> st(Tb, N, pad, buf, lane);
#pragma unroll 1
  for (int k0 = -pad; k0 < m;) {
    const double *rows = st.turn();
#pragma unroll 1
    for (int g = 0; g < BandStage<KD>::G && k0 < m; ++g, k0 += W)
      lane_steps<KD, 0>(rows + g * W * W, k0, sigma, pivmin, R, L, Dinv, dir, lane);
  }
}

// The middle block: lane l < KD holds its row l.
template <int KD>
__device__ __forceinline__ void lane_middle(int m1, double pivmin, double (&R)[KD + 1], double *L,
                                            double *Dinv, int lane) {
#pragma unroll
  for (int s = 0; s < KD; ++s) {
    double d = lane_value(R[s], s);
    if (fabs(d) < pivmin) d = d > 0.0 ? pivmin : -pivmin;
    const double inv = newton_inv(d);
    const double w = R[s] * inv;
    if (lane == s) Dinv[m1 + s] = inv;
    else if (lane > s && lane < KD) L[(m1 + s) * KD + lane - s - 1] = w;
#pragma unroll
    for (int j = s + 1; j < KD; ++j) R[j] = fma(-w, lane_value(R[s], j), R[j]);
  }
}

// Steps S .. KD of a forward group: q -= c y, y = row j0 + S's finished value,
// which the lane of its slot keeps before the entering row xn takes the slot.
template <int KD, int S>
__device__ __forceinline__ void fwd_steps(const double (&c)[KD], double xn, int lane, double &q,
                                          double &y) {
  if constexpr (S < KD) {
    const double ys = row_value<S>(q);
    y = lane == S ? ys : y;
    q = fma(-c[S], ys, lane == S ? xn : q);
    fwd_steps<KD, S + 1>(c, xn, lane, q, y);
  }
}

// Forward elimination over rows -pad .. m of one end (pad: (m + pad) % KD ==
// 0; rows before 0 are zero) by one wave, lane l < KD holding the pending row
// in circular slot l: z_j = y_j / d_j in place of x_j, j < m; q leaves holding
// rows m .. m + KD, what both ends have to say about them still to be merged.
// Row j is at L[dir j KD ..], Dinv[dir j], X[dir j].
template <int KD>
__device__ __forceinline__ void fwd_end(const double *L, const double *Dinv, double *X, int dir,
                                        int m, double &q, int lane) {
  const int pad = (KD - m % KD) % KD;
  const int l = lane < KD ? lane : KD - 1;
  q = l >= pad ? X[dir * (l - pad)] : 0.0;
  double c[KD];
  auto load = [&](int j0, double (&cc)[KD]) {
#pragma unroll
    for (int s = 0; s < KD; ++s) {
      const int r = l > s ? l - s : l - s + KD;  // 1 .. KD
      cc[s] = L[dir * max(j0 + s, 0) * KD + r - 1];
    }
  };
  if (-pad < m) load(-pad, c);
#pragma unroll 1
  for (int j0 = -pad; j0 < m; j0 += KD) {
    const double xn = X[dir * (j0 + KD + l)], dv = Dinv[dir * max(j0 + l, 0)];
    double nc[KD], y = 0.0;
    if (j0 + KD < m) load(j0 + KD, nc);
    fwd_steps<KD, 0>(c, xn, lane, q, y);
    if (lane < KD && j0 + lane >= 0) X[dir * (j0 + lane)] = y * dv;
#pragma unroll
    for (int s = 0; s < KD; ++s) c[s] = nc[s];
  }
}

// Steps S .. KD of a backward group: row i0 - S's value is z - acc of its slot
// (SOLVED: z), and c x goes to the pending rows' sums.
template <int KD, int S, bool SOLVED>
__device__ __forceinline__ void bwd_steps(const double (&c)[KD], double z, int lane, double &acc,
                                          double &xv) {
  if constexpr (S < KD) {
    const double x = row_value<S>(SOLVED ? z : z - acc);
    xv = lane == S ? x : xv;
    acc = fma(c[S], x, lane == S ? 0.0 : acc);
    bwd_steps<KD, S + 1, SOLVED>(c, z, lane, acc, xv);
  }
}

// Back substitution from the solved rows m .. m + KD outwards to row 0: lane l
// holds sum_r l_{i+r,i} x_{i+r} over the solved rows for the pending row i in
// its slot.
template <int KD>
__device__ __forceinline__ void bwd_end(const double *L, double *X, int dir, int m, double &nrm2,
                                        int lane) {
  const int l = lane < KD ? lane : KD - 1;
  double c[KD], nc[KD], acc = 0.0, xv = 0.0;
  auto load = [&](int i0, double (&cc)[KD]) {
#pragma unroll
    for (int s = 0; s < KD; ++s) {
      const int r = l > s ? l - s : l - s + KD, row = i0 - s - r;
      const double v = L[dir * max(row, 0) * KD + r - 1];
      cc[s] = row >= 0 ? v : 0.0;
    }
  };
  load(m + KD - 1, c);
  load(m - 1, nc);
  bwd_steps<KD, 0, true>(c, X[dir * (m + KD - 1 - l)], lane, acc, xv);
#pragma unroll 1
  for (int i0 = m - 1; i0 >= 0; i0 -= KD) {
#pragma unroll
    for (int s = 0; s < KD; ++s) c[s] = nc[s];
    const double z = X[dir * max(i0 - l, 0)];
    if (i0 - KD >= 0) load(i0 - KD, nc);
    bwd_steps<KD, 0, false>(c, z, lane, acc, xv);
    if (lane < KD && i0 - lane >= 0) {
      X[dir * (i0 - lane)] = xv;
      nrm2 = fma(xv, xv, nrm2);
    }
  }
}

// dynamic LDS of the inverse iteration: factors and vector, or vectors
constexpr size_t kInvLds = 158 * 1024;

// Doubles of LDS of k_invit_two without and with room for the stages of the
// factorisation's two sweeps.  Matrices too long for that have them where the
// vector goes later (with kd = 8, k = 32, N = 1920 left to k_invit_reg 12.3 ms,
// so 9.3); the others keep them apart, as the vector is then set up first (0.5 %).
template <int KD>
__host__ __device__ constexpr size_t invit_two_doubles(int N) {
  return (size_t)N * (KD + 2) + KD * KD + 2 * KD + 8;
}
template <int KD>
__host__ __device__ constexpr bool invit_two_apart(int N) {
  return (invit_two_doubles<KD>(N) + 2 * BandStage<KD>::E) * sizeof(double) <= kInvLds;
}

// Inverse iteration (as k_invit_reg) with one workgroup per target and the
// factors and vector in dynamic LDS (N (KD + 2) doubles and a little), so that
// the solves never wait on global memory, whose latency grows under the load
// of the recurrence running beside a check.  Two waves factor and solve from
// the two ends, KD + 1 lanes of each sharing the window (split_rows, with m2 =
// 0 for short matrices; N >= KD).  Workgroup k only writes the last target's
// bracket.  Bound by the chain of rows: measured at N = 1448, kd = 8, k = 10
// 289 us (772 with one lane over all rows), N = 352, kd = 4, k = 4 78 (133).
template <int KD>
__global__ __launch_bounds__(128) void k_invit_two(const double *__restrict__ T,
                                                   const double *__restrict__ Tr, int N, Bisect B,
                                                   int rounds, double pivmin, double *brk,
                                                   double *X, int niter) {
  extern __shared__ double smem_inv[];
  double *L = smem_inv, *Dinv = L + (size_t)N * KD, *x = Dinv + N;
  constexpr int E = BandStage<KD>::E;
  double *ex = x + N, *eq = ex + KD * KD, *en = eq + 2 * KD, *buf = invit_two_apart<KD>(N) ? en + 8 : x;
  const int t = threadIdx.x, lane = t & 63, up = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tg = blockIdx.x, k = B.k;
  double lo, hi;
  bracket<128>(B, rounds, tg, en, lo, hi);
  if (t == 0) {
    brk[2 * tg] = lo;
    brk[2 * tg + 1] = hi;
  }
  if (tg >= k) return;
  const double theta = 0.5 * (lo + hi);
  auto start_vector = [&](int first, int step) {
    for (int i = first; i < N; i += step)
      x[i] = hash_unit((uint32_t)(i * 40503u + tg * 2654435761u + 7u));
  };
  if (invit_two_apart<KD>(N)) start_vector(t, 128);
  const Split sp = split_rows(N, KD);
  const int dir = up ? -1 : 1, m = up ? sp.m2 : sp.m1, e0 = up ? N - 1 : 0;
  double *Le = L + (size_t)e0 * KD, *De = Dinv + e0, *xe = x + e0;
  {
    double R[KD + 1];
    lane_sweep<KD>(up ? Tr : T, N, m, up ? 0 : sp.pad, theta, pivmin, R, Le, De, dir,
                   buf + up * E, lane);
    if (up && lane < KD) {
#pragma unroll
      for (int j = 0; j < KD; ++j) ex[lane * KD + j] = R[j];
    }
    __syncthreads();
    if (up) {
      if (!invit_two_apart<KD>(N)) start_vector(lane, 64);
    } else {
      // both windows hold T - theta I of the middle, so it is taken out once
      if (lane < KD) {
#pragma unroll
        for (int j = 0; j < KD; ++j) {
          const int a = sp.m1 + max(lane, j), c = sp.m1 + min(lane, j);
          const double v = T[(int64_t)a * (KD + 1) + (a - c)] - (lane == j ? theta : 0.0);
          R[j] += ex[(KD - 1 - lane) * KD + KD - 1 - j] - v;
        }
      }
      lane_middle<KD>(sp.m1, pivmin, R, L, Dinv, lane);
    }
    __syncthreads();
  }
  for (int it = 0; it < niter; ++it) {
    double q, nrm2 = 0.0;
    fwd_end<KD>(Le, De, xe, dir, m, q, lane);
    if (up && lane < KD) eq[lane] = q;
    __syncthreads();
    if (!up) {  // the middle rows: merge, solve, hand out
      const int l = lane < KD ? lane : KD - 1;
      const double *Lm = L + (size_t)sp.m1 * KD;
      q += eq[KD - 1 - l] - x[sp.m1 + l];
#pragma unroll
      for (int s = 0; s < KD; ++s) {
        const double ys = lane_value(q, s);
        if (lane > s && lane < KD) q = fma(-Lm[s * KD + lane - s - 1], ys, q);
      }
      q *= Dinv[sp.m1 + l];
#pragma unroll
      for (int u = 0; u < KD; ++u) {
        const int s = KD - 1 - u;
        const double xs = lane_value(q, s);
        if (lane < s) q = fma(-Lm[lane * KD + s - lane - 1], xs, q);
      }
      if (lane < KD) {
        x[sp.m1 + lane] = q;
        nrm2 = q * q;
      }
    }
    __syncthreads();
    bwd_end<KD>(Le, xe, dir, m, nrm2, lane);
    nrm2 = wave_sum(nrm2);
    if (lane == 0) en[up] = nrm2;
    __syncthreads();
    const double n2 = en[0] + en[1];
    const double sc = n2 > 0.0 ? 1.0 / sqrt(n2) : 1.0;
    for (int i = t; i < N; i += 128) x[i] *= sc;
    __syncthreads();
  }
  for (int i = t; i < N; i += 128) X[(int64_t)i * k + tg] = x[i];
}

__device__ double wg_sum(double v, double *red) {
  // sum over a 256-thread workgroup (fixed order)
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

__device__ __forceinline__ double band_at(const double *Tb, int kd, int i, int j) {
  const int d = i - j;
  if (d >= 0) return d <= kd ? Tb[(int64_t)i * (kd + 1) + d] : 0.0;
  return -d <= kd ? Tb[(int64_t)j * (kd + 1) - d] : 0.0;
}

// Residual estimates rho_c = ||Bj S[N-b:N, c]|| (Bj = coupling block to the
// next Lanczos block, or null) and the results: res: theta[0..k), rho[k..2k),
// res[2k] = ||T||_est = max(|theta_0|, |top|), res[2k+1] = largest eigenvalue.
__device__ void write_results(int t, int N, int k, const double *__restrict__ Bj, int b,
                              const double *S, const double *lam, const double *brk,
                              double *res) {
  if (t < k) {
    double rho = 0.0;
    if (Bj) {
      for (int r = 0; r < b; ++r) {
        double v = 0.0;
        for (int m = 0; m < b; ++m) v += Bj[r * b + m] * S[(int64_t)(N - b + m) * k + t];
        rho += v * v;
      }
    }
    res[t] = lam[t];
    res[k + t] = sqrt(rho);
  }
  if (t == 0) {
    const double top = 0.5 * (brk[2 * k] + brk[2 * k + 1]);
    res[2 * k] = fmax(fabs(lam[0]), fabs(top));
    res[2 * k + 1] = top;
  }
}

// Rayleigh-Ritz on span(X): X <- orthonormal basis (modified Gram-Schmidt,
// twice), K = X^T T X, K = Y diag(theta) Y^T, S = X Y.  K, Y: kMaxBlock^2
// doubles of LDS each; lam: kMaxBlock; cs: 4; red: one per thread.
// Inlined into k_rr, so that its LDS is addressed as LDS (as a call, through flat
// addresses, k_rr took 6.69 ms at N = 1136, kd = 16, k = 32; inlined 6.11).
__device__ __forceinline__ void rr_gram_schmidt(const double *__restrict__ Tb, int N, int kd,
                                                int k, double *X, double *TX,
                                                const double *__restrict__ Bj, int b,
                                                const double *__restrict__ brk, double *S,
                                                double *res, double *K, double *Y, double *lam,
                                                double *cs, double *red) {
  const int t = threadIdx.x;
  for (int c = 0; c < k; ++c) {
    for (int attempt = 0; attempt < 2; ++attempt) {
      for (int pass = 0; pass < 2; ++pass) {
        for (int a = 0; a < c; ++a) {
          double p = 0.0;
          for (int i = t; i < N; i += blockDim.x) p += X[(int64_t)i * k + a] * X[(int64_t)i * k + c];
          const double dot = wg_sum(p, red);
          for (int i = t; i < N; i += blockDim.x) X[(int64_t)i * k + c] -= dot * X[(int64_t)i * k + a];
          __syncthreads();
        }
      }
      double p = 0.0;
      for (int i = t; i < N; i += blockDim.x) p += X[(int64_t)i * k + c] * X[(int64_t)i * k + c];
      const double nrm = sqrt(wg_sum(p, red));
      if (nrm > 1e-8) {
        for (int i = t; i < N; i += blockDim.x) X[(int64_t)i * k + c] /= nrm;
        __syncthreads();
        break;
      }
      // the vector collapsed onto earlier ones: restart it from a fresh direction
      for (int i = t; i < N; i += blockDim.x)
        X[(int64_t)i * k + c] = hash_unit((uint32_t)(i * 2246822519u + c * 3266489917u + 11u));
      __syncthreads();
    }
  }
  __threadfence();
  __syncthreads();
  for (int64_t e = t; e < (int64_t)N * k; e += blockDim.x) {
    const int i = (int)(e / k), c = (int)(e % k);
    double s = 0.0;
    const int j0 = max(0, i - kd), j1 = min(N - 1, i + kd);
    for (int j = j0; j <= j1; ++j) s += band_at(Tb, kd, i, j) * X[(int64_t)j * k + c];
    TX[e] = s;
  }
  __threadfence();
  __syncthreads();
  for (int e = t; e < k * k; e += blockDim.x) {
    const int a = e / k, c = e % k;
    double s = 0.0;
    for (int i = 0; i < N; ++i) s += X[(int64_t)i * k + a] * TX[(int64_t)i * k + c];
    K[e] = s;
  }
  __syncthreads();
  for (int e = t; e < k * k; e += blockDim.x) {
    const int a = e / k, c = e % k;
    if (a < c) {
      const double m = 0.5 * (K[a * k + c] + K[c * k + a]);
      K[a * k + c] = m;
      K[c * k + a] = m;
    }
  }
  __syncthreads();
  wg_jacobi_eig(K, Y, lam, k, cs);
  for (int64_t e = t; e < (int64_t)N * k; e += blockDim.x) {
    const int i = (int)(e / k), c = (int)(e % k);
    double s = 0.0;
    for (int a = 0; a < k; ++a) s += X[(int64_t)i * k + a] * Y[a * k + c];
    S[e] = s;
  }
  __threadfence();
  __syncthreads();
  write_results(t, N, k, Bj, b, S, lam, brk, res);
}

__global__ __launch_bounds__(256) void k_rr(const double *__restrict__ Tb, int N, int kd, int k,
                                            double *X, double *TX,
                                            const double *__restrict__ Bj, int b,
                                            const double *__restrict__ brk, double *S,
                                            double *res) {
  __shared__ double K[kMaxBlock * kMaxBlock], Y[kMaxBlock * kMaxBlock];
  __shared__ double lam[kMaxBlock], cs[4], red[256];
  rr_gram_schmidt(Tb, N, kd, k, X, TX, Bj, b, brk, S, res, K, Y, lam, cs, red);
}

// The same for k_rr_fast, which rarely needs it and would spill more registers
// with it inlined.
__device__ __noinline__ void rr_gram_schmidt_call(const double *Tb, int N, int kd, int k,
                                                  double *X, double *TX, const double *Bj, int b,
                                                  const double *brk, double *S, double *res,
                                                  double *K, double *Y, double *lam, double *cs,
                                                  double *red) {
  rr_gram_schmidt(Tb, N, kd, k, X, TX, Bj, b, brk, S, res, K, Y, lam, cs, red);
}

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kRrMax = kWaveMat;  // pairs of k_rr_fast: one 16 x 16 matrix-core tile
constexpr int kRrWaves = 16;
constexpr int kRrStage = 4 * (2 * kMaxBlock + 1) + 4;  // doubles a wave stages (4 band rows)
static_assert(kRrStage >= 256, "a wave's 16 x 16 partial product fits its stage");

// Jacobi by one wave on the symmetric n x n matrix A (16-wide rows in LDS, n
// <= 16): each step rotates n / 2 disjoint pairs of a round-robin schedule.
// lam ascending, Y's columns the matching eigenvectors.
__device__ void wave_jacobi(double *A, double *V, double *Y, double *lam, int n, double *cs,
                            int *pq, int lane) {
  const int ne = (n + 1) & ~1, half = ne / 2;
  const int i = lane & 15, u0 = lane >> 4;
#pragma unroll
  for (int e = lane; e < kRrMax * kRrMax; e += 64) V[e] = (e >> 4) == (e & 15) ? 1.0 : 0.0;
  wave_fence();
  for (int sweep = 0; sweep < 60 && n > 1; ++sweep) {
    double off = 0.0, dia = 0.0;
#pragma unroll
    for (int r = u0; r < kRrMax; r += 4) {
      const double v = r < n && i < n ? A[r * kRrMax + i] : 0.0;
      if (r == i) dia = fma(v, v, dia);
      else off = fma(v, v, off);
    }
    off = wave_sum(off);
    dia = wave_sum(dia);
    if (off <= 1e-32 * dia || off < 1e-300) break;
    for (int step = 0; step < ne - 1; ++step) {
      // pair u: players (step + u, step - u) of a circle of ne - 1; pair 0: step and the last
      if (lane < half) {
        int p = step + lane, q = step - lane;
        p -= p >= ne - 1 ? ne - 1 : 0;
        q += q < 0 ? ne - 1 : 0;
        if (lane == 0) q = ne - 1;
        const int lo = min(p, q), hi = max(p, q);
        double c = 1.0, s = 0.0;
        if (hi < n) {
          const double apq = A[lo * kRrMax + hi], app = A[lo * kRrMax + lo],
                       aqq = A[hi * kRrMax + hi];
          if (fabs(apq) > 1e-300 && apq * apq > 1e-36 * fabs(app * aqq)) {
            const double tau = (aqq - app) / (2.0 * apq);
            const double w = fma(tau, tau, 1.0);
            // |tau| past 1e150: t = 1 / (2 tau) to rounding
            const double tt = fabs(tau) > 1e150 ? 0.5 / tau
                                                : copysign(newton_inv(fabs(tau) + w * newton_rsqrt(w)), tau);
            c = newton_rsqrt(fma(tt, tt, 1.0));
            s = tt * c;
          }
        }
        cs[2 * lane] = c;
        cs[2 * lane + 1] = s;
        pq[2 * lane] = lo;
        pq[2 * lane + 1] = hi;
      }
      wave_fence();
#pragma unroll
      for (int u = u0; u < kRrMax / 2; u += 4) {  // columns of A and V
        if (u < half && i < n && cs[2 * u + 1] != 0.0) {
          const double c = cs[2 * u], s = cs[2 * u + 1];
          const int p = pq[2 * u], q = pq[2 * u + 1];
          const double ap = A[i * kRrMax + p], aq = A[i * kRrMax + q];
          const double vp = V[i * kRrMax + p], vq = V[i * kRrMax + q];
          A[i * kRrMax + p] = c * ap - s * aq;
          A[i * kRrMax + q] = s * ap + c * aq;
          V[i * kRrMax + p] = c * vp - s * vq;
          V[i * kRrMax + q] = s * vp + c * vq;
        }
      }
      wave_fence();
#pragma unroll
      for (int u = u0; u < kRrMax / 2; u += 4) {  // rows of A
        if (u < half && i < n && cs[2 * u + 1] != 0.0) {
          const double c = cs[2 * u], s = cs[2 * u + 1];
          const int p = pq[2 * u], q = pq[2 * u + 1];
          const double ap = A[p * kRrMax + i], aq = A[q * kRrMax + i];
          A[p * kRrMax + i] = c * ap - s * aq;
          A[q * kRrMax + i] = s * ap + c * aq;
        }
      }
      wave_fence();
    }
  }
  if (lane < n) {
    const double l = A[lane * kRrMax + lane];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double o = A[j * kRrMax + j];
      rank += o < l || (o == l && j < lane) ? 1 : 0;
    }
    lam[rank] = l;
    for (int j = 0; j < n; ++j) Y[j * kRrMax + rank] = V[j * kRrMax + lane];
  }
  wave_fence();
}

// Rayleigh-Ritz for k <= 16 by one workgroup (the same step as k_rr):
//   Q = X R^{-1}, twice: Cholesky QR of the inverse-iteration vectors;
//   K = Q^T T Q (symmetrised), K = Y diag(theta) Y^T (Jacobi);
//   S = Q Y and the residual estimates.
// Both k x k products run on FP64 matrix cores: a wave's four rows of Q are at
// once the A and the B operand of v_mfma_f64_16x16x4.  A Cholesky pivot below
// 1e-12 of its diagonal entry (columns nearly dependent) redoes the step with
// Gram-Schmidt and restarts from X, which is left unchanged until then.  SQ:
// Q is kept in dynamic LDS (N k doubles); otherwise in the global scratch Qg.
// Bound by latency (one workgroup).  Measured at N = 1448, kd = 8, k = 10: 89
// us (390 us on one wave with the sums in vector registers), N = 352, kd = 4,
// k = 4 27 (60).
template <bool SQ>
__global__ __launch_bounds__(64 * kRrWaves) void k_rr_fast(
    const double *__restrict__ Tb, int N, int kd, int k, double *X, double *Qg,
    const double *__restrict__ Bj, int b, const double *__restrict__ brk, double *S, double *res) {
  extern __shared__ double sQ[];
  __shared__ double stage[kRrWaves * kRrStage];
  __shared__ double M0[kRrMax * kRrMax], M1[kRrMax * kRrMax], M2[kRrMax * kRrMax];
  __shared__ double lam[kMaxBlock], cs[kRrMax];
  __shared__ int sbad, pq[kRrMax];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, lr = lane & 15, lk = lane >> 4;
  constexpr int T = 64 * kRrWaves;
  double *Q = SQ ? sQ : Qg;
  double *st = stage + wave * kRrStage;
#pragma unroll 8
  for (int e = t; e < N * k; e += T) Q[e] = X[e];
  __syncthreads();
  // M0 = sum of the waves' 16 x 16 products
  auto collect = [&](d4 acc) {
#pragma unroll
    for (int q = 0; q < 4; ++q) st[(lk + 4 * q) * kRrMax + lr] = acc[q];
    __syncthreads();
    if (t < kRrMax * kRrMax) {
      double s = 0.0;
      for (int w = 0; w < kRrWaves; ++w) s += stage[w * kRrStage + t];
      M0[t] = s;
    }
    __syncthreads();
  };
  // out = Q M (M 16 x 16, zero past k), 16 rows a wave and step; out may be Q
  auto times = [&](const double *M, double *out) {
    double b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = M[(lk + 4 * q) * kRrMax + lr];
    for (int r0 = 16 * wave; r0 < N; r0 += 16 * kRrWaves) {
      double a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = lk + 4 * q;
        a[q] = r0 + lr < N && c < k ? Q[(int64_t)(r0 + lr) * k + c] : 0.0;
      }
      d4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], acc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = r0 + lk + 4 * q;
        if (row < N && lr < k) out[(int64_t)row * k + lr] = acc[q];
      }
    }
  };
  for (int pass = 0; pass < 2; ++pass) {
    d4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int r0 = 4 * wave; r0 < N; r0 += 4 * kRrWaves) {
      const int row = r0 + lk;
      const double v = row < N && lr < k ? Q[(int64_t)row * k + lr] : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, acc, 0, 0, 0);
    }
    collect(acc);
    if (wave == 0) {
      // a squared pivot below 1e-12 of its diagonal entry: nearly dependent
      double r[kWaveMat], x[kWaveMat], pmin;
      const int bad = wave_chol(M0, kRrMax, k, 1e-12, 0.0, lane, r, x, pmin);
      if (lane < kRrMax) {
#pragma unroll
        for (int a = 0; a < kRrMax; ++a) M1[a * kRrMax + lane] = lane < k ? x[a] : 0.0;
      }
      if (lane == 0) sbad = bad;
    }
    __syncthreads();
    if (sbad) {
      double *K = stage, *Y = stage + kMaxBlock * kMaxBlock;
      __syncthreads();
      rr_gram_schmidt_call(Tb, N, kd, k, X, Qg, Bj, b, brk, S, res, K, Y, lam, cs,
                           Y + kMaxBlock * kMaxBlock);
      return;
    }
    times(M1, Q);
    __syncthreads();
  }
  // K = Q^T (T Q), four rows of T at a time: their band entries (offsets -kd ..
  // kd) are staged by the wave, the next four rows' loaded meanwhile
  {
    const int D = 2 * kd + 1, per = 4 * D;
    constexpr int U = (4 * (2 * kMaxBlock + 1) + 63) / 64;
    double nx[U];
    int di[U], dj[U];  // row and column of the lane's entries, from the first row
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = lane + 64 * u;
      di[u] = e < per ? e / D : N;
      dj[u] = di[u] + e % D - kd;
    }
    auto load = [&](int r0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = r0 + di[u], j = r0 + dj[u];
        nx[u] = 0.0;
        if (64 * u < per && i < N && j >= 0 && j < N) nx[u] = band_at(Tb, kd, i, j);
      }
    };
    d4 acc{0.0, 0.0, 0.0, 0.0};
    load(4 * wave);
    for (int r0 = 4 * wave; r0 < N; r0 += 4 * kRrWaves) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (64 * u < per && lane + 64 * u < per) st[lane + 64 * u] = nx[u];
      wave_fence();
      load(r0 + 4 * kRrWaves);
      const int row = r0 + lk;
      const bool in = row < N && lr < k;
      double a0 = 0.0, a1 = 0.0;
      for (int o = 0; o < D; o += 2) {
        const int j0 = min(max(row + o - kd, 0), N - 1), j1 = min(max(row + o + 1 - kd, 0), N - 1);
        const double t0 = st[lk * D + o], t1 = o + 1 < D ? st[lk * D + o + 1] : 0.0;
        const int c = lr < k ? lr : 0;
        a0 = fma(t0, Q[(int64_t)j0 * k + c], a0);
        a1 = fma(t1, Q[(int64_t)j1 * k + c], a1);
      }
      const double tq = in ? a0 + a1 : 0.0;
      const double v = in ? Q[(int64_t)row * k + lr] : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v, tq, acc, 0, 0, 0);
      wave_fence();
    }
    __syncthreads();  // the stages are read
    collect(acc);
  }
  if (t < kRrMax * kRrMax) {
    const int i = t / kRrMax, j = t % kRrMax;
    M1[t] = 0.5 * (M0[i * kRrMax + j] + M0[j * kRrMax + i]);
  }
  __syncthreads();
  if (t < kRrMax * kRrMax) M0[t] = 0.0;
  __syncthreads();
  if (wave == 0) wave_jacobi(M1, M2, M0, lam, k, cs, pq, lane);
  __syncthreads();
  times(M0, S);
  __threadfence();
  __syncthreads();
  write_results(t, N, k, Bj, b, S, lam, brk, res);
}

// Shifts.  Register-window bandwidths: 8192 shifts per round (128 workgroups
// of two waves, a quarter of the SIMDs, so that an overlapped check leaves most
// of the chip to the recurrence); other bandwidths (one workgroup per shift):
// 2048.  The first round spreads the shifts over the Gershgorin interval,
// later rounds give each target its own run of shifts / (k + 1), rounded down
// to whole waves.  Rounds continue until every bracket has narrowed by at least
// kNarrow (four rounds for k = 10 on the register path: 8193 * 705^3 ~
// 2.9e12).  Inverse iteration and Rayleigh-Ritz then refine the pairs.
constexpr int kShiftsReg = 8192;
constexpr int kShiftsLds = 2048;
constexpr double kNarrow = 2e12;
constexpr int kInvIters = 2;
constexpr double kPivmin = 1e-290, kInvPivmin = 1e-200;
// dynamic LDS of the Rayleigh-Ritz basis beside its 42 KB of static LDS
constexpr size_t kRrLds = 118 * 1024;

bool reg_bandwidth(int kd) {
  return kd == 1 || kd == 2 || kd == 4 || kd == 8 || kd == 10 || kd == 16;
}
int shifts_per_target(int nsh, int NT) { return std::max(64, (nsh / NT) / 64 * 64); }

// Lets a kernel use up to `bytes` of dynamic LDS on the current device.  Each
// device has its own limit, so it is set before each launch.
template <typename K>
void allow_lds(K *kernel, size_t bytes) {
  BBL_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
}

// LDS bytes and launch of k_invit: a 64-lane workgroup a target.
size_t invit_bytes(int N, int kd) {
  return (size_t)((kd + 1) * (kd + 1) + kChunk * (kd + 1) + N) * sizeof(double);
}
constexpr size_t kInvitLds = 150 * 1024;
void invit_launch(const double *band, int N, int kd, const double *brk, int k, double *Lscr,
                  double *Dscr, double *X, hipStream_t s) {
  allow_lds(&k_invit, kInvitLds);
  hipLaunchKernelGGL(k_invit, dim3(k), dim3(64), invit_bytes(N, kd), s, band, N, kd, brk, k,
                     kInvPivmin, Lscr, Dscr, X, kInvIters);
  check_launch("k_invit");
}

template <int KD>
void invit_reg_launch(const double *band, const double *rev, int N, const Bisect &B, int rounds,
                      double *brk, double *Lscr, double *Dscr, double *X, hipStream_t s) {
  const int k = B.k;
  const size_t two =
      (invit_two_doubles<KD>(N) + (invit_two_apart<KD>(N) ? 2 * BandStage<KD>::E : 0)) * sizeof(double);
  if (N >= KD && two <= kInvLds) {
    allow_lds(&k_invit_two<KD>, kInvLds);
    hipLaunchKernelGGL(k_invit_two<KD>, dim3(k + 1), dim3(128), two, s, band, rev, N, B, rounds,
                       kInvPivmin, brk, X, kInvIters);
    check_launch("k_invit_two");
    return;
  }
  hipLaunchKernelGGL(k_final_brackets, dim3(k + 1), dim3(128), 0, s, B, rounds, brk);
  check_launch("k_final_brackets");
  // At 16 a lane's window and block of multipliers overflow the registers, and a
  // workgroup a target is faster (us, k = 4 / 32: N = 1136 2130 / 2150 against
  // 4260 / 6000, N = 3200 6030 / 6150 against 11820 / 21070).
  if (KD == 16 && invit_bytes(N, KD) <= kInvitLds) {
    invit_launch(band, N, KD, brk, k, Lscr, Dscr, X, s);
    return;
  }
  const size_t xbytes = (size_t)N * k * sizeof(double);
  if (xbytes <= kInvLds) {
    allow_lds(&k_invit_reg<KD, true>, kInvLds);
    hipLaunchKernelGGL((k_invit_reg<KD, true>), dim3(1), dim3(64), xbytes, s, band, N, brk, k,
                       kInvPivmin, Lscr, Dscr, X, kInvIters);
  } else {
    hipLaunchKernelGGL((k_invit_reg<KD, false>), dim3(1), dim3(64), 0, s, band, N, brk, k,
                       kInvPivmin, Lscr, Dscr, X, kInvIters);
  }
  check_launch("k_invit_reg");
}

}  // namespace

BandEigLayout band_eig_layout(int N, int kd, int k) {
  BandEigLayout L;
  const int NT = k + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align_up(bytes);
    return o;
  };
  const int nshift = std::max(kShiftsReg, NT * 64);
  L.gersh = take(2 * sizeof(double));
  L.shifts_a = take(nshift * sizeof(double));
  L.shifts_b = take(nshift * sizeof(double));
  L.counts = take(nshift * sizeof(int));
  L.brk = take(2 * NT * sizeof(double));
  L.Lscr = take((size_t)k * N * std::max(kd, 1) * sizeof(double));
  L.Dscr = take((size_t)k * N * sizeof(double));
  L.rev = L.Lscr;
  off = std::max(off, L.rev + align_up((size_t)N * (kd + 1) * sizeof(double)));
  L.X = take((size_t)N * k * sizeof(double));
  L.TX = take((size_t)N * k * sizeof(double));
  L.bytes = off;
  return L;
}

void band_eigensolve(const double *band, int N, int kd, int k, void *ws, const BandEigLayout &L,
                     const double *Bj, int b, double *S, double *res, hipStream_t s) {
  BBL_REQUIRE(N >= 1 && k >= 1 && k <= N && k <= kMaxBlock && kd >= 0 && kd <= kMaxBlock,
              "band eigensolve: bad sizes");
  char *base = static_cast<char *>(ws);
  double *gersh = reinterpret_cast<double *>(base + L.gersh);
  double *sh_a = reinterpret_cast<double *>(base + L.shifts_a);
  double *sh_b = reinterpret_cast<double *>(base + L.shifts_b);
  int *counts = reinterpret_cast<int *>(base + L.counts);
  double *brk = reinterpret_cast<double *>(base + L.brk);
  double *Lscr = reinterpret_cast<double *>(base + L.Lscr);
  double *Dscr = reinterpret_cast<double *>(base + L.Dscr);
  double *X = reinterpret_cast<double *>(base + L.X);
  double *TX = reinterpret_cast<double *>(base + L.TX);
  BBL_REQUIRE(kd >= 1, "band eigensolve: kd must be >= 1");
  const int NT = k + 1;
  const bool regk = reg_bandwidth(kd);
  const int nsh = regk ? kShiftsReg : kShiftsLds;
  const int SP = shifts_per_target(nsh, NT);
  int rounds = 1;
  for (double f = nsh + 1.0; f < kNarrow; f *= SP + 1.0) ++rounds;
  if (regk) {
    // the counts and the rounds' brackets take the place of the shift lists
    double *rev = reinterpret_cast<double *>(base + L.rev);
    const int ng = std::min(kGershMax, (N + 127) / 128);
    double *bounds = sh_a + kShiftsReg / 2;  // past the brackets
    Bisect B{bounds, ng, sh_a, {counts, reinterpret_cast<int *>(sh_b)}, nsh, SP, k, N};
    hipLaunchKernelGGL(k_gersh, dim3(ng), dim3(128), 0, s, band, N, kd, bounds, rev);
    check_launch("k_gersh");
    for (int r = 0; r < rounds; ++r) sturm_reg(band, rev, N, kd, B, r, kPivmin, s);
    switch (kd) {
      case 1: invit_reg_launch<1>(band, rev, N, B, rounds, brk, Lscr, Dscr, X, s); break;
      case 2: invit_reg_launch<2>(band, rev, N, B, rounds, brk, Lscr, Dscr, X, s); break;
      case 4: invit_reg_launch<4>(band, rev, N, B, rounds, brk, Lscr, Dscr, X, s); break;
      case 8: invit_reg_launch<8>(band, rev, N, B, rounds, brk, Lscr, Dscr, X, s); break;
      case 10: invit_reg_launch<10>(band, rev, N, B, rounds, brk, Lscr, Dscr, X, s); break;
      default: invit_reg_launch<16>(band, rev, N, B, rounds, brk, Lscr, Dscr, X, s); break;
    }
  } else {
    hipLaunchKernelGGL(k_gersh, dim3(1), dim3(128), 0, s, band, N, kd, gersh, (double *)nullptr);
    hipLaunchKernelGGL(k_bisect_init, dim3(16), dim3(256), 0, s, gersh, nsh, sh_a, brk, NT);
    check_launch("k_bisect_init");
    const size_t smem_s = (size_t)((kd + 1) * (kd + 1) + kChunk * (kd + 1)) * sizeof(double);
    for (int r = 0; r < rounds; ++r) {
      const int count = r == 0 ? nsh : NT * SP;
      hipLaunchKernelGGL(k_sturm, dim3(count), dim3(64), smem_s, s, band, N, kd, sh_a, counts,
                         kPivmin);
      check_launch("k_sturm");
      hipLaunchKernelGGL(k_bisect_update, dim3(NT), dim3(256), 0, s, r == 0 ? 1 : 0, sh_a, counts,
                         r == 0 ? nsh : SP, N, k, brk, SP, r == rounds - 1 ? nullptr : sh_b);
      check_launch("k_bisect_update");
      std::swap(sh_a, sh_b);
    }
    BBL_REQUIRE(invit_bytes(N, kd) <= kInvitLds,
                "band eigensolve: band matrix too large for LDS staging");
    invit_launch(band, N, kd, brk, k, Lscr, Dscr, X, s);
  }
  // Rayleigh-Ritz: Cholesky QR on matrix cores up to 16 pairs, else Gram-Schmidt
  if (k <= kRrMax) {
    const size_t qbytes = (size_t)N * k * sizeof(double);
    if (qbytes <= kRrLds) {
      allow_lds(&k_rr_fast<true>, kRrLds);
      hipLaunchKernelGGL(k_rr_fast<true>, dim3(1), dim3(64 * kRrWaves), qbytes, s, band, N, kd, k,
                         X, TX, Bj, b, brk, S, res);
    } else {
      hipLaunchKernelGGL(k_rr_fast<false>, dim3(1), dim3(64 * kRrWaves), 0, s, band, N, kd, k, X,
                         TX, Bj, b, brk, S, res);
    }
    check_launch("k_rr_fast");
  } else {
    hipLaunchKernelGGL(k_rr, dim3(1), dim3(256), 0, s, band, N, kd, k, X, TX, Bj, b, brk, S, res);
    check_launch("k_rr");
  }
}

}  // namespace bbl
