// Discrete Zak transform of received time-domain frames (Sec. III-A, Eq. zak) and its
// inverse (Eq. iZak): the batched unitary DFTs of Sec. IV-A (Eq. zak_gemm) along the slots.
//
// For a frame of M delay x N Doppler bins, the time-domain samples y[i M + k] (slot i,
// delay k) form an N x M matrix In[i][k] in memory order, and the DD frame in vector order
// q = l M + k is the N x M matrix Out[l][k] = sum_i F[l][i] In[i][k] with the unitary kernel
// F[l][i] = e^{-j 2 pi l i / N} / sqrt(N) (Eq. zak as written; the printed kernel matrix of
// Eq. zak_exp differs from it by the factor sqrt(N) (-1)^l, and the transform is kept
// unitary so that DD noise equals time-domain noise).  The inverse takes conj(F)^T, i.e.
// the same product with the opposite twiddle sign.
//
// k_dzt runs the dense contraction on MFMA (any N): FP32 inputs (v_mfma_f32_16x16x4_f32),
// complex products as four real products, FP32 accumulation.  One wave computes a 16 x 64
// block of Out (four 16 x 16 tiles side by side in k): per step of 4 slots i, the A operand
// F[l][i] comes from a twiddle table in LDS (index l i mod N, exact), the B operand In[i][k]
// straight from memory (one complex per lane per tile), and 16 MFMAs (4 tiles x 4 real
// products) accumulate.  A workgroup is 4 waves covering 16 x 256 of one frame.  Rows l >= N
// and columns k >= M are computed on zero-padded operands and not stored; slots i >= N
// contribute zero.  8 N operations per element: near the memory's time for small N only.
//
// k_dzt_fft runs the same sums as two or three passes of short DFTs (N = r0 r1 [r2], each
// <= 16) over column strips held in LDS: one read and one write of the frame whatever N is,
// bound by memory.  Against k_dzt (time of one transform, bytes read and written per second):
//   64 frames of 1024 x 256   364 -> 46 us (5.8 TB/s)   32 of 1024 x 512    715 -> 61 us
//   128 of 1024 x 128         189 -> 45 us              16 of 1024 x 1024  1419 -> 82 us
//   60 of 1024 x 243          327 -> 66 us              16 of 512 x 2048   2817 -> 133 us
//   1 of 64 x 128            17.6 -> 8.9 us (a launch)
#include <hip/hip_runtime.h>

#include <math.h>

#include "otfs_internal.h"

namespace otfs {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kDztThreads = 256;                 // 4 waves
constexpr int kDztRows = 16;                     // l per workgroup
constexpr int kDztCols = 256;                    // k per workgroup (64 per wave)
constexpr int kDztFftThreads = 512;
constexpr int kDztFftMinN = 65;                  // rule of launch_dzt
constexpr int kDztFftMaxN = 2048;
constexpr int kDztFftLdsBytes = 150 * 1024;
static_assert((1 + 2 * 4) * kDztFftMaxN * (int)sizeof(float2) <= kDztFftLdsBytes, "strips of 4 columns fit");

__global__ __launch_bounds__(kDztThreads) void k_dzt(int M, int N, int nframes, float sign,
                                                     const float2* __restrict__ in,
                                                     float2* __restrict__ out) {
  extern __shared__ float2 tw[];                 // tw[m] = e^{sign j 2 pi m / N} / sqrt(N)
  const int nlb = (N + kDztRows - 1) / kDztRows;
  const int nkb = (M + kDztCols - 1) / kDztCols;
  const int64_t b = blockIdx.x;
  const int f = (int)(b / ((int64_t)nlb * nkb));
  const int rem = (int)(b - (int64_t)f * nlb * nkb);
  const int l0 = (rem / nkb) * kDztRows;
  const int kb0 = (rem % nkb) * kDztCols;
  if (f >= nframes) return;
  const double scale = 1.0 / sqrt((double)N);
  for (int m = threadIdx.x; m < N; m += kDztThreads) {
    double s, c;
    sincospi(2.0 * (double)m / (double)N, &s, &c);
    tw[m] = make_float2((float)(c * scale), (float)(sign * s * scale));
  }
  __syncthreads();
  const int64_t E = (int64_t)M * N;
  const float2* src = in + (int64_t)f * E;
  float2* dst = out + (int64_t)f * E;
  const int lane = (int)threadIdx.x & 63;
  const int wave = (int)threadIdx.x >> 6;
  const int k0 = kb0 + wave * 64;                // this wave's 64 columns
  const int am = lane & 15, ak = lane >> 4;      // A[m][kk], B[kk][n]: lane = m + 16 kk
  const int la = l0 + am;                        // row of this lane's A element
  f32x4 re[4], im[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    re[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    im[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // twiddle index (la * i) mod N for i = i0 + ak, advanced by 4 la per step
  const int64_t lan = la < N ? la : 0;
  int64_t idx = (lan * ak) % N;
  const int64_t step = (4 * lan) % N;
  for (int i0 = 0; i0 < N; i0 += 4) {
    const int i = i0 + ak;
    float2 a = make_float2(0.f, 0.f);
    if (la < N && i < N) a = tw[idx];
    idx += step;
    if (idx >= N) idx -= N;
    float2 v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = k0 + t * 16 + am;
      v[t] = (i < N && k < M) ? src[(int64_t)i * M + k] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      // (a.x + j a.y)(v.x + j v.y): re += a.x v.x - a.y v.y, im += a.x v.y + a.y v.x
      re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, v[t].x, re[t], 0, 0, 0);
      re[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(-a.y, v[t].y, re[t], 0, 0, 0);
      im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, v[t].y, im[t], 0, 0, 0);
      im[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, v[t].x, im[t], 0, 0, 0);
    }
  }
  // D[m][n]: lane holds rows 4 (lane / 16) + r, r = 0..3, column lane % 16
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int k = k0 + t * 16 + am;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int l = l0 + 4 * ak + r;
      if (l < N && k < M) dst[(int64_t)l * M + k] = make_float2(re[t][r], im[t][r]);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Short DFTs in registers (forward sign).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float uniform_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
// A uniform value that the optimiser forms where it is used, instead of keeping what follows
// from it in registers for every radix that the strip loop could run.
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+s"(v));
  return v;
}
__device__ __forceinline__ void dft2(float2& a, float2& b) {
  const float2 t = a;
  a = cadd(t, b);
  b = csub(t, b);
}
// natural order in and out
__device__ __forceinline__ void dft4(float2& a, float2& b, float2& c, float2& d) {
  dft2(a, c);
  dft2(b, d);
  d = make_float2(d.y, -d.x);   // times -j
  dft2(a, b);
  dft2(c, d);
  const float2 t = b;           // bins 0, 2, 1, 3 sit in a, b, c, d
  b = c;
  c = t;
}
// R = 4 S: 4-point DFTs over i1 (i = S i1 + i2), twiddles e^{-j 2 pi i2 l1 / R}, S-point DFTs
// over i2 (l = l1 + 4 l2)
template <int S, class Emit>
__device__ __forceinline__ void dft4s(float2 (&v)[4 * S], Emit emit) {
  // cos(2 pi m / 16)
  constexpr float C[5] = {1.f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f, 0.f};
#pragma unroll
  for (int i2 = 0; i2 < S; ++i2) dft4(v[i2], v[S + i2], v[2 * S + i2], v[3 * S + i2]);
#pragma unroll
  for (int l1 = 0; l1 < 4; ++l1) {
#pragma unroll
    for (int i2 = 1; i2 < S; ++i2) {
      const int m = l1 * i2 * (4 / S);   // of 16; at most 9
      float2& e = v[S * l1 + i2];
      if (m == 4)
        e = make_float2(e.y, -e.x);
      else if (m > 4)                    // e^{-j(pi/2 + a)} = -j e^{-j a}
        e = m == 8 ? make_float2(-e.x, -e.y)
                   : cmul(make_float2(e.y, -e.x), m < 8 ? make_float2(C[(m - 4) & 3], -C[(8 - m) & 3])
                                                        : make_float2(-C[3], -C[1]));
      else if (m > 0)
        e = cmul(e, make_float2(C[m & 3], -C[4 - (m & 3)]));
    }
    if constexpr (S == 4)
      dft4(v[S * l1], v[S * l1 + 1], v[S * l1 + 2], v[S * l1 + 3]);
    else
      dft2(v[S * l1], v[S * l1 + 1]);
#pragma unroll
    for (int l2 = 0; l2 < S; ++l2) emit(l1 + 4 * l2, v[S * l1 + l2]);
  }
}
// The R bins of v, each given to emit(bin, value).  w[m] = e^{-j 2 pi m / R} (unused by the
// powers of two); other radices take the sums as they stand, the terms i and R - i together.
template <int R, class Emit>
__device__ __forceinline__ void short_dft(float2 (&v)[R], const float2 (&w)[R], Emit emit) {
  if constexpr (R == 2) {
    dft2(v[0], v[1]);
    emit(0, v[0]);
    emit(1, v[1]);
  } else if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3]);
#pragma unroll
    for (int l = 0; l < 4; ++l) emit(l, v[l]);
  } else if constexpr (R == 8 || R == 16) {
    dft4s<R / 4>(v, emit);
  } else {
    constexpr int H = (R - 1) / 2;
    float2 sum = v[0];
#pragma unroll
    for (int i = 1; i <= H; ++i) {
      dft2(v[i], v[R - i]);              // the sum and the difference of the pair
      sum = cadd(sum, v[i]);
    }
    if (R % 2 == 0) sum = cadd(sum, v[R / 2]);
    emit(0, sum);
#pragma unroll
    for (int l = 1; 2 * l <= R; ++l) {
      float2 a = R % 2 ? v[0] : (l % 2 ? csub(v[0], v[R / 2]) : cadd(v[0], v[R / 2]));
      float2 d = make_float2(0.f, 0.f);
#pragma unroll
      for (int i = 1; i <= H; ++i) {
        const float2 c = w[(l * i) % R];
        a.x += c.x * v[i].x;
        a.y += c.x * v[i].y;
        d.x += c.y * v[R - i].x;
        d.y += c.y * v[R - i].y;
      }
      emit(l, make_float2(a.x - d.y, a.y + d.x));
      if (2 * l != R) emit(R - l, make_float2(a.x + d.y, a.y - d.x));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// One strip of C columns in one pass of radix R (auto-sorting order: L = product of the radices
// before).  Butterfly j of N / R takes rows j + q N / R, times e^{-j 2 pi q (j mod L) / (L R)},
// and leaves its R bins at rows (j / L) L R + j mod L + q L.  GIN / GOUT: the frame in memory
// instead of the strip in LDS.
struct DztStrip {
  int M, N, C, tx, ty, TY, L;
  bool live, inverse;        // the column exists; bins in the opposite order
  float scale;
  const float2* tw;          // LDS: e^{-j 2 pi m / N}
  const float2* gin;         // this lane's column of the frame
  float2* gout;
  const float2* in;          // this lane's column of the strip in LDS
  float2* out;
};
template <int R, bool GIN, bool GOUT>
__device__ __forceinline__ void dzt_pass(const DztStrip& s) {
  const int M = here(s.M), N = here(s.N), C = here(s.C), L = GIN ? 1 : here(s.L);
  const int nb = N / R, ts = nb / L;   // ts = N / (L R)
  float2 w[R];
  if constexpr (R & (R - 1)) {
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const float2 t = s.tw[m * nb];
      w[m] = make_float2(uniform_f(t.x), uniform_f(t.y));
    }
  }
  int j = s.ty;
  asm volatile("" : "+v"(j));
  for (; j < nb; j += s.TY) {
    float2 v[R];
    const int jl = GIN ? 0 : j % L;
    if (GIN) {
      const float2* p = s.gin + (int64_t)j * M;
      const int64_t step = (int64_t)nb * M;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        v[q] = make_float2(0.f, 0.f);
        if (s.live) v[q] = *p;
        p += step;
      }
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = make_float2(v[q].x * s.scale, v[q].y * s.scale);
    } else {
      const float2* p = s.in + j * C;
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = p[q * (nb * C)];
#pragma unroll
      for (int q = 1; q < R; ++q) v[q] = cmul(v[q], s.tw[q * (jl * ts)]);
    }
    const int o = (j - jl) * R + jl;
    if (GOUT) {
      if (s.live)
        short_dft<R>(v, w, [&](int q, float2 x) __attribute__((always_inline)) {
          const int row = o + q * L;
          s.gout[(int64_t)(s.inverse && row ? N - row : row) * M] = x;
        });
    } else {
      float2* const p = s.out + o * C;
      short_dft<R>(v, w, [&](int q, float2 x) __attribute__((always_inline)) { p[q * (L * C)] = x; });
    }
  }
}
template <bool GIN, bool GOUT>
__device__ __forceinline__ void dzt_pass_any(int r, const DztStrip& s) {
  switch (r) {
    case 2: dzt_pass<2, GIN, GOUT>(s); break;
    case 3: dzt_pass<3, GIN, GOUT>(s); break;
    case 4: dzt_pass<4, GIN, GOUT>(s); break;
    case 5: dzt_pass<5, GIN, GOUT>(s); break;
    case 6: dzt_pass<6, GIN, GOUT>(s); break;
    case 7: dzt_pass<7, GIN, GOUT>(s); break;
    case 8: dzt_pass<8, GIN, GOUT>(s); break;
    case 9: dzt_pass<9, GIN, GOUT>(s); break;
    case 10: dzt_pass<10, GIN, GOUT>(s); break;
    case 11: dzt_pass<11, GIN, GOUT>(s); break;
    case 12: dzt_pass<12, GIN, GOUT>(s); break;
    case 13: dzt_pass<13, GIN, GOUT>(s); break;
    case 14: dzt_pass<14, GIN, GOUT>(s); break;
    case 15: dzt_pass<15, GIN, GOUT>(s); break;
    default: dzt_pass<16, GIN, GOUT>(s); break;
  }
}

// Strips are walked by a fixed grid, so that a workgroup forms its twiddles once.  launch bounds:
// two workgroups of 512 threads per CU, one loading while the other transforms.
struct DztPlan {
  int r[3];       // radices; r[2] = 1: two passes
  int C, TY;      // columns per strip (a power of two), threads per column
};
__global__ __launch_bounds__(kDztFftThreads, 4) void k_dzt_fft(int M, int N, int64_t nstrips, int per_frame,
                                                            DztPlan P, bool inverse,
                                                            const float2* __restrict__ in,
                                                            float2* __restrict__ out) {
  extern __shared__ float2 tw[];   // N twiddles, then one or two strips of N x C
  const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
  for (int m = tid; m < N; m += nt) {
    double sn, c;
    sincospi(2.0 * (double)m / (double)N, &sn, &c);
    tw[m] = make_float2((float)c, (float)-sn);
  }
  __syncthreads();
  DztStrip s;
  s.M = M;
  s.N = N;
  s.C = P.C;
  s.tx = tid & (P.C - 1);
  s.ty = tid / P.C;
  s.TY = P.TY;
  s.inverse = inverse;
  s.scale = (float)(1.0 / sqrt((double)N));
  s.tw = tw;
  float2* const a = tw + N + s.tx;
  float2* const b = a + N * P.C;
  for (int64_t it = blockIdx.x; it < nstrips; it += gridDim.x) {
    const int64_t f = it / per_frame;
    const int k = (int)(it - f * per_frame) * P.C + s.tx;
    s.live = k < M;
    s.gin = in + f * M * N + (s.live ? k : 0);
    s.gout = out + f * M * N + (s.live ? k : 0);
    s.out = a;
    s.L = 1;
    dzt_pass_any<true, false>(P.r[0], s);
    __syncthreads();
    s.in = a;
    s.L = P.r[0];
    if (P.r[2] > 1) {
      s.out = b;
      dzt_pass_any<false, false>(P.r[1], s);
      __syncthreads();
      s.in = b;
      s.L *= P.r[1];
    }
    dzt_pass_any<false, true>(P.r[2] > 1 ? P.r[2] : P.r[1], s);
    __syncthreads();
  }
}

// The radices: two passes if N has them, else three (false: N has a prime factor above 13, or
// does not split into three); fewest passes, then the smallest largest radix.
bool dzt_radices(int N, int (&r)[3]) {
  int best = 0;
  for (int a = 16; a >= 2; --a)
    if (N % a == 0 && N / a <= a && N / a >= 2) best = a;
  if (best) {
    r[0] = best;
    r[1] = N / best;
    r[2] = 1;
    return true;
  }
  int top = 17;
  for (int a = 16; a >= 2; --a)
    for (int b = a; b >= 2; --b) {
      if (N % (a * b) != 0) continue;
      const int c = N / (a * b);
      if (c < 2 || c > b || a >= top) continue;
      top = a;
      r[0] = a;
      r[1] = b;
      r[2] = c;
    }
  return top <= 16;
}

}  // namespace

hipError_t launch_dzt(int M, int N, int nframes, bool inverse, const float2* in, float2* out,
                      hipStream_t s) {
  if (nframes <= 0) return hipSuccess;
  const int64_t nb = (int64_t)((N + kDztRows - 1) / kDztRows) * ((M + kDztCols - 1) / kDztCols) *
                     nframes;
  if (nb > 0x7fffffff) return hipErrorInvalidValue;
  if (N > kDztMaxN) return hipErrorInvalidValue;
  // From 65 bins on the passes are the faster (80 bins: 67 -> 25 us for 100 frames of 1024
  // columns).  Below, speed does not draw the line: at full batches k_dzt is up to 2.5 times
  // slower (64 bins: 105 against 43 us, 16 bins: equal).  It stays because the receiver's short
  // frames are decided on its rounding; the passes would move single decisions there.  Above 2048 bins a strip of 4 columns
  // no longer fits the LDS twice, and a prime factor above 13 has no short DFT.
  DztPlan P;
  if (N >= kDztFftMinN && N <= kDztFftMaxN && dzt_radices(N, P.r)) {
    // strips as wide as two workgroups per CU (one with three passes, which need a second
    // buffer) leave room for, narrower while they do not fill the chip's 256 CUs
    const int bufs = P.r[2] > 1 ? 2 : 1;
    auto bytes = [&](int C) { return ((size_t)N + (size_t)bufs * N * C) * sizeof(float2); };
    P.C = 64;
    while (P.C > 4 && bytes(P.C) > (bufs == 1 ? 80 * 1024u : (unsigned)kDztFftLdsBytes)) P.C /= 2;
    while (P.C > 8 && (int64_t)nframes * ((M + P.C - 1) / P.C) < 256) P.C /= 2;
    P.TY = N / P.r[0] < kDztFftThreads / P.C ? N / P.r[0] : kDztFftThreads / P.C;
    const int per_frame = (M + P.C - 1) / P.C;
    const int64_t strips = (int64_t)per_frame * nframes;
    const size_t lds = bytes(P.C);
    const int grid = (int)(strips < 1024 ? strips : 1024);
    static std::atomic<uint64_t> done;
    const hipError_t e = lds_limit(reinterpret_cast<const void*>(&k_dzt_fft), kDztFftLdsBytes, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dzt_fft, dim3((unsigned)grid), dim3((unsigned)(P.C * P.TY)), lds, s, M, N,
                       strips, per_frame, P, inverse, in, out);
    return hipGetLastError();
  }
  const size_t lds = (size_t)N * sizeof(float2);
  hipLaunchKernelGGL(k_dzt, dim3((unsigned)nb), dim3(kDztThreads), lds, s, M, N, nframes,
                     inverse ? 1.f : -1.f, in, out);
  return hipGetLastError();
}

}  // namespace otfs
