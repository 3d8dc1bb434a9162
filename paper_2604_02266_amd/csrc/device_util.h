// Device helpers shared by the kernels: complex arithmetic, memory views, reductions,
// decisions and per-frame state.  Not part of the public ABI.
#pragma once

#include <math.h>

#include "otfs_internal.h"

namespace otfs {
namespace {

// ---------------------------------------------------------------------------------------
// small complex helpers
// ---------------------------------------------------------------------------------------
// explicit fused multiply-adds: the rounding does not depend on how the compiler would
// contract the expression in each kernel, so every kernel forms the same coefficients
__device__ __forceinline__ float2 cmulf(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ void cmacf(float2& acc, float2 c, float2 v) {
  acc.x = fmaf(c.x, v.x, acc.x);
  acc.x = fmaf(-c.y, v.y, acc.x);
  acc.y = fmaf(c.x, v.y, acc.y);
  acc.y = fmaf(c.y, v.x, acc.y);
}
__device__ __forceinline__ double2 cmuld(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ void cmacd(double2& acc, double2 c, double2 v) {
  acc.x = fma(c.x, v.x, acc.x);
  acc.x = fma(-c.y, v.y, acc.x);
  acc.y = fma(c.x, v.y, acc.y);
  acc.y = fma(c.y, v.x, acc.y);
}
// e^{j 2 pi num / mn}, num in [0, mn)
__device__ __forceinline__ double2 reduced_phasor(int64_t num, int64_t mn) {
  double sn, cs;
  sincospi(2.0 * ((double)num / (double)mn), &sn, &cs);
  return make_double2(cs, sn);
}
// the same for any num
__device__ __forceinline__ double2 unit_phasor(int64_t num, int64_t mn) {
  num %= mn;
  return reduced_phasor(num < 0 ? num + mn : num, mn);
}
// bf16 pair (re in the low half, im in the high half) -> complex64
__device__ __forceinline__ float2 bf16x2_to_f2(uint32_t w) {
  return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
}
// round-to-nearest-even float -> bf16 bits
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (u >> 16) | ((u & 0xffffu) ? 0x40u : 0u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ float2 load_y(const void* y, int64_t i, bool bf16) {
  if (bf16) return bf16x2_to_f2(static_cast<const uint32_t*>(y)[i]);
  return static_cast<const float2*>(y)[i];
}
// c + s * p, one rounding per component (used identically wherever a value is recomputed)
__device__ __forceinline__ float2 axpyf(float s, float2 p, float2 c) {
  return make_float2(fmaf(s, p.x, c.x), fmaf(s, p.y, c.y));
}

// ---------------------------------------------------------------------------------------
// memory views
// ---------------------------------------------------------------------------------------
// Pointers kept in frame descriptors are generic; these casts tell the compiler which
// memory they address, so that accesses become global (not flat) instructions, and
// wave-uniform table reads through a constant view become scalar loads.
template <class T>
using gptr = __attribute__((address_space(1))) T*;
template <class T>
using kptr = __attribute__((address_space(4))) T*;
template <class T>
using lptr = __attribute__((address_space(3))) T*;
template <class T>
__device__ __forceinline__ gptr<T> glb(T* p) {
  return (gptr<T>)p;
}
typedef unsigned long long u64;
// 8-byte pairs (complex64, int pairs) are moved as 64-bit words through these views.
struct GPairs {   // global table
  gptr<const u64> p;
  __device__ __forceinline__ float2 f(int64_t i) const { return __builtin_bit_cast(float2, p[i]); }
};
struct KPairs {   // wave-uniform table: scalar loads
  kptr<const u64> p;
  __device__ __forceinline__ float2 f(int i) const { return __builtin_bit_cast(float2, p[i]); }
  __device__ __forceinline__ int2 i2(int i) const { return __builtin_bit_cast(int2, p[i]); }
};
struct LdsC {     // complex64 array in LDS
  lptr<u64> p;
  __device__ __forceinline__ float2 ld(int i) const { return __builtin_bit_cast(float2, p[i]); }
  __device__ __forceinline__ void st(int i, float2 v) const { p[i] = __builtin_bit_cast(u64, v); }
  __device__ __forceinline__ LdsC operator+(int o) const { return LdsC{p + o}; }
};
__device__ __forceinline__ GPairs gpairs(const void* t) { return GPairs{(gptr<const u64>)t}; }
__device__ __forceinline__ KPairs kpairs(const void* t) { return KPairs{(kptr<const u64>)t}; }
__device__ __forceinline__ LdsC lds_c(void* t) { return LdsC{(lptr<u64>)t}; }

// A vector of `bytes` bytes read through a buffer resource: the base stays in SGPRs and
// each read takes one 32-bit byte offset (frames hold at most 2^28 elements, so every
// offset fits).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, int64_t bytes) {
  const uint32_t n = bytes > 0xffffffffLL ? 0xffffffffu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)n, 0x00020000);
}

// Source views of a band application: load(i) issues the reads of element i, value(raw)
// forms the element from them; load_b(vb, sb) reads the element at byte offset vb + sb of
// a complex64 vector, where sb is the same for the whole wave when the caller can prove
// it (it then goes into the instruction's scalar offset).  A stageable view also names the kNV complex64 vectors it
// reads (rsrc(j)) and forms the element from their values (combine); own(i, v) reads them
// at element i.
// Cache policy kL2 (the sc1 bit, agent scope): the read misses this CU's L1 and is served by
// the L2.  Vectors that other workgroups of the launch write are read this way, so a wait
// needs no invalidate after it: the agent-scope invalidate walks the whole L2 and took 13.5 of
// the 14.9 us of a barrier of 8 workgroups (1.0 us without it).
constexpr int kL2 = 16;
template <int POLICY = 0>
__device__ __forceinline__ float2 buf_ld2(__amdgpu_buffer_rsrc_t r, uint32_t i) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, i * 8u, 0, POLICY));
}
template <int POLICY = 0>
__device__ __forceinline__ float2 buf_ld2b(__amdgpu_buffer_rsrc_t r, uint32_t vb, uint32_t sb) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, vb, sb, POLICY));
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Two adjacent complex64 elements moved as one 16-byte access (the paired gathers).
template <int POLICY = 0>
__device__ __forceinline__ u32x4 buf_ld4b(__amdgpu_buffer_rsrc_t r, uint32_t vb, uint32_t sb) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, vb, sb, POLICY));
}
__device__ __forceinline__ void unpack2(u32x4 v, float2& a, float2& b) {
  a = __builtin_bit_cast(float2, u32x2{v.x, v.y});
  b = __builtin_bit_cast(float2, u32x2{v.z, v.w});
}
__device__ __forceinline__ u32x4 pack2(float2 a, float2 b) {
  const u32x2 x = __builtin_bit_cast(u32x2, a), y = __builtin_bit_cast(u32x2, b);
  return u32x4{x.x, x.y, y.x, y.y};
}
template <int POL>
struct SrcBufT {   // complex64 vector
  __amdgpu_buffer_rsrc_t r;
  static constexpr int kPol = POL;
  static constexpr int kNV = 1;
  static constexpr bool kStageable = true;
  static constexpr bool kPairs = true;
  using Raw = float2;
  using Raw2 = u32x4;
  __device__ __forceinline__ Raw load(uint32_t i) const { return buf_ld2<POL>(r, i); }
  __device__ __forceinline__ Raw load_b(uint32_t vb, uint32_t sb) const { return buf_ld2b<POL>(r, vb, sb); }
  __device__ __forceinline__ float2 value(Raw v) const { return v; }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int) const { return r; }
  __device__ __forceinline__ float2 combine(const float2* v) const { return v[0]; }
  __device__ __forceinline__ void own(uint32_t i, float2* v) const { v[0] = buf_ld2<POL>(r, i); }
  // pairs: the elements at byte offsets vb + sb and vb + sb + 8
  __device__ __forceinline__ Raw2 load2_b(uint32_t vb, uint32_t sb) const { return buf_ld4b<POL>(r, vb, sb); }
  __device__ __forceinline__ void value2(const Raw2& v, float2& a, float2& b) const { unpack2(v, a, b); }
  __device__ __forceinline__ void own2(uint32_t i, float2* a, float2* b) const {
    unpack2(buf_ld4b<POL>(r, i * 8u, 0), a[0], b[0]);
  }
};
using SrcBuf = SrcBufT<0>;       // written before the launch
using SrcShared = SrcBufT<kL2>;  // written by the frame's workgroups during the launch
struct SrcBf16 {  // complex stored as a bf16 pair per element (not staged)
  __amdgpu_buffer_rsrc_t r;
  static constexpr int kPol = 0;
  static constexpr int kNV = 1;
  static constexpr bool kStageable = false;
  static constexpr bool kPairs = false;
  using Raw = uint32_t;
  __device__ __forceinline__ Raw load(uint32_t i) const {
    return __builtin_amdgcn_raw_buffer_load_b32(r, i * 4u, 0, 0);
  }
  __device__ __forceinline__ Raw load_b(uint32_t vb, uint32_t sb) const {   // bytes of complex64
    return __builtin_amdgcn_raw_buffer_load_b32(r, vb >> 1, sb >> 1, 0);
  }
  __device__ __forceinline__ float2 value(Raw v) const { return bf16x2_to_f2(v); }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int) const { return r; }
  __device__ __forceinline__ float2 combine(const float2* v) const { return v[0]; }
  __device__ __forceinline__ void own(uint32_t i, float2* v) const { v[0] = value(load(i)); }
};
struct SrcDir {   // the new direction c + beta p, formed from c and the old p
  __amdgpu_buffer_rsrc_t c, p;
  float beta;
  static constexpr int kPol = kL2;
  static constexpr int kNV = 2;
  static constexpr bool kStageable = true;
  struct Raw {
    float2 c, p;
  };
  __device__ __forceinline__ Raw load(uint32_t i) const { return Raw{buf_ld2<kL2>(c, i), buf_ld2<kL2>(p, i)}; }
  __device__ __forceinline__ Raw load_b(uint32_t vb, uint32_t sb) const {
    return Raw{buf_ld2b<kL2>(c, vb, sb), buf_ld2b<kL2>(p, vb, sb)};
  }
  __device__ __forceinline__ float2 value(const Raw& v) const { return axpyf(beta, v.p, v.c); }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int j) const { return j == 0 ? c : p; }
  __device__ __forceinline__ float2 combine(const float2* v) const { return axpyf(beta, v[1], v[0]); }
  __device__ __forceinline__ void own(uint32_t i, float2* v) const {
    v[0] = buf_ld2<kL2>(c, i);
    v[1] = buf_ld2<kL2>(p, i);
  }
  static constexpr bool kPairs = true;
  struct Raw2 {
    u32x4 c, p;
  };
  __device__ __forceinline__ Raw2 load2_b(uint32_t vb, uint32_t sb) const {
    return Raw2{buf_ld4b<kL2>(c, vb, sb), buf_ld4b<kL2>(p, vb, sb)};
  }
  __device__ __forceinline__ void value2(const Raw2& v, float2& a, float2& b) const {
    float2 c0, c1, p0, p1;
    unpack2(v.c, c0, c1);
    unpack2(v.p, p0, p1);
    a = axpyf(beta, p0, c0);
    b = axpyf(beta, p1, c1);
  }
  __device__ __forceinline__ void own2(uint32_t i, float2* a, float2* b) const {
    unpack2(buf_ld4b<kL2>(c, i * 8u, 0), a[0], b[0]);
    unpack2(buf_ld4b<kL2>(p, i * 8u, 0), a[1], b[1]);
  }
};
struct SrcLds {   // complex64 vector in LDS
  LdsC v;
  using Raw = float2;
  __device__ __forceinline__ Raw load(uint32_t i) const { return v.ld((int)i); }
  __device__ __forceinline__ Raw load_b(uint32_t vb, uint32_t sb) const {
    return v.ld((int)((vb + sb) >> 3));
  }
  __device__ __forceinline__ float2 value(Raw x) const { return x; }
};

// A complex64 vector read and written element-wise through a buffer resource (one 32-bit
// offset per element, shared by every vector accessed at that element).
// NT: non-temporal cache policy (streamed data that should not displace gather sources
// in L2).
struct CVec {
  __amdgpu_buffer_rsrc_t r;
  template <bool NT = false>
  __device__ __forceinline__ float2 ld(uint32_t i) const {
    return __builtin_bit_cast(float2,
                              __builtin_amdgcn_raw_buffer_load_b64(r, i * 8u, 0, NT ? 2 : 0));
  }
  template <bool NT = false>
  __device__ __forceinline__ void st(uint32_t i, float2 v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, i * 8u, 0,
                                          NT ? 2 : 0);
  }
  // elements i and i + 1 as one 16-byte access
  template <bool NT = false>
  __device__ __forceinline__ void ld2(uint32_t i, float2& a, float2& b) const {
    unpack2(buf_ld4b<NT ? 2 : 0>(r, i * 8u, 0), a, b);
  }
  template <bool NT = false>
  __device__ __forceinline__ void st2(uint32_t i, float2 a, float2 b) const {
    __builtin_amdgcn_raw_buffer_store_b128(pack2(a, b), r, i * 8u, 0, NT ? 2 : 0);
  }
};

__device__ __forceinline__ CVec cvec(const float2* p, int64_t n) { return CVec{buf_rsrc(p, n * 8)}; }

// ---------------------------------------------------------------------------------------
// reductions: wave64 butterfly, then the waves of the block in a fixed order
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) s += red[i];
  __syncthreads();
  return s;
}
__device__ __forceinline__ double block_sum_d(double v, double* red) {
  v = wave_sum_d(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) s += red[i];
  __syncthreads();
  return s;
}
// a value that another workgroup of this launch stored: read past this CU's L1
template <class T>
__device__ __forceinline__ T shared_ld(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Sum of the T per-tile partials of a frame, in tile order, by every thread: every workgroup of
// the frame forms the same value, independent of the rest of the batch.  The loads go in groups
// of 8 in flight together.  PAST_L1: the partials are stores of this launch's other workgroups,
// after which nothing was invalidated; else a launch boundary or an acquire fence orders them,
// and the L1 serves the 512 threads' reads of one word.  Read past it all the same, the unfused
// form on 256 tiles per frame took 15.4 ms instead of 8.3 (16 frames of 1024 x 256, 10
// iterations), and the fused form with device-wide fences 95.4 ms instead of 68.8 (20
// iterations).  By whole waves, one word per lane and 256 readlanes: 9.9 and 75.8 ms.
template <bool PAST_L1, class V>
__device__ __forceinline__ V part_ld(const V* p) {
  if constexpr (PAST_L1) return shared_ld(p);
  return *p;
}
template <bool PAST_L1>
__device__ __forceinline__ float tile_sum(const float* part, int T) {
  float s = 0.f;
  int i = 0;
  for (; i + 8 <= T; i += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = part_ld<PAST_L1>(part + i + j);
#pragma unroll
    for (int j = 0; j < 8; ++j) s = __fadd_rn(s, v[j]);
  }
  for (; i < T; ++i) s = __fadd_rn(s, part_ld<PAST_L1>(part + i));
  return s;
}
template <bool PAST_L1>
__device__ __forceinline__ double tile_sum_d(const double* part, int T) {
  double s = 0.0;
  int i = 0;
  for (; i + 8 <= T; i += 8) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = part_ld<PAST_L1>(part + i + j);
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
  }
  for (; i < T; ++i) s += part_ld<PAST_L1>(part + i);
  return s;
}

// ---------------------------------------------------------------------------------------
// hard decisions (Eq. demod): nearest square-QAM level per axis, ties to the upper level
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int decide_axis(float v, float s, int m) {
  float t = __fmul_rn(v, s);
  t = __fadd_rn(t, (float)m);
  t = __fmul_rn(t, 0.5f);
  t = t == t ? t : 0.f;                         // NaN -> lowest level
  t = fminf(fmaxf(t, 0.f), (float)(m - 1));
  return (int)floorf(t);
}
__device__ __forceinline__ uint8_t decide(float2 x, float s, int m) {
  return (uint8_t)(decide_axis(x.x, s, m) * m + decide_axis(x.y, s, m));
}

struct FrameVecs {
  const void* y;
  float2* x;
  uint8_t* sym;
  otfs_frame_stats* stats;
  bool ybf16;
};
__device__ __forceinline__ FrameVecs frame_vecs(const FrameDev& F, const Bases& B) {
  FrameVecs v;
  v.ybf16 = (F.flags & OTFS_Y_BF16) != 0;
  if (B.y)
    v.y = static_cast<const char*>(B.y) + F.off * (v.ybf16 ? 4 : 8);
  else
    v.y = F.y;
  v.x = B.x ? B.x + F.off : F.x;
  v.sym = B.sym ? B.sym + F.off : F.sym;
  v.stats = B.stats ? B.stats + F.index : F.stats;
  return v;
}

struct LaunchCtx {
  unsigned* abort_flag;
  uint64_t timeout;
  int xcd_local;     // barrier coherence mode (see frame_barrier)
};

// A frame's state as every lane holds it: read through the vector path (other workgroups
// write it), then taken from the first lane, so that what is derived from it (which
// direction buffer is current, and the buffer descriptors built on that) stays in scalar
// registers instead of every buffer access being repeated per distinct descriptor.
__device__ __forceinline__ FrameState uniform_state(const FrameState* p) {
  FrameState s = *p;
  s.iter = __builtin_amdgcn_readfirstlane(s.iter);
  s.status = __builtin_amdgcn_readfirstlane(s.status);
  s.pbuf = __builtin_amdgcn_readfirstlane(s.pbuf);
  s.pending = __builtin_amdgcn_readfirstlane(s.pending);
  s.init = __builtin_amdgcn_readfirstlane(s.init);
  s.refresh = __builtin_amdgcn_readfirstlane(s.refresh);
  return s;
}

// XCC (XCD) this wave runs on, from the hardware register XCC_ID, bits [3:0].
__device__ __forceinline__ int xcc_id() {
  return (int)(__builtin_amdgcn_s_getreg((15 << 11) | (0 << 6) | 20) & 0xfu);
}

// Item of this workgroup in a launch of one workgroup per item.  Workgroup b runs on XCD b % nxcd; the
// workgroups of one XCD take consecutive items (the items of a frame are consecutive), so
// the tiles of a frame, whose windows share the rows of the Doppler range, read them
// through one L2.  A bijection of [0, nitems) for any nitems and nxcd >= 1.
__device__ __forceinline__ int xcd_item(int nitems, int nxcd) {
  if (nxcd <= 1) return (int)blockIdx.x;
  const int b = (int)blockIdx.x, x = b % nxcd;
  int o = 0;
  for (int y = 0; y < x; ++y) o += (nitems - y + nxcd - 1) / nxcd;
  return o + b / nxcd;
}

}  // namespace
}  // namespace otfs
