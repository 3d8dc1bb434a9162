// Register-resident CG tiles: the fused solve with every CG vector of a frame kept in the
// register files of the workgroups that share it.
//
// A frame of M delay by N Doppler bins is cut into tk_nbr row bands x tk_nbc column strips,
// one 512-thread workgroup (one per CU) per tile of at most 8192 elements; all tiles of a
// frame run on one XCD.  x, c and p of the tile live in registers for the whole solve, and a
// in the accumulators of the pass that forms it.  Per iteration only p' and t leave the
// workgroup, through the XCD's L2, for the neighbouring tiles:
//   A: x += alpha p, p' = c + beta p, p' stored                              | neighbours
//      window of p' -> LDS, t = H p', t stored                               | neighbours
//   B: window of t -> LDS, a = H^H t + lam p', Re(p'^H a)                    | all tiles
//   C: c -= alpha a, ||c||^2                                                 | all tiles
// The streaming form of the same loop moves 96 bytes per element and iteration through the
// memory system; this one moves 16 plus the windows' halos through L2.
//
// Window.  A tile of TR rows x TC columns gathers from rows [r0 - nu_hi, r1 - nu_lo) (H; H^H:
// [r0 + nu_lo, r1 + nu_hi)) and columns [c0 - tau_hi, c1 - tau_lo) (H^H: + tau) of the source,
// copied once per pass into LDS with wrapped rows and columns laid out in place, so no gather
// tests for a wrap.  A delay wrap's factor W[l0]^n (l0 the source row, n the wrap count)
// depends only on the window element, so the few wrapped columns are multiplied by it once
// after the copy: the window holds the quasi-periodic extension of the source, and the
// path loop is coefficient times element.  For H^H the same extension holds with the
// coefficient S_p[k] = conj(R_p[k + tau]) continued past the row's end, where it takes
// W[nu]^-n: a table of its own (k_tile_tables), so H^H costs what H does.
//
// Lanes.  In the two-column form (CW = 2, strips of up to 128 columns) lane i owns columns i
// and i + 64 of its rows: both reads of a row come from one address (ds_read2st64_b64), each
// a run of 64 consecutive elements, free of bank conflicts.  The one-column form (CW = 1)
// serves every other width.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "device_util.h"
#include "otfs_internal.h"

namespace otfs {
namespace {

constexpr int kStepElems = 8;   // elements of one thread read from the window per step

// Sum over the wave by DPP row operations; every lane receives it.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_total(float v) {
  v += dpp_mov<0xB1, 0xf>(v);    // quad_perm 1,0,3,2
  v += dpp_mov<0x4E, 0xf>(v);    // quad_perm 2,3,0,1
  v += dpp_mov<0x141, 0xf>(v);   // row_half_mirror
  v += dpp_mov<0x140, 0xf>(v);   // row_mirror: every lane holds its row's sum
  v += dpp_mov<0x142, 0xa>(v);   // row_bcast15 into rows 1 and 3
  v += dpp_mov<0x143, 0xc>(v);   // row_bcast31 into rows 2 and 3: lane 63 holds the total
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float uniform_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ int wrap_once(int v, int n) {   // v in [-n, 2n)
  v += v < 0 ? n : 0;
  return v - (v >= n ? n : 0);
}
__device__ __forceinline__ int wrap_row(int v, int n) {    // v in [-n, 4n)
  v += v < 0 ? n : 0;
  v -= v >= 2 * n ? 2 * n : 0;
  return v - (v >= n ? n : 0);
}
__device__ __forceinline__ int mod_pos(int a, int n) {
  const int r = a % n;
  return r < 0 ? r + n : r;
}

// The thread's index, hidden from the optimiser: what is derived from it is formed where it
// is used, instead of being kept in registers across the iteration loop.
__device__ __forceinline__ int tid_here() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Meeting of a frame's tiles.  Each tile owns one 64-bit word {epoch, value} per kind of
// meeting; a tile stores its word and one wave polls the words of the tiles it needs, one lane
// per tile, until all carry the epoch: arrival and reduction in one round trip.  The word's
// store stays in the shared L2 (an agent-scope store writes through it: 1.0 us per meeting of
// 8 workgroups and 1.9 us of 32, against 0.67 and 0.69 us).  The stores of p' and t before it are released by
// s_waitcnt vmcnt(0) (they are in the shared L2); the reads after it pass the L1.  A word
// is not stored again before every tile has passed the next all-tiles meeting, so no value
// is overwritten unread.  Bounded as the other kinds' waits are.
struct Meet {
  u64* slots;
  unsigned* abort_flag;
  uint64_t timeout;
  int T, me;
  float* red;      // kWaves floats of LDS
  float* out;      // LDS
  int* ok;         // LDS
};
// need: this lane's tile takes part (lanes of the first wave).  REDUCE: the sum of val over
// all threads of all T tiles, the same bits in every tile; else 0.
// between(): work of every wave after the workgroup's own meeting, while the other tiles' words
// are on their way.
template <bool REDUCE, bool RELEASE, class F>
__device__ __forceinline__ bool meet(const Meet& m, int kind, unsigned epoch, bool need, float val,
                                     float* sum, F between) {
  if (RELEASE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const int tid = tid_here();
  if (REDUCE) {
    const float w = wave_total(val);
    if ((tid & 63) == 0) m.red[tid >> 6] = w;
  }
  __syncthreads();
  float tot = 0.f;
  if (tid < 64) {
    if (REDUCE) {
#pragma unroll
      for (int i = 0; i < kWaves; ++i) tot += m.red[i];
    }
    if (m.T > 1 && tid == 0)
      __hip_atomic_store(m.slots + kind * m.T + m.me, ((u64)epoch << 32) | (u64)__float_as_uint(tot),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  between();
  if (tid < 64) {
    const int lane = tid;
    int ok = 1;
    if (m.T > 1) {
      const u64* sl = m.slots + kind * m.T;
      bool done = lane >= m.T || !need;
      u64 w = 0;
      const uint64_t t0 = wall_clock64();
      for (;;) {
        if (!done) {
          w = __hip_atomic_load(sl + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          done = (unsigned)(w >> 32) >= epoch;
        }
        if (__builtin_amdgcn_ballot_w64(!done) == 0) break;
        if (__hip_atomic_load(m.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u ||
            wall_clock64() - t0 > m.timeout) {
          if (lane == 0)
            __hip_atomic_store(m.abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
      }
      if (REDUCE) tot = wave_total(lane < m.T ? __uint_as_float((unsigned)w) : 0.f);
    }
    if (lane == 0) {
      *m.ok = ok;
      if (REDUCE) *m.out = tot;
    }
  }
  __syncthreads();
  if (REDUCE) *sum = uniform_f(*m.out);
  return __builtin_amdgcn_readfirstlane(*m.ok) != 0;
}

template <bool REDUCE, bool RELEASE>
__device__ __forceinline__ bool meet(const Meet& m, int kind, unsigned epoch, bool need, float val,
                                     float* sum) {
  return meet<REDUCE, RELEASE>(m, kind, epoch, need, val, sum, [] {});
}

// Whether the cyclic ranges [a, a + na) and [b, b + nb) modulo n meet.
__device__ __forceinline__ bool cyc_meet(int a, int na, int b, int nb, int n) {
  return mod_pos(b - a, n) < na || mod_pos(a - b, n) < nb;
}

struct Window {   // of one direction (H or H^H)
  int row0, col0;      // source row and column (unwrapped) of window element (0, 0)
  int orow, ocol;      // where the tile's own elements sit in it
  int cend;            // columns that any path reaches
  const float2* wrow;  // LDS: W of each window row
};

// Copy a window's halo straight into LDS (16-byte direct-to-LDS loads; M, the strips and every
// window's first column are even), then multiply the wrapped columns.  The tile's own TR x TC
// elements are already there (written from registers).  A wave copies whole rows: the source
// row goes into the instruction's scalar offset and the lanes' column offsets are the same for
// every row, so the copy loops have no vector arithmetic (walking the window as one run of
// 128-element pieces took 25 vector instructions per load).
__device__ __forceinline__ void window_dma(__amdgpu_buffer_rsrc_t r, const Window& w, int WR, int WC,
                                           int TR, int TC, int M, int N, lptr<u64> win,
                                           bool factors = true) {
  const int tid = tid_here();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  // columns [q0, q1) of n rows: `own` the tile's rows, else the rows above and below them
  auto copy = [&](int q0, int q1, int n, bool own) __attribute__((always_inline)) {
    for (int q = q0; q < q1; q += 128) {
      const uint32_t vo = 8u * (uint32_t)wrap_once(w.col0 + q + 2 * lane, M);
      if (q + 2 * lane < q1) {
        for (int h = wave; h < n; h += kWaves) {
          const int rr = own ? w.orow + h : (h < w.orow ? h : h + TR);
          __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr<void>)(win + rr * WC + q), 16, vo,
                                                   (uint32_t)(wrap_row(w.row0 + rr, N) * M) * 8u,
                                                   0, kL2);
        }
      }
    }
  };
  copy(0, w.cend, WR - TR, false);
  copy(0, w.ocol, TR, true);
  copy(w.ocol + TC, w.cend, TR, true);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const int nlo = max(0, -w.col0), nhi = max(0, w.col0 + w.cend - M), nw = nlo + nhi;
  if (nw == 0 || !factors) return;
  for (int q = lane; q < nw; q += 64) {
    const lptr<u64> col = win + (q < nlo ? q : w.cend - nw + q);
    const float sg = q < nlo ? -1.f : 1.f;
#pragma unroll 4
    for (int rr = wave; rr < WR; rr += kWaves) {
      const float2 f = w.wrow[rr];
      col[rr * WC] = __builtin_bit_cast(
          u64, cmulf(__builtin_bit_cast(float2, col[rr * WC]), make_float2(f.x, sg * f.y)));
    }
  }
  __syncthreads();
}

// The same window through registers, one element per lane: any M, any source view.
template <class Src>
__device__ __forceinline__ void window_fill(const Src& src, const Window& w, int WR, int WC, int M,
                                            int N, lptr<u64> win, bool factors = true) {
  constexpr int U = 4;
  const int total = WR * WC;
  const int dr = kBlock / WC, dc = kBlock - dr * WC;
  const int tid = tid_here();
  int rr = tid / WC, cc = tid - rr * WC;
  for (int e = tid; e < total; e += U * kBlock) {
    typename Src::Raw raw[U];
    int row[U], col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      row[u] = min(rr, WR - 1);
      col[u] = w.col0 + cc;
      const int sc = wrap_once(col[u], M);
      raw[u] = src.load((uint32_t)(wrap_row(w.row0 + row[u], N) * M + min(sc, M - 1)));
      rr += dr;
      cc += dc;
      if (cc >= WC) {
        cc -= WC;
        ++rr;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (e + u * kBlock < total) {
        float2 v = src.value(raw[u]);
        if (factors && (col[u] < 0 || col[u] >= M)) {
          const float2 f = w.wrow[row[u]];
          v = cmulf(v, make_float2(f.x, col[u] < 0 ? -f.y : f.y));
        }
        win[e + u * kBlock] = __builtin_bit_cast(u64, v);
      }
    }
  }
  __syncthreads();
}

// What one thread knows of its tile (the same for every pass).
template <int NJ, int CW>
struct Lanes {
  uint32_t la;         // LDS byte address of its first row at its first column, shift 0
  uint32_t lstep;      // LDS bytes from one of its rows to the next (uniform)
  uint32_t k8[CW];     // byte offset of its columns inside a table row (clamped to the tile)
  int full, last;      // rows that every thread holds; index of the last row any holds (uniform)
  bool tail;           // holds row `full` too
  bool col[CW];        // the thread holds elements of this column
  uint32_t ov[CW];     // byte offset of its first element in a frame vector
  uint32_t rstep;      // bytes from one of its rows to the next in a frame vector (uniform)
};

// The cut's tile: rows [r0, r0 + TR), columns [c0, c0 + TC), its thread layout (TY row groups
// of LX columns) and its window size.
struct TileBox {
  int r0, TR, c0, TC, LX, TY, tx, ty, WC, WR;
};
template <int CW>
__device__ __forceinline__ TileBox tile_box(const FrameDev& F, int nbr, int nbc, int tc, int tile) {
  TileBox b;
  const int rb = tile / nbc, sb = tile - rb * nbc;
  b.r0 = (int)((int64_t)rb * F.N / nbr);
  b.TR = (int)((int64_t)(rb + 1) * F.N / nbr) - b.r0;
  b.c0 = sb * tc;
  b.TC = min(tc, F.M - b.c0);
  b.LX = CW == 2 ? 64 : tc;
  b.TY = kBlock / b.LX;
  b.tx = (int)threadIdx.x % b.LX;
  b.ty = CW == 2 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / b.LX) : (int)threadIdx.x / b.LX;
  b.WC = (CW == 2 ? 128 : tc) + (F.tau_hi - F.tau_lo) + 1;
  b.WC += b.WC & 1;
  b.WR = b.TR + (F.nu_hi - F.nu_lo);
  return b;
}
// the windows of H (ADJ: H^H)
template <bool ADJ>
__device__ __forceinline__ Window tile_window(const FrameDev& F, const TileBox& b, const float2* wrow) {
  const int col0 = (ADJ ? b.c0 + F.tau_lo : b.c0 - F.tau_hi) & ~1;
  return ADJ ? Window{b.r0 + F.nu_lo, col0, -F.nu_lo, b.c0 - col0, b.c0 + b.TC + F.tau_hi - col0, wrow}
             : Window{b.r0 - F.nu_hi, col0, F.nu_hi, b.c0 - col0, b.c0 + b.TC - F.tau_lo - col0, wrow};
}
// byte offset in the window of this lane's path's source for a shift-0 element
template <bool ADJ>
__device__ __forceinline__ int path_offset(const FrameDev& F, const TileBox& b, const Window& w, int lane) {
  if (lane >= F.P) return 0;
  const int2 tn = __builtin_bit_cast(int2, ((gptr<const u64>)F.paths)[lane]);
  const int row = ADJ ? tn.y - F.nu_lo : F.nu_hi - tn.y, col = ADJ ? b.c0 + tn.x : b.c0 - tn.x;
  return 8 * (row * b.WC + col - w.col0);
}
template <int NJ, int CW>
__device__ __forceinline__ Lanes<NJ, CW> tile_lanes(const TileBox& b, int M, lptr<u64> win) {
  Lanes<NJ, CW> ln;
#pragma unroll
  for (int w = 0; w < CW; ++w) {
    ln.col[w] = b.ty < b.TY && b.tx + 64 * w < b.TC;
    ln.k8[w] = 8u * (uint32_t)(b.c0 + min(b.tx + 64 * w, b.TC - 1));
    ln.ov[w] = (uint32_t)((b.r0 + b.ty) * M) * 8u + ln.k8[w];
  }
  ln.full = b.TR / b.TY;
  ln.tail = b.ty < b.TR - ln.full * b.TY;
  // (whole row groups: the last one read is the last one held)
  ln.last = b.TR == ln.full * b.TY ? ln.full - 1 : ln.full;
  ln.la = (uint32_t)(uintptr_t)win + 8u * (uint32_t)(min(b.ty, b.TY - 1) * b.WC + b.tx);
  ln.lstep = 8u * (uint32_t)(b.TY * b.WC);
  ln.rstep = 8u * (uint32_t)(b.TY * M);
  return ln;
}
// f(i, j, w) for every element i of the thread, its row j and column w.  The row test is
// uniform but for the last row; the count is hidden from the optimiser at each use, or it
// would keep one mask per element in scalar registers.
template <int NJ, int CW, class F>
__device__ __forceinline__ void tile_each(const Lanes<NJ, CW>& ln, F f) {
  int full = ln.full;
  asm volatile("" : "+s"(full));
#pragma unroll
  for (int w = 0; w < CW; ++w) {
    if (ln.col[w]) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j < full)
          f(j * CW + w, j, w);
        else if (j == full && ln.tail)
          f(j * CW + w, j, w);
      }
    }
  }
}
template <int NJ, int CW>
__device__ __forceinline__ void tile_store(const Lanes<NJ, CW>& ln, __amdgpu_buffer_rsrc_t r,
                                           const float2* v) {
  tile_each(ln, [&](int i, int j, int w) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v[i]), r, ln.ov[w],
                                          (uint32_t)j * ln.rstep, 0);
  });
}

// acc = sum over the paths of coefficient x window element, for every element of the thread.
// Per path and step of 8 elements: 8 LDS reads of 8 bytes, 32 multiply-adds, at most 8 address
// adds.  The reads of the next step and the coefficients of the next path are issued before
// the products of the current step.  The path offsets sit one path per lane (off) and are
// fetched with readlane: scalar loads would share the LDS reads' wait counter out of order.
// ca: the coefficients of the first two paths (tile_first).
template <int NJ, int CW>
__device__ __forceinline__ void tile_first(const Lanes<NJ, CW>& t, int P, int M,
                                           __amdgpu_buffer_rsrc_t tab, float2 (&c)[2][CW]) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int w = 0; w < CW; ++w) c[i][w] = buf_ld2b(tab, t.k8[w], 8u * (uint32_t)(min(i, P - 1) * M));
}
template <int NJ, int CW>
__device__ __forceinline__ void tile_paths(const Lanes<NJ, CW>& t, int P, int M, int off,
                                           __amdgpu_buffer_rsrc_t tab, float2 (&ca)[2][CW],
                                           float2* acc) {
  constexpr int JS = kStepElems / CW < NJ ? kStepElems / CW : NJ;
  constexpr int STEPS = NJ / JS;   // 1 or 2
  const uint32_t M8 = 8u * (uint32_t)M;
  auto coef = [&](int p, float2* c) __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < CW; ++w) c[w] = buf_ld2b(tab, t.k8[w], (uint32_t)p * M8);
  };
  auto rd = [&](int p, int h, float2* v) __attribute__((always_inline)) {
    // (rows past the last one a thread may hold repeat it)
    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane(off, p);
#pragma unroll
    for (int i = 0; i < JS; ++i) {
      const uint32_t so = o + (uint32_t)min(h * JS + i, t.last) * t.lstep;
      const lptr<const u64> a = (lptr<const u64>)(uintptr_t)(t.la + so);
      v[i * CW] = __builtin_bit_cast(float2, a[0]);
      if (CW == 2) v[i * CW + 1] = __builtin_bit_cast(float2, a[64]);
    }
  };
  auto mac = [&](const float2* c, int h, const float2* v) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < JS; ++i)
#pragma unroll
      for (int w = 0; w < CW; ++w) cmacf(acc[(h * JS + i) * CW + w], c[w], v[i * CW + w]);
  };
  // coefficients two paths at a time, one pair ahead: a pair's products cover the table
  // read's round trip to L2 (one path ahead did not)
  float2 cb[2][CW];
  float2 va[JS * CW], vb[JS * CW];
  auto pair = [&](int p, float2 (&c)[2][CW]) __attribute__((always_inline)) {
    coef(min(p, P - 1), c[0]);
    coef(min(p + 1, P - 1), c[1]);
  };
  auto path = [&](int p, const float2* c, float2* v0, float2* v1) __attribute__((always_inline)) {
    const int pn = min(p + 1, P - 1);
    if (STEPS == 2) {
      rd(p, 1, v1);
      mac(c, 0, v0);
      rd(pn, 0, v0);
      mac(c, 1, v1);
    } else {
      rd(pn, 0, v1);
      mac(c, 0, v0);
    }
  };
  auto both = [&](int p, float2 (&c)[2][CW]) __attribute__((always_inline)) {
    path(p, c[0], va, vb);
    if (STEPS == 2)
      path(p + 1, c[1], va, vb);
    else
      path(p + 1, c[1], vb, va);
  };
  rd(0, 0, va);
  int p = 0;
  for (; p + 1 < P; p += 2) {
    pair(p + 2, cb);
    both(p, ca);
#pragma unroll
    for (int i = 0; i < 2 * CW; ++i) ca[i / CW][i % CW] = cb[i / CW][i % CW];
  }
  if (p < P) path(p, ca[0], va, vb);
}

template <int NE, int CW>
__device__ __forceinline__ void cg_tile_item(const FrameDev& F, int tile, int budget, const Bases& B,
                                             const LaunchCtx& L, float2* lds, float* red,
                                             float* s_out, int* s_ok) {
  constexpr int NJ = NE / CW;
  const FrameVecs V = frame_vecs(F, B);
  FrameState s = uniform_state(F.st);
  s.cn = uniform_f(s.cn);
  s.cn0 = uniform_f(s.cn0);
  s.alpha = uniform_f(s.alpha);
  s.beta = uniform_f(s.beta);
  s.rel = uniform_f(s.rel);
  if (s.status != OTFS_FRAME_RUNNING) return;
  const int M = F.M, N = F.N, P = F.P;
  const int64_t E = (int64_t)M * N;
  const TileBox box = tile_box<CW>(F, F.tk_nbr, F.tk_nbc, F.tk_tc, tile);
  const int TR = box.TR, TC = box.TC, TY = box.TY, WC = box.WC, WR = box.WR;
  const float lam = F.lam;
  // (the host's cut guarantees that the window and its rows' factors fit the LDS, and that a
  // last row group which only some threads hold reads past the window but inside the LDS)
  const lptr<u64> win = (lptr<u64>)lds;
  float2* const wrow = lds + WR * WC;
  const Window wh = tile_window<false>(F, box, wrow), wa = tile_window<true>(F, box, wrow + WR);
  {
    const GPairs wt = gpairs(F.wtab);
    for (int i = (int)threadIdx.x; i < 2 * WR; i += kBlock)
      wrow[i] = wt.f(mod_pos(i < WR ? wh.row0 + i : wa.row0 + i - WR, N));
  }
  const int lane = (int)threadIdx.x & 63;
  const int off_h = path_offset<false>(F, box, wh, lane), off_a = path_offset<true>(F, box, wa, lane);
  const Lanes<NJ, CW> ln = tile_lanes<NJ, CW>(box, M, win);
  const __amdgpu_buffer_rsrc_t rtab = buf_rsrc(F.rtab, (int64_t)P * M * 8);
  const __amdgpu_buffer_rsrc_t stab = buf_rsrc(F.stab, (int64_t)P * M * 8);
  const __amdgpu_buffer_rsrc_t rp = buf_rsrc(F.p0, E * 8), rt = buf_rsrc(F.t, E * 8);
  auto load = [&](__amdgpu_buffer_rsrc_t r, float2* v) __attribute__((always_inline)) {
    tile_each(ln, [&](int i, int j, int w) __attribute__((always_inline)) {
      v[i] = buf_ld2b(r, ln.ov[w], (uint32_t)j * ln.rstep);
    });
  };

  // ---- which tiles' rows and columns the two windows read ----
  bool need_h = false, need_a = false;
  if (lane < F.tk_T) {
    const TileBox o = tile_box<CW>(F, F.tk_nbr, F.tk_nbc, F.tk_tc, lane);
    need_h = cyc_meet(wh.row0, min(WR, N), o.r0, o.TR, N) && cyc_meet(wh.col0, min(WC, M), o.c0, o.TC, M);
    need_a = cyc_meet(wa.row0, min(WR, N), o.r0, o.TR, N) && cyc_meet(wa.col0, min(WC, M), o.c0, o.TC, M);
  }
  Meet m{F.slots, L.abort_flag, L.timeout, F.tk_T, tile, red, s_out, s_ok};
  enum { kMeetP = 0, kMeetT = 1, kMeetDot = 2, kMeetNorm = 3 };
  unsigned ep = 0, ep_norm = 0;   // epochs of this launch (the words are cleared before it)

  float2 x[NE], c[NE], p[NE], acc[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) x[i] = c[i] = p[i] = make_float2(0.f, 0.f);

  // the window's halo (with odd M: all of it), then the sums over the paths
  const bool even = (M & 1) == 0;
  auto own = [&](const float2* v, const Window& w) __attribute__((always_inline)) {
    if (!even) return;
    const uint32_t o = ln.la + 8u * (uint32_t)(w.orow * WC + w.ocol);
    tile_each(ln, [&](int i, int j, int q) __attribute__((always_inline)) {
      const lptr<u64> a = (lptr<u64>)(uintptr_t)(o + (uint32_t)j * ln.lstep);
      a[64 * q] = __builtin_bit_cast(u64, v[i]);
    });
  };
  float2 cf[2][CW];
  auto window = [&](__amdgpu_buffer_rsrc_t r, const Window& w) __attribute__((always_inline)) {
    if (even)
      window_dma(r, w, WR, WC, TR, TC, M, N, win);
    else
      window_fill(SrcShared{r}, w, WR, WC, M, N, win);
  };
  auto sums = [&](int off, __amdgpu_buffer_rsrc_t tab) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NE; ++i) acc[i] = make_float2(0.f, 0.f);
    tile_paths<NJ, CW>(ln, P, M, off, tab, cf, acc);
  };

  // how the tile's share ends: kRun (still running), kTimeout, kSave (leave the launch and
  // resume in the next one), or the frame's final status
  constexpr int kRun = -1, kTimeout = -2, kSave = -3;
  int end = kRun;
  bool xpend = false;   // x += alpha p is still to be applied to the result
  // the stop test on the residual norm cn_new after iteration s.iter, else beta
  auto next = [&](float cn_new, bool pend) __attribute__((always_inline)) {
    s.rel = uniform_f(sqrtf(cn_new / s.cn0));
    if (!isfinite(cn_new))
      end = OTFS_FRAME_NONFINITE;
    else if (F.tol > 0.f && s.rel <= F.tol)
      end = OTFS_FRAME_CONVERGED;
    else if (s.iter >= F.max_iters)
      end = OTFS_FRAME_CAPPED;
    xpend = pend;
    s.beta = uniform_f(cn_new / s.cn);
    s.cn = end == kRun ? cn_new : s.cn;
    s.pending = (pend ? 1 : 0) | 2;
  };

  bool start = !s.init;   // the pass forms b = H^H y (the initialisation of Algorithm 1)
  if (!start) {
    load(buf_rsrc(V.x, E * 8), x);
    load(buf_rsrc(F.c, E * 8), c);
    load(rp, p);
    // every tile has read the state before any of them can finish the frame and write it
    float zero;
    if (!meet<true, false>(m, kMeetNorm, ++ep_norm, true, 0.f, &zero)) end = kTimeout;
    if (end == kRun && s.refresh) {   // after the refresh launches: the true residual's norm
      s.refresh = 0;
      next(uniform_f((float)tile_sum_d<false>(F.part_d, F.ref_T)), false);
    }
  }
  // One straight-line body for the start (b = H^H y) and every iteration, left at its end
  // only: with exits or skips in the middle the compiler keeps a second copy of x, c and p.
  // A failed meeting or a breakdown sets `end`; what follows it is then without effect on x.
  int step = 0;
  if (end == kRun) do {
    // ---- A: the deferred updates, p' to the neighbours, t = H p' ----
    ++ep;
    const float al = (s.pending & 1) ? s.alpha : 0.f, be = (s.pending & 2) ? s.beta : 0.f;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      x[i] = axpyf(al, p[i], x[i]);
      p[i] = axpyf(be, p[i], c[i]);
    }
    float none;
    if (!start) {
      tile_store(ln, rp, p);
      own(p, wh);   // the window's last readers met twice since
      if (!meet<false, true>(m, kMeetP, ep, need_h, 0.f, &none)) end = kTimeout;
      tile_first<NJ, CW>(ln, P, M, rtab, cf);
      window(rp, wh);
      sums(off_h, rtab);
      tile_store(ln, rt, acc);
      // (the workgroup has met: nobody reads the window of p' any more)
      if (end == kRun && !meet<false, true>(m, kMeetT, ep, need_a, 0.f, &none,
                                            [&]() __attribute__((always_inline)) { own(acc, wa); }))
        end = kTimeout;
      tile_first<NJ, CW>(ln, P, M, stab, cf);
      window(rt, wa);
    } else {
      tile_first<NJ, CW>(ln, P, M, stab, cf);
      __syncthreads();   // the window rows' factors are in place
      if (V.ybf16)
        window_fill(SrcBf16{buf_rsrc(V.y, E * 4)}, wa, WR, WC, M, N, win);
      else
        window_fill(SrcBuf{buf_rsrc(V.y, E * 8)}, wa, WR, WC, M, N, win);
    }
    // ---- B: a = H^H t + lam p', Re(p'^H a), alpha.  At the start x = c = p = 0 and alpha = -1:
    // the same steps give c = H^H y exactly, and p = c follows with beta = 0. ----
    sums(off_a, stab);
    // What the thread does not hold stays zero.
    float part = 0.f, alpha = -1.f;
    int full = ln.full;
    asm volatile("" : "+s"(full));
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int j = i / CW;
      const bool held = ln.col[i % CW] && (j < full || (j == full && ln.tail));
      acc[i] = axpyf(lam, p[i], acc[i]);
      acc[i].x = held ? acc[i].x : 0.f;
      acc[i].y = held ? acc[i].y : 0.f;
      part = fmaf(p[i].x, acc[i].x, part);
      part = fmaf(p[i].y, acc[i].y, part);
    }
    if (!start && end == kRun) {
      float den;
      if (!meet<true, false>(m, kMeetDot, ep, true, part, &den)) end = kTimeout;
      alpha = uniform_f(s.cn / den);
      if (end == kRun && (!(den > 0.f) || !isfinite(alpha))) {   // x already holds x_{xi-1}
        xpend = false;
        end = (isfinite(den) && isfinite(s.cn)) ? OTFS_FRAME_BREAKDOWN : OTFS_FRAME_NONFINITE;
      }
    }
    // ---- C: c -= alpha a, ||c||^2 ----
    part = 0.f;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      c[i] = axpyf(-alpha, acc[i], c[i]);
      part = fmaf(c[i].x, c[i].x, part);
      part = fmaf(c[i].y, c[i].y, part);
    }
    float cn = 0.f;
    if (end == kRun && !meet<true, false>(m, kMeetNorm, ++ep_norm, true, part, &cn)) end = kTimeout;
    if (end == kRun) {
      if (start) {
        start = false;
        s.init = 1;
        s.iter = 0;
        s.pbuf = 0;
        s.pending = 0;
        s.cn = cn;
        s.cn0 = cn;
        s.alpha = 0.f;
        s.beta = 0.f;
        s.rel = cn > 0.f ? 1.f : 0.f;
        xpend = false;
        if (!(cn > 0.f)) end = cn == 0.f ? OTFS_FRAME_CONVERGED : OTFS_FRAME_NONFINITE;
      } else {
        ++step;
        ++s.iter;
        s.alpha = alpha;
        if (F.refresh_every > 0 && s.iter % F.refresh_every == 0 && s.iter < F.max_iters) {
          // leave the launch: the refresh launches form the true residual of x
          xpend = true;
          end = isfinite(cn) ? kSave : OTFS_FRAME_NONFINITE;
          s.refresh = end == kSave ? 1 : 0;
          s.pending = 0;
        } else {
          next(cn, true);
          if (end == kRun && step == budget) end = kSave;
        }
      }
    }
  } while (end == kRun);

  const bool saved = end == kSave;
  if (end != kTimeout) {
    if (saved ? s.refresh != 0 : xpend) {
#pragma unroll
      for (int i = 0; i < NE; ++i) x[i] = axpyf(s.alpha, p[i], x[i]);
    }
    tile_store(ln, buf_rsrc(V.x, E * 8), x);
    if (saved) {
      tile_store(ln, buf_rsrc(F.c, E * 8), c);
      tile_store(ln, rp, p);
      s.pbuf = 0;
    } else {
      s.pending = 0;
      if (V.sym != nullptr && F.qside > 0) {   // a rolled loop over the estimates just stored
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int n = ln.full + (ln.tail ? 1 : 0);
#pragma unroll 1
        for (int i = 0; i < n * CW; ++i) {
          const int w = CW == 2 ? i & 1 : 0, j = CW == 2 ? i >> 1 : i;
          if (!(w ? ln.col[CW - 1] : ln.col[0])) continue;
          const int64_t q = (int64_t)((w ? ln.ov[CW - 1] : ln.ov[0]) >> 3) + (int64_t)j * TY * M;
          V.sym[q] = decide(V.x[q], F.qscale, F.qside);
        }
      }
    }
  }
  if (tile == 0 && threadIdx.x == 0) {
    if (!saved) s.status = end == kTimeout ? OTFS_FRAME_TIMEOUT : end;
    *F.st = s;
    if (V.stats && !saved) *V.stats = otfs_frame_stats{s.iter, s.rel, s.status, F.tk_T};
  }
}

// S_p[k] of every frame with a cut: conj(R_p[k + tau]), past the row's end times
// W[nu] (below) or conj(W[nu]) (above): with it conj(D_{p,q}) W[l']^-n' = S_p[k], where l' and
// n' are the row and the wrap count of the gathered element, whose factor the window carries.
// Either way that is conj(h_p) e^{-j 2 pi nu k / (MN)}, R_p continued past its row: the wrapped
// entries are formed so in FP64 and rounded once, as those of R are (the product of the two FP32
// tables rounded three times).
__global__ __launch_bounds__(256) void k_tile_tables(const FrameDev* __restrict__ frames) {
  const FrameDev& F = frames[blockIdx.x];
  if (F.tk_T == 0 && F.ap_T == 0) return;
  const int M = F.M;
  const int64_t MN = (int64_t)M * F.N;
  for (int i = (int)(blockIdx.y * blockDim.x + threadIdx.x); i < F.P * M; i += (int)(gridDim.y * blockDim.x)) {
    const int p = i / M, k = i - p * M;
    const int2 tn = F.paths[p];
    const int K = k + tn.x;
    float2 c;
    if (K >= 0 && K < M) {
      c = F.rtab[p * M + K];
      c.y = -c.y;
    } else {
      const float2 h = F.gain[p];
      const double2 v = cmuld(make_double2((double)h.x, -(double)h.y), unit_phasor(-(int64_t)tn.y * k, MN));
      c = make_float2((float)v.x, (float)v.y);
    }
    F.stab[i] = c;
  }
}

// Work queues as in k_cg_fused; a queue entry is frame * kTileStride + tile.
template <int NE>
__global__ __launch_bounds__(kBlock, 2) void k_cg_tile(const FrameDev* __restrict__ frames,
                                                       const int32_t* __restrict__ qitems,
                                                       const int2* __restrict__ qrange,
                                                       unsigned* __restrict__ qhead, int ngroups,
                                                       int budget, Bases B, LaunchCtx L) {
  __shared__ float red[kWaves];
  __shared__ float s_out;
  __shared__ int s_ok, s_item;
  extern __shared__ float2 tile_lds[];
  // (the launch boundaries order this launch's data against other XCDs' writes)
  const int g = xcc_id();
  if (g < ngroups) {
    const int2 r = qrange[g];
    for (;;) {
      if (threadIdx.x == 0) {
        const unsigned j =
            __hip_atomic_fetch_add(&qhead[g], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_item = (int)j < r.y - r.x ? qitems[r.x + (int)j] : -1;
      }
      __syncthreads();
      const int it = __builtin_amdgcn_readfirstlane(s_item);
      __syncthreads();
      if (it < 0) break;
      // the descriptor by scalar loads: all that steers the iteration loop is then provably
      // uniform (a loop exit that may differ between lanes keeps a second copy of x, c and p)
      FrameDev F;
      {
        static_assert(sizeof(FrameDev) % 4 == 0, "copied by words");
        const kptr<const uint32_t> src = (kptr<const uint32_t>)(frames + it / kTileStride);
        uint32_t w[sizeof(FrameDev) / 4];
#pragma unroll
        for (int i = 0; i < (int)(sizeof(FrameDev) / 4); ++i) w[i] = src[i];
        __builtin_memcpy(&F, w, sizeof F);
      }
      if (F.tk_cw == 2)
        cg_tile_item<NE, 2>(F, it % kTileStride, budget, B, L, tile_lds, red, &s_out, &s_ok);
      else
        cg_tile_item<NE, 1>(F, it % kTileStride, budget, B, L, tile_lds, red, &s_out, &s_ok);
      __syncthreads();
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------------------
// Standalone H (H^H) over the frames with an apply cut: one workgroup per tile, its window read
// from memory once, the sums over the paths from LDS, the outputs stored.  Bound by memory
// (16 bytes per element plus the windows' halos, which the tiles of a frame, placed on one
// XCD, read through one L2).  Tiles of at most 8 elements per thread with windows of at most
// half the LDS: two workgroups per CU, so one copies while the other computes.
// ---------------------------------------------------------------------------------------
template <bool ADJ, int NE, int CW>
__device__ __forceinline__ void apply_tile(const FrameDev& F, int tile, const float2* in, float2* out,
                                           float2* lds) {
  constexpr int NJ = NE / CW;
  const TileBox box = tile_box<CW>(F, F.ap_nbr, F.ap_nbc, F.ap_tc, tile);
  const int64_t E = (int64_t)F.M * F.N;
  const lptr<u64> win = (lptr<u64>)lds;
  float2* const wrow = lds + box.WR * box.WC;
  Window w = tile_window<ADJ>(F, box, wrow);
  const int off = path_offset<ADJ>(F, box, w, (int)threadIdx.x & 63);
  const Lanes<NJ, CW> ln = tile_lanes<NJ, CW>(box, F.M, win);
  const __amdgpu_buffer_rsrc_t tab = buf_rsrc(ADJ ? F.stab : F.rtab, (int64_t)F.P * F.M * 8);
  float2 cf[2][CW], acc[NE];
  tile_first<NJ, CW>(ln, F.P, F.M, tab, cf);
  if (w.col0 < 0 || w.col0 + box.WC > F.M) {
    const GPairs wt = gpairs(F.wtab);
    for (int i = (int)threadIdx.x; i < box.WR; i += kBlock) wrow[i] = wt.f(mod_pos(w.row0 + i, F.N));
    __syncthreads();
  }
  const __amdgpu_buffer_rsrc_t rin = buf_rsrc(in + F.off, E * 8);
  // 16-byte copies need pairs that start at even elements of a 16-byte aligned buffer
  if ((F.M & 1) == 0 && ((uintptr_t)(in + F.off) & 15u) == 0) {
    w.orow = box.WR;   // nothing of the window is in LDS yet
    window_dma(rin, w, box.WR, box.WC, 0, 0, F.M, F.N, win);
  } else {
    window_fill(SrcBuf{rin}, w, box.WR, box.WC, F.M, F.N, win);
  }
#pragma unroll
  for (int i = 0; i < NE; ++i) acc[i] = make_float2(0.f, 0.f);
  tile_paths<NJ, CW>(ln, F.P, F.M, off, tab, cf, acc);
  tile_store(ln, buf_rsrc(out + F.off, E * 8), acc);
}
template <bool ADJ>
__global__ __launch_bounds__(kBlock, 4) void k_apply_tile(const FrameDev* __restrict__ frames,
                                                          const int2* __restrict__ items, int nxcd,
                                                          const float2* __restrict__ in,
                                                          float2* __restrict__ out) {
  extern __shared__ float2 tile_lds[];
  const int2 it = items[xcd_item((int)gridDim.x, nxcd)];
  const FrameDev& F = frames[it.x];
  if (F.ap_cw == 2)
    apply_tile<ADJ, kTileElemsSmall, 2>(F, it.y, in, out, tile_lds);
  else
    apply_tile<ADJ, kTileElemsSmall, 1>(F, it.y, in, out, tile_lds);
}

hipError_t launch_apply_tile(bool adjoint, const FrameDev* frames, const int2* items, int nitems,
                             int nxcd, const float2* in, float2* out, int lds_bytes, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  if (lds_bytes > kApplyLdsBytes) return hipErrorInvalidValue;
  static std::atomic<uint64_t> done[2];
  const hipError_t e = lds_limit(adjoint ? reinterpret_cast<const void*>(&k_apply_tile<true>)
                                         : reinterpret_cast<const void*>(&k_apply_tile<false>),
                                 kApplyLdsBytes, done[adjoint ? 1 : 0]);
  if (e != hipSuccess) return e;
  if (adjoint)
    hipLaunchKernelGGL(k_apply_tile<true>, dim3(nitems), dim3(kBlock), lds_bytes, s, frames, items,
                       nxcd, in, out);
  else
    hipLaunchKernelGGL(k_apply_tile<false>, dim3(nitems), dim3(kBlock), lds_bytes, s, frames, items,
                       nxcd, in, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// The FP64 refresh on the tiles of the solve, for batches that run whole on register-resident
// tiles: u = y - H x (k_refresh_tile<false>), then c = H^H u - lam x and its
// FP64 partial norms (<true>); x, u and c in FP32, products and sums in FP64.
//
// Windows as in the applications, but without the wrap factors, which would round in FP32.  The
// factor of a wrapped gather depends on the output row alone, but for W[nu] of its path (H:
// W[l0]^n with l0 = l - nu; H^H: conj(D) carries W[l]^n itself), so a tile at the frame's edge
// runs its wrapped gathers first, times the row's factor once, and the others last; a lane's
// coefficient is zero in the passes that its column has no part in.
//
// One workgroup per CU: a tile's window copy, path loop and stores follow one another.  128
// frames of 1024 x 256 with 16 paths: 377 and 413 us against 627 and 567 us of the streaming
// launches, whose windows of whole rows hold three times their band (of 392: 276 without the
// path loop, 386 without the window copy; the vectors' 24 bytes per element alone take 146).
// On the applications' cut, two workgroups per CU, windows 4.5 times the tile: 434 and 466;
// elements read one path ahead: 411 and 447.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double2 ld_d2(__amdgpu_buffer_rsrc_t r, uint32_t vb, uint32_t sb) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, vb, sb, 0));
}
template <bool ADJ, int NJ, int CW, bool WRAPPED>
__device__ __forceinline__ void refresh_paths(const Lanes<NJ, CW>& t, const TileBox& b, const FrameDev& F,
                                              int off, int wrap, double2* acc) {
  const __amdgpu_buffer_rsrc_t tab = buf_rsrc(F.rtab64, (int64_t)F.P * F.M * 16);
  const int M = F.M, P = F.P;
  auto column = [&](int w) __attribute__((always_inline)) { return (int)(t.k8[w] >> 3); };
  // the coefficient of path p at the lane's column (ADJ: of the column it gathers from)
  auto coef = [&](int p, double2* c) __attribute__((always_inline)) {
    const int tau = ((kptr<const int>)F.paths)[2 * p];
#pragma unroll
    for (int w = 0; w < CW; ++w) {
      const int k = ADJ ? wrap_once(column(w) + tau, M) : column(w);
      c[w] = ld_d2(tab, 16u * (uint32_t)k, 16u * (uint32_t)(p * M));
    }
  };
  auto rd = [&](int p, float2* v) __attribute__((always_inline)) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane(off, p);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const lptr<const u64> a = (lptr<const u64>)(uintptr_t)(t.la + o + (uint32_t)min(j, t.last) * t.lstep);
      v[j * CW] = __builtin_bit_cast(float2, a[0]);
      if (CW == 2) v[j * CW + 1] = __builtin_bit_cast(float2, a[64]);
    }
  };
  auto mac = [&](int p, double2* c, const float2* v) __attribute__((always_inline)) {
    const int tau = ((kptr<const int>)F.paths)[2 * p];
#pragma unroll
    for (int w = 0; w < CW; ++w) {
      const int k = ADJ ? column(w) + tau : column(w) - tau;
      if (wrap < 0 ? k >= 0 : (wrap > 0 ? k < M : (k < 0 || k >= M))) c[w] = make_double2(0.0, 0.0);
      if (ADJ) c[w].y = -c[w].y;
    }
#pragma unroll
    for (int i = 0; i < NJ * CW; ++i)
      cmacd(acc[i], c[i % CW], make_double2((double)v[i].x, (double)v[i].y));
  };
  if constexpr (WRAPPED) {
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
      const int tau = ((kptr<const int>)F.paths)[2 * p], nu = ((kptr<const int>)F.paths)[2 * p + 1];
      const int s0 = ADJ ? b.c0 + tau : b.c0 - tau, s1 = s0 + b.TC - 1;   // columns gathered from
      if (wrap < 0 ? s0 >= 0 : s1 < M) continue;
      double2 c[CW];
      float2 v[NJ * CW];
      coef(p, c);
      rd(p, v);
      if (!ADJ) {
        double2 f = __builtin_bit_cast(double2, ((kptr<const u32x4>)F.wtab64)[nu < 0 ? nu + F.N : nu]);
        if (wrap > 0) f.y = -f.y;
#pragma unroll
        for (int w = 0; w < CW; ++w) c[w] = cmuld(c[w], f);
      }
      mac(p, c, v);
    }
  } else {
    double2 cn[CW];
    coef(0, cn);
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
      double2 c[CW];
      float2 v[NJ * CW];
#pragma unroll
      for (int w = 0; w < CW; ++w) c[w] = cn[w];
      coef(min(p + 1, P - 1), cn);
      rd(p, v);
      mac(p, c, v);
    }
  }
}
template <bool ADJ, int NE, int CW>
__device__ __forceinline__ void refresh_tile(const FrameDev& F, const FrameVecs& V, int tile, float2* lds,
                                             double* red) {
  constexpr int NJ = NE / CW;
  const TileBox box = tile_box<CW>(F, F.tk_nbr, F.tk_nbc, F.tk_tc, tile);
  const int64_t E = (int64_t)F.M * F.N;
  const lptr<u64> win = (lptr<u64>)lds;
  Window w = tile_window<ADJ>(F, box, nullptr);
  const int off = path_offset<ADJ>(F, box, w, (int)threadIdx.x & 63);
  const Lanes<NJ, CW> ln = tile_lanes<NJ, CW>(box, F.M, win);
  const float2* in = ADJ ? F.u : V.x;
  const __amdgpu_buffer_rsrc_t rin = buf_rsrc(in, E * 8);
  if ((F.M & 1) == 0 && ((uintptr_t)in & 15u) == 0) {
    w.orow = box.WR;
    window_dma(rin, w, box.WR, box.WC, 0, 0, F.M, F.N, win, false);
  } else {
    window_fill(SrcBuf{rin}, w, box.WR, box.WC, F.M, F.N, win, false);
  }
  // y or x of the tile, on its way during the path loop (together with the window: +40 us)
  float2 own[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) own[i] = make_float2(0.f, 0.f);
  if (!ADJ && V.ybf16) {
    tile_each(ln, [&](int i, int j, int c) __attribute__((always_inline)) {
      own[i] = load_y(V.y, (ln.ov[c] + (uint32_t)j * ln.rstep) >> 3, true);
    });
  } else {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(ADJ ? V.x : V.y, E * 8);
    tile_each(ln, [&](int i, int j, int c) __attribute__((always_inline)) {
      own[i] = buf_ld2b(r, ln.ov[c], (uint32_t)j * ln.rstep);
    });
  }
  double2 acc[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) acc[i] = make_double2(0.0, 0.0);
  // wrapped gathers: the sums W[l] hi + conj(W[l]) lo as (hi W[l]^2 + lo) conj(W[l])
  const int c1 = box.c0 + box.TC - 1;
  const bool lo = ADJ ? box.c0 + F.tau_lo < 0 : box.c0 - F.tau_hi < 0;
  const bool hi = ADJ ? c1 + F.tau_hi >= F.M : c1 - F.tau_lo >= F.M;
  if (lo || hi) {
    auto rows = [&](bool square) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int l = min(box.r0 + box.ty + j * box.TY, F.N - 1);
        double2 f = __builtin_bit_cast(double2, ((gptr<const u32x4>)F.wtab64)[l]);
        f = square ? cmuld(f, f) : make_double2(f.x, -f.y);
#pragma unroll
        for (int c = 0; c < CW; ++c) acc[j * CW + c] = cmuld(acc[j * CW + c], f);
      }
    };
    if (hi) {
      refresh_paths<ADJ, NJ, CW, true>(ln, box, F, off, 1, acc);
      rows(true);
    }
    if (lo) refresh_paths<ADJ, NJ, CW, true>(ln, box, F, off, -1, acc);
    rows(false);
  }
  refresh_paths<ADJ, NJ, CW, false>(ln, box, F, off, 0, acc);
  float2 res[NE];
  if (ADJ) {
    const double lam = (double)F.lam;
#pragma unroll
    for (int i = 0; i < NE; ++i)
      res[i] = make_float2((float)(acc[i].x - lam * (double)own[i].x), (float)(acc[i].y - lam * (double)own[i].y));
    tile_store(ln, buf_rsrc(F.c, E * 8), res);
    double s = 0.0;
    tile_each(ln, [&](int i, int, int) __attribute__((always_inline)) {
      s = fma((double)res[i].x, (double)res[i].x, s);
      s = fma((double)res[i].y, (double)res[i].y, s);
    });
    s = block_sum_d(s, red);
    if (threadIdx.x == 0) F.part_d[tile] = s;
  } else {
#pragma unroll
    for (int i = 0; i < NE; ++i)
      res[i] = make_float2((float)((double)own[i].x - acc[i].x), (float)((double)own[i].y - acc[i].y));
    tile_store(ln, buf_rsrc(F.u, E * 8), res);
  }
}
// The launch boundaries order these kernels against the fused launches: no fence inside.
template <bool ADJ, int NE>
__global__ __launch_bounds__(kBlock, 2) void k_refresh_tile(const FrameDev* __restrict__ frames,
                                                            const int2* __restrict__ items, int nxcd,
                                                            Bases B, unsigned* qhead, int nq) {
  __shared__ double red[kWaves];
  extern __shared__ float2 tile_lds[];
  const int2 it = items[xcd_item((int)gridDim.x, nxcd)];
  const FrameDev& F = frames[it.x];
  if (!ADJ) {   // for the next fused launch of the solve
    if (blockIdx.x == 0 && (int)threadIdx.x < nq) qhead[threadIdx.x] = 0u;
    if (it.y == 0 && (int)threadIdx.x < kTileMeets * F.tk_T) F.slots[threadIdx.x] = 0ull;
  }
  if (F.st->refresh == 0 || F.st->status != OTFS_FRAME_RUNNING) return;
  const FrameVecs V = frame_vecs(F, B);
  if (F.tk_cw == 2)
    refresh_tile<ADJ, NE, 2>(F, V, it.y, tile_lds, red);
  else
    refresh_tile<ADJ, NE, 1>(F, V, it.y, tile_lds, red);
}

template <int NE>
hipError_t refresh_tiles(const FrameDev* frames, const int2* items, int nitems, int nxcd, Bases bases,
                         unsigned* qhead, int nq, int lds_bytes, hipStream_t s) {
  const void* fns[] = {reinterpret_cast<const void*>(&k_refresh_tile<false, NE>),
                       reinterpret_cast<const void*>(&k_refresh_tile<true, NE>)};
  for (const void* fn : fns) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_refresh_tile<false, NE>), dim3(nitems), dim3(kBlock), lds_bytes, s, frames, items,
                     nxcd, bases, qhead, nq);
  hipLaunchKernelGGL((k_refresh_tile<true, NE>), dim3(nitems), dim3(kBlock), lds_bytes, s, frames, items,
                     nxcd, bases, qhead, nq);
  return hipGetLastError();
}
hipError_t launch_refresh_tile(int kind, const FrameDev* frames, const int2* items, int nitems, int nxcd,
                               Bases bases, unsigned* qhead, int nq, int lds_bytes, hipStream_t s) {
  return kind == kKindTile
             ? refresh_tiles<kTileElems>(frames, items, nitems, nxcd, bases, qhead, nq, lds_bytes, s)
             : refresh_tiles<kTileElemsSmall>(frames, items, nitems, nxcd, bases, qhead, nq, lds_bytes, s);
}

hipError_t launch_tile_tables(const FrameDev* frames, int nframes, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_tables, dim3((unsigned)nframes, 8), dim3(256), 0, s, frames);
  return hipGetLastError();
}

const void* tile_fn(int kind) {
  return kind == kKindTile ? reinterpret_cast<const void*>(&k_cg_tile<kTileElems>)
                           : reinterpret_cast<const void*>(&k_cg_tile<kTileElemsSmall>);
}

void launch_tile(int kind, const FrameDev* frames, const int32_t* qitems, const int2* qrange,
                 unsigned* qhead, int ngroups, int grid, int budget, const Bases& bases,
                 unsigned* abort_flag, uint64_t timeout, int lds_bytes, hipStream_t s) {
  const LaunchCtx L{abort_flag, timeout, 1};
  if (kind == kKindTile)
    hipLaunchKernelGGL(k_cg_tile<kTileElems>, dim3(grid), dim3(kBlock), lds_bytes, s, frames, qitems,
                       qrange, qhead, ngroups, budget, bases, L);
  else
    hipLaunchKernelGGL(k_cg_tile<kTileElemsSmall>, dim3(grid), dim3(kBlock), lds_bytes, s, frames,
                       qitems, qrange, qhead, ngroups, budget, bases, L);
}

}  // namespace otfs
