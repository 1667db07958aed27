// Device-side building blocks of the tesseract encoding, shared by the
// standalone encoding kernels and the fused encoding + MLP kernels.
#pragma once
#include <hip/hip_fp16.h>

#include <utility>

#include "common.h"

namespace fh {

// The F values of a table row whose first element is at offset e.
template <int F, typename T>
struct RowLoad;

template <>
struct RowLoad<1, float> {
  static __device__ __forceinline__ void load(const float* t, int64_t e, float* o) { o[0] = t[e]; }
};
template <>
struct RowLoad<2, float> {
  static __device__ __forceinline__ void load(const float* t, int64_t e, float* o) {
    const float2 v = *reinterpret_cast<const float2*>(t + e);
    o[0] = v.x;
    o[1] = v.y;
  }
};
template <>
struct RowLoad<4, float> {
  static __device__ __forceinline__ void load(const float* t, int64_t e, float* o) {
    const float4 v = *reinterpret_cast<const float4*>(t + e);
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
  }
};
template <>
struct RowLoad<8, float> {
  static __device__ __forceinline__ void load(const float* t, int64_t e, float* o) {
    const float4 a = *reinterpret_cast<const float4*>(t + e);
    const float4 b = *reinterpret_cast<const float4*>(t + e + 4);
    o[0] = a.x, o[1] = a.y, o[2] = a.z, o[3] = a.w;
    o[4] = b.x, o[5] = b.y, o[6] = b.z, o[7] = b.w;
  }
};
template <>
struct RowLoad<1, __half> {
  static __device__ __forceinline__ void load(const __half* t, int64_t e, float* o) {
    o[0] = __half2float(t[e]);
  }
};
template <>
struct RowLoad<2, __half> {
  static __device__ __forceinline__ void load(const __half* t, int64_t e, float* o) {
    const __half2 v = *reinterpret_cast<const __half2*>(t + e);
    const float2 f = __half22float2(v);
    o[0] = f.x;
    o[1] = f.y;
  }
};
template <>
struct RowLoad<4, __half> {
  static __device__ __forceinline__ void load(const __half* t, int64_t e, float* o) {
    const uint2 raw = *reinterpret_cast<const uint2*>(t + e);
    const __half2* h = reinterpret_cast<const __half2*>(&raw);
    const float2 a = __half22float2(h[0]), b = __half22float2(h[1]);
    o[0] = a.x, o[1] = a.y, o[2] = b.x, o[3] = b.y;
  }
};
template <>
struct RowLoad<8, __half> {
  static __device__ __forceinline__ void load(const __half* t, int64_t e, float* o) {
    const uint4 raw = *reinterpret_cast<const uint4*>(t + e);
    const __half2* h = reinterpret_cast<const __half2*>(&raw);
    for (int i = 0; i < 4; ++i) {
      const float2 a = __half22float2(h[i]);
      o[2 * i] = a.x;
      o[2 * i + 1] = a.y;
    }
  }
};

// Rows e and e + F of a table (two consecutive rows) in one load of 2F
// elements, at most 16 bytes; the address is aligned to a row only.
template <int F, typename T>
constexpr bool wide_pair() {
  return 2 * F * (int)sizeof(T) <= 16;
}

template <int F, typename T>
struct __attribute__((packed, aligned(F * sizeof(T)))) TwoRows {
  T v[2 * F];
};

__device__ __forceinline__ float row_value(float x) { return x; }
__device__ __forceinline__ float row_value(_Float16 x) { return (float)x; }
template <typename T>
struct RowElem {
  typedef T type;
};
template <>
struct RowElem<__half> {
  typedef _Float16 type;
};

template <int F, typename T>
__device__ __forceinline__ void load_two_rows(const T* t, int64_t e, float* a, float* b) {
  typedef typename RowElem<T>::type E;
  const TwoRows<F, E> r = *reinterpret_cast<const TwoRows<F, E>*>(t + e);
#pragma unroll
  for (int k = 0; k < F; ++k) {
    a[k] = row_value(r.v[k]);
    b[k] = row_value(r.v[F + k]);
  }
}

// Forward of NL levels for one sample, rows layout: out[j][k] = sum_c w_c
// E[slot_c][k] of level lv[l[j]].  All NL * 8 directory loads are issued
// together, then all table loads, so the levels cost two memory latencies
// however many corners they have.  Where the second row of a pair is the next
// table row (every dense and active index) and the table is not in runs, a
// pair's two rows come in one load of up to 16 bytes: half the table loads,
// and the number of lines an instruction touches is what the vector memory
// path spends its time on.  Pairs without an active corner read the table's
// first rows, which stay in the cache (a query of the whole box has about half
// its corners there: sent to the rows at their rank instead, 2^20 random points
// took 2.39 ms).  An inactive corner counts as 0 whatever was read.  Measured,
// row by row before / this: 2^20 random points on 288^3 x 40 (16 levels, FP16)
// 1.80 / 1.46 ms, 1000 points (FP32) 28.9 / 22.5 us in the kernel, a served mix
// of renders and queries 11.9 / 9.1 ms.  Requires a table of at least two rows.
template <int NL, int F, typename T>
__device__ __forceinline__ void encode_rows(const GridDev& g, const LevelDev* lv,
                                            const int (&l)[NL], const float4 p,
                                            const T* __restrict__ table, float (&out)[NL][F]) {
  const bool active = g.active != 0;
  Cell c[NL];
  RowEntries q[NL];
  RowPairs s[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    c[j] = locate_cell(lv[l[j]], p);
    row_fetch(lv[l[j]], g.dir, active, c[j], q[j]);
  }
#pragma unroll
  for (int j = 0; j < NL; ++j) row_slots(lv[l[j]], active, c[j], q[j], s[j]);
  float e0[NL][8][F], e1[NL][8][F];
  if (wide_pair<F, T>() && g.next_row && g.tmask == 0) {
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const bool any = (s[j].v >> r) & 0x101u;
        const int64_t b = s[j].s[r] < g.last_pair ? s[j].s[r] : g.last_pair;
        load_two_rows<F, T>(table, (any ? b : 0) * F, e0[j][r], e1[j][r]);
      }
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        // a pair moved back from the table's end has its first row second, and
        // x + 1 sits where x would when x is inactive
        const bool moved = s[j].s[r] > g.last_pair, v0 = (s[j].v >> r) & 1u;
#pragma unroll
        for (int k = 0; k < F; ++k) {
          if (moved) e0[j][r][k] = e1[j][r][k];
          if (!v0) e1[j][r][k] = e0[j][r][k];
        }
      }
  } else {
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const bool v0 = (s[j].v >> r) & 1u, v1 = (s[j].v >> (8 + r)) & 1u;
        const int64_t s1 = pair_second(s[j].s[r], v0, s[j].hx, lv[l[j]].slot_off);
        RowLoad<F, T>::load(table, run_off((v0 ? s[j].s[r] : 0) * F, g.tmask), e0[j][r]);
        RowLoad<F, T>::load(table, run_off((v1 ? s1 : 0) * F, g.tmask), e1[j][r]);
      }
  }
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    float acc[F];
#pragma unroll
    for (int k = 0; k < F; ++k) acc[k] = 0.0f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const bool v0 = (s[j].v >> r) & 1u, v1 = (s[j].v >> (8 + r)) & 1u;
      const float wr = row_weight(c[j], r);
      const float w0 = wr * (1.0f - c[j].fx);
      const float w1 = wr * c[j].fx;
#pragma unroll
      for (int k = 0; k < F; ++k) {
        const float a = v0 ? e0[j][r][k] : 0.0f, b = v1 ? e1[j][r][k] : 0.0f;
        acc[k] += w0 * a + w1 * b;
      }
    }
#pragma unroll
    for (int k = 0; k < F; ++k) out[j][k] = acc[k];
  }
}

// Forward of one brick-ordered level for one sample: out[k] = sum_c w_c
// E[slot_c][k].  Invalid (inactive) corners get weight 0 and read row 0, so every
// load is unconditional.  (The rows order goes through encode_rows.)
// Requires a table with at least one row.  tmask: the table's run mask
// (run_off; F divides 16, so a row never straddles a run).
template <int F, typename T>
__device__ __forceinline__ void encode_brick_level(const LevelDev& d, const ulonglong2* dir,
                                                   bool active, const float4 p,
                                                   const T* __restrict__ table, float* out,
                                                   int64_t tmask) {
  int ix, iy, iz, it;
  float fx, fy, fz, ft;
  locate(p.x, d.rx, d.sx, ix, fx);
  locate(p.y, d.ry, d.sy, iy, fy);
  locate(p.z, d.rz, d.sz, iz, fz);
  locate(p.w, d.rt, d.st, it, ft);
  float acc[F];
#pragma unroll
  for (int k = 0; k < F; ++k) acc[k] = 0.0f;
  const int a = pair_axis<true>(ix, iy, iz, it);
  const float fa = pair_frac(a, fx, fy, fz, ft);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    float wr;
    int64_t s0, s1;
    bool v0, v1;
    corner_pair<true>(d, dir, active, ix, iy, iz, it, fx, fy, fz, ft, a, r, s0, s1, v0, v1, wr);
    float e0[F], e1[F];
    RowLoad<F, T>::load(table, run_off((v0 ? s0 : 0) * F, tmask), e0);
    RowLoad<F, T>::load(table, run_off((v1 ? s1 : 0) * F, tmask), e1);
    const float w0 = v0 ? wr * (1.0f - fa) : 0.0f;
    const float w1 = v1 ? wr * fa : 0.0f;
#pragma unroll
    for (int k = 0; k < F; ++k) acc[k] += w0 * e0[k] + w1 * e1[k];
  }
#pragma unroll
  for (int k = 0; k < F; ++k) out[k] = acc[k];
}

// Touched-segment flag of a gradient write at float index fidx: the segment of
// FHASH_TOUCH_FLOATS floats that holds it is flagged (a plain byte store; all
// writers store the same value).  Only floats at or after `tbeg` are tracked.
__device__ __forceinline__ void mark_touched(uint8_t* touch, int64_t tbeg, int64_t fidx) {
  if (touch != nullptr && fidx >= tbeg) touch[fidx / FHASH_TOUCH_FLOATS] = 1;
}

// One lane's share of a level's scatter-add, brick order.  The lane owns pair
// element e (the first or second corner of every corner pair, corner_pair) and
// feature f of one sample: 2F consecutive lanes own one sample, so the 2F
// atomics they issue together hit the two slots of one pair (8F contiguous
// bytes for x pairs inside a brick; 4F-byte halves a few rows apart inside one
// brick otherwise).  Atomics of one instruction that fall in the same 64-byte
// segment are performed as one memory transaction, which is what bounds the
// scatter on gfx950.
template <int F>
__device__ __forceinline__ void scatter_brick_lane(const LevelDev& d, const ulonglong2* dir,
                                                   bool active, const float4 p, int e, int f,
                                                   float gval, float* __restrict__ d_table,
                                                   uint8_t* touch, int64_t tbeg, int64_t gmask) {
  const Cell c = locate_cell(d, p);
  const int a = pair_axis<true>(c.x, c.y, c.z, c.t);
  const float fa = pair_frac(a, c.fx, c.fy, c.fz, c.ft);
  const float wx = e ? fa : 1.0f - fa;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    float wr;
    int64_t s0, s1;
    bool v0, v1;
    corner_pair<true>(d, dir, active, c.x, c.y, c.z, c.t, c.fx, c.fy, c.fz, c.ft, a, r, s0, s1,
                      v0, v1, wr);
    const int64_t s = e ? s1 : s0;
    if (e ? v1 : v0) {
      unsafeAtomicAdd(d_table + run_off(s * F, gmask) + f, wr * wx * gval);
      if (f == 0) mark_touched(touch, tbeg, s * F);  // F divides the segment: one flag per slot
    }
  }
}

// The value lane K of the caller's group of Q lanes holds (K a constant): a
// DPP move inside groups of 2 and 4, a swizzle inside groups of 8 and 16.
template <int Q, int K>
__device__ __forceinline__ int group_get(int x) {
  static_assert(Q == 2 || Q == 4 || Q == 8 || Q == 16, "group size");
  if constexpr (Q == 2)
    return __builtin_amdgcn_update_dpp(0, x, K ? 0xF5 : 0xA0, 0xF, 0xF, false);
  else if constexpr (Q == 4)
    return __builtin_amdgcn_update_dpp(0, x, K * 0x55, 0xF, 0xF, false);
  else
    return __builtin_amdgcn_ds_swizzle(x, (32 - Q) | (K << 5));
}
template <int Q, int K>
__device__ __forceinline__ float group_get(float x) {
  return __int_as_float(group_get<Q, K>(__float_as_int(x)));
}
template <int Q, int K>
__device__ __forceinline__ int64_t group_get(int64_t x) {
  const uint32_t lo = (uint32_t)group_get<Q, K>((int)(uint32_t)x);
  const uint32_t hi = (uint32_t)group_get<Q, K>((int)(x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// What a lane brings to the scatter of its own sample and level, rows layout.
template <int F>
struct ScatterLane {
  RowPairs p;  // p.v = 0: nothing to add
  float wr[8], fx, g[F];
  int64_t slot_off;
};

// Adjoint of encode_rows for one sample and level per lane: d_table[slot_c][k]
// += w_c g[k] with FP32 hardware atomics.  Each lane has looked its own cell
// up; pass K of 2F then has the 2F lanes of a group add the sample of the
// group's lane K, lane (e, f) its pair element e and feature f, so the 2F
// atomics of a pair fall in one or two 64-byte segments: atomics of one
// instruction into one segment are performed as one memory transaction, which
// is what bounds the scatter on gfx950.  Looking the cell up once and handing
// the slots round takes the place of a lookup by every lane in every pass
// (2F times the directory loads, each waited for): the fused training kernel of
// 2^18 samples (16 levels, F = 2, FP32) took 1.87 ms so and takes 1.58, of 2^20
// samples (FP16 decoder) 6.31 and 5.62, of 20,011 samples at F = 4 295 and 234
// us.  Every lane of the wave calls it.
template <int F, int K>
__device__ __forceinline__ void scatter_pass(const GridDev& gd, const ScatterLane<F>& s, int e,
                                             int f, float* __restrict__ d_table) {
  constexpr int Q = 2 * F;
  const uint32_t v = (uint32_t)group_get<Q, K>((int)s.p.v);
  const float fx = group_get<Q, K>(s.fx);
  const float wx = e ? fx : 1.0f - fx;
  float g = group_get<Q, K>(s.g[0]);
#pragma unroll
  for (int q = 1; q < F; ++q) {
    const float t = group_get<Q, K>(s.g[q]);
    if (f == q) g = t;
  }
  uint32_t hx = 0;
  int64_t off = 0;
  if (!gd.next_row) {  // hashed levels
    hx = (uint32_t)group_get<Q, K>((int)s.p.hx);
    off = group_get<Q, K>(s.slot_off);
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t s0 = group_get<Q, K>(s.p.s[r]);
    const float w = group_get<Q, K>(s.wr[r]);
    if ((v >> (8 * e + r)) & 1u) {
      const int64_t sl = e ? pair_second(s0, (v >> r) & 1u, hx, off) : s0;
      unsafeAtomicAdd(d_table + run_off(sl * F, gd.gmask) + f, w * wx * g);
      if (f == 0) mark_touched(gd.touch, gd.touch_begin, sl * F);  // one flag per slot
    }
  }
}

template <int F, int... K>
__device__ __forceinline__ void scatter_passes(const GridDev& gd, const ScatterLane<F>& s, int e,
                                               int f, float* __restrict__ d_table,
                                               std::integer_sequence<int, K...>) {
  (scatter_pass<F, K>(gd, s, e, f, d_table), ...);
}

// own: the lane has a sample and a level to add (with gradient g); the others
// only help.
template <int F>
__device__ __forceinline__ void scatter_rows(const GridDev& gd, const LevelDev& d, const float4 p,
                                             bool own, const float (&g)[F],
                                             float* __restrict__ d_table) {
  ScatterLane<F> s;
  s.p.v = 0;
  s.p.hx = 0;
  s.fx = 0.0f;
  s.slot_off = 0;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    s.p.s[r] = 0;
    s.wr[r] = 0.0f;
  }
#pragma unroll
  for (int k = 0; k < F; ++k) s.g[k] = g[k];
  if (own) {
    const Cell c = locate_cell(d, p);
    RowEntries q;
    row_fetch(d, gd.dir, gd.active != 0, c, q);
    row_slots(d, gd.active != 0, c, q, s.p);
    s.fx = c.fx;
    s.slot_off = d.slot_off;
#pragma unroll
    for (int r = 0; r < 8; ++r) s.wr[r] = row_weight(c, r);
  }
  const int lane = threadIdx.x & (2 * F - 1);
  scatter_passes<F>(gd, s, lane / F, lane % F, d_table,
                    std::make_integer_sequence<int, 2 * F>());
}

}  // namespace fh
