// Scatter-add of the coarsest levels' encoding gradient through LDS.  The
// backward calls leave the gradient of levels 0 .. g.coarse - 1 (value k of
// sample s and level l at grad[l * level_step + s * sample_step + k]) to this
// kernel instead of adding it into the table.  Each workgroup takes one
// level and a contiguous chunk of the batch (neighbours in space when the batch is
// sorted), finds the box of the level's vertices its samples touch, sums the
// 16 corner contributions of every sample into an LDS image of that box, and
// adds the box into the table gradient with one atomic per touched vertex and
// feature.  At the coarse levels a vertex collects the contributions of many
// samples, so the memory-side atomic requests, which bound the scatter, drop
// from one per sample, corner and instruction to one per vertex and chunk.  A
// chunk whose box does not fit the LDS image is retried in kParts parts, and a
// part that still does not fit adds its samples directly.
// The sum over samples is the adjoint of the quadrilinear blend (Sec. 3.2.3),
// reordered: the same result up to FP32 summation order.
#include <climits>
#include <type_traits>
#include <utility>

#include "common.h"
#include "encode_dev.h"
#include "kernels.h"

namespace fh {

namespace {

constexpr int kWhole = 4096;  // floats of a level that can be the box itself
constexpr int kThreads = 1024;  // 16 waves: the loops below wait on L2 latency
constexpr int kChunk = 2048;    // samples per workgroup, at most
constexpr int kChunkMin = 256;  // and at least: a box is cleared and added per chunk
constexpr int kUnroll = 2;      // independent loads in flight per thread (4 take 4 more registers)
constexpr int kParts = 4;       // a chunk whose box does not fit is retried in 4 parts
constexpr int kTries = 3;       // compare-and-swaps before the float atomic
constexpr int kCap = kCoarseFloats;  // floats of the LDS image (with the reduction slots, under 64 KiB)

// Slot of vertex (x, y, z, t) of a rows-ordered level: dense, hashed, or
// through the rank directory (valid = false for an inactive vertex).  Reads
// only the directory entry that holds x.
__device__ __forceinline__ int64_t vertex_slot(const LevelDev& d, const ulonglong2* dir,
                                               bool active, int t, int z, int y, int x,
                                               bool& valid) {
  if (d.hash_bits) {
    const uint32_t yzt = (uint32_t)y * 2654435761u ^ (uint32_t)z * 805459861u ^
                         (uint32_t)t * 3674653429u;
    const uint32_t mask = (d.hash_bits >= 32) ? 0xffffffffu : ((1u << d.hash_bits) - 1u);
    valid = true;
    return d.slot_off + spatial_hash((uint32_t)x, yzt, mask);
  }
  if (!active) {
    valid = true;
    return d.slot_off + ((int64_t)(t * d.rz + z) * d.ry + y) * d.rx + x;
  }
  const int32_t tz = t * d.rz + z;
  const ulonglong2 e = dir[d.dir_off + (int64_t)((tz * d.wv + (x >> 6)) * d.ry + y)];
  return entry_slot(e, x & 63, d.slot_off, valid);
}

// The value lane K of the caller's row of 16 lanes holds.
template <int K>
__device__ __forceinline__ int row_get(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x150 + K, 0xF, 0xF, false);
}
template <int K>
__device__ __forceinline__ float row_get(float x) {
  return __int_as_float(row_get<K>(__float_as_int(x)));
}

template <typename Fn, int... U>
__device__ __forceinline__ void each(Fn& fn, std::integer_sequence<int, U...>) {
  (fn(std::integral_constant<int, U>{}), ...);
}

// Adds the F values of run to the vertex's floats at `at` in LDS (8-byte aligned
// for F > 1).  A float atomic in LDS is performed lane after lane: with
// ds_add_f32 the sums of six levels of a sorted batch of 2^20 took 875 us, with
// integer atomics in their place 376.  So the sum is written by compare-and-swap
// of the bits, two features at a time, and after kTries only the lanes whose
// vertex others kept changing use the float atomic: 601 us with one try, 510 with
// three, 508 with six; levels of 16 to 2,760 vertices, F = 1, 65,537 samples:
// 39.2 us with float atomics, 33.3 now.
template <int F>
__device__ __forceinline__ void lds_add(float* at, const float* run) {
  if constexpr (F == 1) {
    unsigned* p = reinterpret_cast<unsigned*>(at);
    unsigned was = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll 1
    for (int t = 0; t < kTries; ++t)
      if (__hip_atomic_compare_exchange_strong(
              p, &was, __float_as_uint(__uint_as_float(was) + run[0]), __ATOMIC_RELAXED,
              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
        return;
    atomicAdd(at, run[0]);
  } else {
    unsigned long long* p = reinterpret_cast<unsigned long long*>(at);
    unsigned long long was[F / 2];
#pragma unroll
    for (int k = 0; k < F / 2; ++k)
      was[k] = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    bool lost[F / 2];
#pragma unroll
    for (int k = 0; k < F / 2; ++k) lost[k] = true;
    bool any = true;
#pragma unroll 1
    for (int t = 0; t < kTries && any; ++t) {
      any = false;
#pragma unroll
      for (int k = 0; k < F / 2; ++k)
        if (lost[k]) {
          const unsigned a = __float_as_uint(__uint_as_float((unsigned)was[k]) + run[2 * k]);
          const unsigned b =
              __float_as_uint(__uint_as_float((unsigned)(was[k] >> 32)) + run[2 * k + 1]);
          lost[k] = !__hip_atomic_compare_exchange_strong(
              p + k, was + k, (unsigned long long)b << 32 | a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
              __HIP_MEMORY_SCOPE_WORKGROUP);
          any = any || lost[k];
        }
    }
#pragma unroll
    for (int k = 0; k < F / 2; ++k)
      if (lost[k]) {
        atomicAdd(at + 2 * k, run[2 * k]);
        atomicAdd(at + 2 * k + 1, run[2 * k + 1]);
      }
  }
}

// Two workgroups (32 waves) to a CU take 64 registers a thread: 2^20 samples, nine
// levels, F = 2: 801 us with 68 registers and one workgroup, 670 with two; 2^18:
// 214 and 188.  For F = 4 the spills take it back (123 and 125 us).
template <int F>
__global__ void __launch_bounds__(kThreads, F <= 2 ? 8 : 4)
    coarse_scatter_kernel(GridDev g, const float4* __restrict__ pos, int64_t n,
                          const float* __restrict__ grad, int64_t level_step,
                          int64_t sample_step, int chunk, float* __restrict__ d_table) {
  extern __shared__ __align__(16) float acc[];  // kCap floats
  __shared__ int red[8][kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  const int cnt = (int)((n - c0) < chunk ? (n - c0) : chunk);
  const bool active = g.active != 0;
  {
    const int l = blockIdx.y;  // one level per workgroup row of the grid
    const LevelDev& d = g.lv[l];
    const float* gl = grad + l * level_step;
    const bool whole = chunk < kChunk && (int64_t)d.rx * d.ry * d.rz * d.rt * F <= kWhole;
    int nparts = 1;
    for (int part = 0; part < nparts; ++part) {
    // samples s0 .. s0 + bn - 1: the chunk, or one of its parts
    const int b0 = (int)((int64_t)cnt * part / nparts);
    const int bn = (int)((int64_t)cnt * (part + 1) / nparts) - b0;
    const int64_t s0 = c0 + b0;
    if (bn == 0) continue;  // a part of a chunk shorter than kParts samples
    // the vertex box: the cells the range's samples fall in (per-axis minimum and
    // maximum), or the whole level for a short batch on a level of at most 16 KiB,
    // where clearing and reading the image costs less than the pass that finds
    // the bounds (512 samples, 16 levels: 19.5 us with the pass, 16.9 without;
    // full chunks of a sorted batch of 2^18 take 212.5 and 212.9, so they keep
    // the smaller box)
    int blo[4] = {0, 0, 0, 0}, ext[4] = {d.rx, d.ry, d.rz, d.rt};
    if (!whole) {
      int lo[4] = {INT_MAX, INT_MAX, INT_MAX, INT_MAX}, hi[4] = {-1, -1, -1, -1};
      for (int i = tid; i < bn; i += kThreads) {
        const Cell c = locate_cell(d, pos[s0 + i]);
        const int cc[4] = {c.x, c.y, c.z, c.t};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          lo[k] = min(lo[k], cc[k]);
          hi[k] = max(hi[k], cc[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        for (int o = 32; o > 0; o >>= 1) {
          lo[k] = min(lo[k], __shfl_xor(lo[k], o, 64));
          hi[k] = max(hi[k], __shfl_xor(hi[k], o, 64));
        }
      if (lane == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          red[k][wid] = lo[k];
          red[4 + k][wid] = hi[k];
        }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        int a = red[k][0], b = red[4 + k][0];
        for (int w = 1; w < kThreads / 64; ++w) {
          a = min(a, red[k][w]);
          b = max(b, red[4 + k][w]);
        }
        blo[k] = a;
        ext[k] = b - a + 2;  // vertices a .. b + 1
      }
      __syncthreads();  // red is rewritten by the next range
    }
    const int64_t V = (int64_t)ext[0] * ext[1] * ext[2] * ext[3];
    if (V * F <= kCap) {
      for (int i = tid; i < (int)V * F; i += kThreads) acc[i] = 0.0f;
      __syncthreads();
      // lane group of 16: one corner per lane (bits x, y, z, t), the group
      // walking a contiguous run of the range's samples and summing in
      // registers while its vertex stays the same (neighbours in a sorted batch
      // often share the cell), so an LDS add is issued per change of vertex.  The
      // four groups of a wave walk runs far apart, so that they seldom add to the
      // same vertex at once (510 -> 499 us).  Lane c of a group locates sample c
      // of the next 16 and the samples are handed round by row broadcasts, for
      // every lane of the group locating each sample: 499 -> 457 us (2^18 samples,
      // five levels: 132 -> 117)
      const int cr = tid & 15;
      // weight of the corner along an axis: f or 1 - f as f * sgn + one
      const float sx = cr & 1 ? 1.0f : -1.0f, qx = cr & 1 ? 0.0f : 1.0f;
      const float sy = cr & 2 ? 1.0f : -1.0f, qy = cr & 2 ? 0.0f : 1.0f;
      const float sz = cr & 4 ? 1.0f : -1.0f, qz = cr & 4 ? 0.0f : 1.0f;
      const float st = cr & 8 ? 1.0f : -1.0f, qt = cr & 8 ? 0.0f : 1.0f;
      const int ny = ext[0], nz = ny * ext[1], nt = nz * ext[2];  // box strides
      const int corner =
          (cr & 1) + (cr & 2 ? ny : 0) + (cr & 4 ? nz : 0) + (cr & 8 ? nt : 0);
      constexpr int kGroups = kThreads / 16;
      const int per = (bn + kGroups - 1) / kGroups;
      const int ib = (((tid >> 4) & 3) * (kGroups / 4) + wid) * per, ie = min(bn, ib + per);
      int cur = -1;
      float run[F];
#pragma unroll
      for (int k = 0; k < F; ++k) run[k] = 0.0f;
      for (int j0 = 0; j0 < per; j0 += 16) {  // the same trips in every lane
        const int i = ib + j0 + cr;
        const bool mine = i < ie;
        Cell c = {};
        float gr[F];
        if (mine) c = locate_cell(d, pos[s0 + i]);
#pragma unroll
        for (int k = 0; k < F; ++k) gr[k] = mine ? gl[(s0 + i) * sample_step + k] : 0.0f;
        const int at = mine ? (c.x - blo[0]) + (c.y - blo[1]) * ny + (c.z - blo[2]) * nz +
                                  (c.t - blo[3]) * nt
                            : -1;
        auto sample = [&](auto u) {  // sample j0 + u of the group's run
          constexpr int U = decltype(u)::value;
          if (j0 + U >= per) return;
          const int a = row_get<U>(at);
          const float w = (fmaf(row_get<U>(c.fx), sx, qx) * fmaf(row_get<U>(c.fy), sy, qy)) *
                          (fmaf(row_get<U>(c.fz), sz, qz) * fmaf(row_get<U>(c.ft), st, qt));
          float gu[F];
#pragma unroll
          for (int k = 0; k < F; ++k) gu[k] = row_get<U>(gr[k]);
          const int li = a + corner;
          if (a >= 0 && li != cur) {
            if (cur >= 0) lds_add<F>(acc + cur * F, run);
            cur = li;
#pragma unroll
            for (int k = 0; k < F; ++k) run[k] = 0.0f;
          }
#pragma unroll
          for (int k = 0; k < F; ++k) run[k] += w * gu[k];
        };
        each(sample, std::make_integer_sequence<int, 16>{});
      }
      if (cur >= 0) lds_add<F>(acc + cur * F, run);
      __syncthreads();
      // the box into the table: x fastest, so neighbouring lanes add into
      // neighbouring slots of a vertex row; kUnroll directory loads in flight
      for (int v0 = tid; v0 < (int)V; v0 += kThreads * kUnroll) {
        float val[kUnroll][F];
        int64_t sv[kUnroll];
        bool add[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          const int v = v0 + u * kThreads;
          bool any = false;
#pragma unroll
          for (int k = 0; k < F; ++k) {
            val[u][k] = v < (int)V ? acc[v * F + k] : 0.0f;
            any = any || val[u][k] != 0.0f;
          }
          add[u] = false;
          sv[u] = 0;
          if (any) {
            int r = v;
            const int x = blo[0] + r % ext[0];
            r /= ext[0];
            const int y = blo[1] + r % ext[1];
            r /= ext[1];
            const int z = blo[2] + r % ext[2];
            const int t = blo[3] + r / ext[2];
            sv[u] = vertex_slot(d, g.dir, active, t, z, y, x, add[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
          if (add[u]) {
#pragma unroll
            for (int k = 0; k < F; ++k)
              unsafeAtomicAdd(d_table + run_off(sv[u] * F, g.gmask) + k, val[u][k]);
            mark_touched(g.touch, g.touch_begin, sv[u] * F);
          }
      }
      __syncthreads();  // the next range clears acc
    } else if (nparts == 1) {
      nparts = kParts;  // the same decision in every thread: retry in parts
      part = -1;
    } else {
      // straight into the table, one lane per sample, corner and feature, so
      // that the lanes of an atomic instruction cover both rows of a corner
      // pair and every feature (one request per pair and sample)
      constexpr int Q = 16 * F;
      const int k = tid % F, cr = (tid / F) & 15;
      const int ox = cr & 1, oy = (cr >> 1) & 1, oz = (cr >> 2) & 1, ot = (cr >> 3) & 1;
      for (int i = tid / Q; i < bn; i += kThreads / Q) {
        const float4 p = pos[s0 + i];
        int cx, cy, cz, ct;
        float fx, fy, fz, ft;
        locate(p.x, d.rx, d.sx, cx, fx);
        locate(p.y, d.ry, d.sy, cy, fy);
        locate(p.z, d.rz, d.sz, cz, fz);
        locate(p.w, d.rt, d.st, ct, ft);
        const float w = ((ox ? fx : 1.0f - fx) * (oy ? fy : 1.0f - fy)) *
                        ((oz ? fz : 1.0f - fz) * (ot ? ft : 1.0f - ft));
        bool valid;
        const int64_t sl = vertex_slot(d, g.dir, active, ct + ot, cz + oz, cy + oy, cx + ox, valid);
        if (valid) {
          unsafeAtomicAdd(d_table + run_off(sl * F, g.gmask) + k, w * gl[(s0 + i) * sample_step + k]);
          if (k == 0) mark_touched(g.touch, g.touch_begin, sl * F);
        }
      }
    }
    }
  }
}

template <int F>
hipError_t launch_f(const GridDev& g, const float* pos, int64_t n, const float* grad,
                    int64_t level_step, int64_t sample_step, float* d_table, hipStream_t st) {
  // at least a workgroup per CU: a short batch in shorter chunks.  Each clears and
  // adds a box of its own, so shorter ones than that cost more (65,537 samples,
  // four levels: 24.8 us in 130 workgroups, 30.6 in 258, 42.4 in 514; 2^18, five
  // levels: 117 in 640, 134 in 1,280, 157 in 2,560)
  int chunk = kChunk;
  while (chunk > kChunkMin && (n + chunk - 1) / chunk * g.coarse < 256) chunk /= 2;
  const int64_t blocks = (n + chunk - 1) / chunk;
  hipLaunchKernelGGL(coarse_scatter_kernel<F>, dim3((unsigned)blocks, (unsigned)g.coarse),
                     dim3(kThreads), kCap * sizeof(float), st, g,
                     reinterpret_cast<const float4*>(pos), n, grad, level_step, sample_step, chunk,
                     d_table);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_coarse_scatter(const GridDev& g, const float* pos, int64_t n, const float* grad,
                                 int64_t level_step, int64_t sample_step, float* d_table,
                                 hipStream_t st) {
  if (g.coarse <= 0 || n == 0) return hipSuccess;
  switch (g.F) {
    case 1: return launch_f<1>(g, pos, n, grad, level_step, sample_step, d_table, st);
    case 2: return launch_f<2>(g, pos, n, grad, level_step, sample_step, d_table, st);
    case 4: return launch_f<4>(g, pos, n, grad, level_step, sample_step, d_table, st);
    case 8: return launch_f<8>(g, pos, n, grad, level_step, sample_step, d_table, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace fh
