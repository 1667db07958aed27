// Multi-resolution tesseract encoding (Sec. 3.2.4): per level, locate the 4D cell,
// look up the 16 corner slots through the per-level hash and blend the corner
// embeddings with quadrilinear weights; and its adjoint (scatter-add).
//
// The 16 corners are visited as 8 pairs: in the rows order the vertex rows (dy, dz,
// dt) of an x-pair (x, x+1), one directory entry serving both vertices unless x
// sits on bit 63 of a word; in the brick order pairs along an axis that keeps both
// in one brick (corner_pair).
#include "encode_dev.h"
#include "kernels.h"

namespace fh {

namespace {

// How a launch walks the samples and levels.
//  0: one thread per sample and level, levels fastest: the lookups of a sample's
//     levels overlap and a wave writes one contiguous range of enc.
//  > 0: one thread per sample and level, that many workgroups of 256 samples
//     through one level after another, then the next as many: the waves in flight
//     share a level and its part of the table stays in the caches.
//  < 0: one thread per sample with a loop over its levels (bricks).
struct Walk {
  int chunk;
  // workgroups for n samples of L levels
  unsigned blocks(int64_t n, int L) const {
    const int64_t b = (n + 255) / 256;
    if (chunk == 0) return (unsigned)((n * L + 255) / 256);
    return (unsigned)(chunk < 0 ? b : (b + chunk - 1) / chunk * chunk * L);
  }
  // the thread's sample, and its levels l0 .. l1 - 1
  __device__ __forceinline__ int64_t at(int L, int& l0, int& l1) const {
    if (chunk > 0) {
      const unsigned group = blockIdx.x / (unsigned)(chunk * L);
      const unsigned in = blockIdx.x - group * (unsigned)(chunk * L);
      l0 = (int)(in / (unsigned)chunk);
      l1 = l0 + 1;
      return ((int64_t)group * chunk + (in - (unsigned)l0 * chunk)) * 256 + threadIdx.x;
    }
    const int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (chunk < 0) {
      l0 = 0;
      l1 = L;
      return t;
    }
    const int64_t s = t / L;
    l0 = (int)(t - s * L);
    l1 = l0 + 1;
    return s;
  }
};

// Forward; row_bytes: of a table row.  us of a thread per sample / levels fastest /
// level by level / in groups of 256 workgroups, 16 levels, FP32, F = 2:
//                                             65,537 samples      262,144
//   active, 240x360x60x50, draw order         147 183 160 152     596 717 548 594
//   dense, 121x90x61x20, draw order            85 118  94  91     369 451 317 342
//   hashed, 2^19 rows a level, draw order      73 136  80  79     308 530 238 308
//   hashed, 2^14 rows a level, draw order      34  38  39  35     135 143 127 128
//   hashed, 2^14 rows a level, sorted          27  25  23  20      64  91  63  53
// Up to 40,960 samples the launch is a few hundred workgroups, and a sample's levels
// side by side shorten its wait: levels fastest where the levels but the largest fit
// the L2 of an XCD together, from F = 4 on, and on a dense index of two features; level
// by level elsewhere.  Larger batches go in groups, whose part of a level's table and
// of enc stays in the caches (active, 121x90x61x20, F = 1, 2^20 sorted samples 282 405
// 282 216; dense, 60x45x30x10, F = 8, 8 levels, 2^18 sorted samples 63 93 66 66), but
// for four levels or fewer over a table past the L2s, of which only the largest misses
// them and the cheap ones hide behind it (active, 240x360x60x50, 150,000 samples 89 82
// 82 85), and for a hashed table past them, whose reads are spread over a whole level,
// so that the waves in flight share one as long as they can (the third row; 2^20
// samples 1,437 2,097 874 1,192).  On bricks a sample's lookups are its longest part,
// and where they miss the caches too, a thread per sample is ahead in draw order from
// where every CU has one workgroup of them (F = 1, 65,537 and 100,003 samples, a thread
// per sample and level by level: 240x360x60x50, 784 MiB of table, 160 and 192, 239 and
// 274; 121x90x61x20, 65 MiB, 132 and 131, 182 and 178, sorted 120 and 65, 140 and 87);
// past 2^19 samples groups are (the first volume, 2^20 samples 2,879 and 2,577, sorted
// 969 and 850).
inline Walk fwd_walk(const GridDev& g, int64_t n, int64_t row_bytes) {
  const int by_level = (int)((n + 255) / 256), groups = by_level < 256 ? by_level : 256;
  if (n <= 4096) return {0};
  const int64_t rows = g.last_pair + 2, bytes = rows * row_bytes;
  if (g.lv[0].brick)
    return {n > 524288 ? groups : n > 40960 && bytes > 80 << 20 ? -1 : by_level};
  if (n > 40960) {
    if (g.next_row) return {g.L <= 4 && bytes > 16 << 20 ? 0 : groups};
    return {bytes > 10 << 20 && n > 81920 ? by_level : groups};
  }
  if (g.active) return {g.F <= 2 ? by_level : 0};
  if (g.next_row && g.F >= 2) return {0};
  int64_t most = rows - g.lv[g.L - 1].slot_off;
  for (int l = 0; l + 1 < g.L; ++l) {
    const int64_t r = g.lv[l + 1].slot_off - g.lv[l].slot_off;
    if (r > most) most = r;
  }
  return {(rows - most) * row_bytes <= 4 << 20 ? 0 : by_level};
}

// Backward.  A batch in cell order wants the waves in flight on one level: lanes of
// neighbouring samples then add into the same 64-byte segments, which one transaction
// performs.  In draw order the walk only costs d_enc read once per level, so it goes
// in groups of workgroups whose part of d_enc stays in the caches.  16 levels, in
// draw order and sorted, us of two threads per sample and feature walking the levels /
// levels fastest / in groups of 128, of 256 and of 512: 200,000 samples, F = 1, 1,565
// 1,463 / 1,402 1,567 / 1,422 1,519 / 1,448 1,500 / 1,461 1,463; F = 2, 1,578 1,583 /
// 1,485 1,590 / 1,520 1,564 / 1,525 1,553 / 1,546 1,534; 1,048,576 samples, F = 1,
// 7,423 8,366 / 7,246 8,554 / 7,267 8,275 / 7,341 8,413 / 7,420 8,418.  From F = 4 on a
// pair fills half a segment and levels fastest is ahead of the threads per sample in
// both orders (F = 8, 5,095 and 5,172; sorted 7,155 and 8,412).
inline Walk bwd_walk(const GridDev& g, int64_t n) {
  if (g.F >= 4) return {0};
  const int64_t blocks = (n + 255) / 256, group = g.F == 1 && n <= 524288 ? 256 : 128;
  return {(int)(blocks < group ? blocks : group)};
}

// LOOP: walk.chunk < 0 (as a loop of one trip the others lost up to 7 %).
template <int F, typename T, bool BRICK, bool LOOP>
__global__ void __launch_bounds__(256)
    encode_fwd_kernel(GridDev g, Walk walk, const float4* __restrict__ pos, int64_t n,
                      const T* __restrict__ table, float* __restrict__ enc) {
  __shared__ LevelDev lv[FHASH_MAX_LEVELS];
  if (threadIdx.x < FHASH_MAX_LEVELS) lv[threadIdx.x] = g.lv[threadIdx.x];
  __syncthreads();
  int l0, l1;
  const int64_t s = walk.at(g.L, l0, l1);
  if (s >= n) return;
  const float4 p = pos[s];
  float* o = enc + (s * g.L + l0) * F;
  for (int i = l0; i < l1; ++i, o += F) {
    const int l[1] = {i};
    float out[1][F];
    if constexpr (BRICK)
      encode_brick_level<F, T>(lv[i], g.dir, g.active != 0, p, table, out[0], g.tmask);
    else
      encode_rows<1, F, T>(g, lv, l, p, table, out);
#pragma unroll
    for (int k = 0; k < F; ++k) o[k] = out[0][k];
    if constexpr (!LOOP) break;
  }
}

// Rows order: one thread per sample and level in groups of 2F that add their
// members' samples one after another (scatter_rows); levels below g.coarse are left
// to the LDS scatter.  Brick order: 2F threads per sample (pair element x feature),
// a loop over the levels.
template <int F, bool BRICK>
__global__ void __launch_bounds__(256)
    encode_bwd_kernel(GridDev g, Walk walk, const float4* __restrict__ pos, int64_t n,
                      const float* __restrict__ d_enc, float* __restrict__ d_table) {
  if constexpr (BRICK) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    constexpr int Q = 2 * F;
    const int64_t s = t / Q;
    if (s >= n) return;
    const int r = (int)(t % Q), e = r / F, f = r % F;
    const float4 p = pos[s];
    const float* gin = d_enc + s * (int64_t)g.L * F;
    for (int l = 0; l < g.L; ++l)
      scatter_brick_lane<F>(g.lv[l], g.dir, g.active != 0, p, e, f, gin[l * F + f], d_table,
                            g.touch, g.touch_begin, g.gmask);
  } else {
    __shared__ LevelDev lv[FHASH_MAX_LEVELS];
    if (threadIdx.x < FHASH_MAX_LEVELS) lv[threadIdx.x] = g.lv[threadIdx.x];
    __syncthreads();
    int l, l1;
    const int64_t s = walk.at(g.L, l, l1);
    const bool own = s < n && l >= g.coarse;
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
    float gr[F];
#pragma unroll
    for (int k = 0; k < F; ++k) gr[k] = 0.0f;
    if (own) {
      p = pos[s];
#pragma unroll
      for (int k = 0; k < F; ++k) gr[k] = d_enc[(s * g.L + l) * F + k];
    }
    scatter_rows<F>(g, lv[l], p, own, gr, d_table);
  }
}

// Instrumentation: per (sample, level) the directory entries and table rows the
// 8 corner pairs of its cell touch (corner_pair: rows layout, pair r = the
// x-pair of row (dy, dz, dt) = (r & 1, r >> 1 & 1, r >> 2); bricks, pairs along
// pair_axis).
__global__ void __launch_bounds__(256)
    corner_rows_kernel(GridDev g, const float4* __restrict__ pos, int64_t n,
                       long long* __restrict__ out_dir, long long* __restrict__ out_slot) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= n * g.L) return;
  const int64_t s = t / g.L;
  const int l = (int)(t % g.L);
  const LevelDev& d = g.lv[l];
  const float4 p = pos[s];
  int ix, iy, iz, it;
  float fx, fy, fz, ft;
  locate(p.x, d.rx, d.sx, ix, fx);
  locate(p.y, d.ry, d.sy, iy, fy);
  locate(p.z, d.rz, d.sz, iz, fz);
  locate(p.w, d.rt, d.st, it, ft);
  const bool active = g.active != 0 && d.hash_bits == 0;
  const int a = d.brick ? pair_axis<true>(ix, iy, iz, it) : 0;
  for (int r = 0; r < 8; ++r) {
    float wr;
    int64_t s0, s1;
    bool v0, v1;
    if (d.brick)
      corner_pair<true>(d, g.dir, g.active != 0, ix, iy, iz, it, fx, fy, fz, ft, a, r, s0, s1,
                        v0, v1, wr);
    else
      corner_pair<false>(d, g.dir, g.active != 0, ix, iy, iz, it, fx, fy, fz, ft, a, r, s0, s1,
                         v0, v1, wr);
    const int64_t o = (t * 8 + r) * 2;
    long long w0 = -1, w1 = -1;
    if (active) {
      int ox = 0, oy = r & 1, oz = (r >> 1) & 1, ot = r >> 2;
      if (d.brick) pair_offsets(r, a, ox, oy, oz, ot);
      int64_t e0, e1;
      int b0, b1;
      // the entries of the pair's first corner and of its x neighbour (the
      // second corner shares the first one's entry unless the pair is along x)
      if (d.brick)
        pair_entries<true>(d, it + ot, iz + oz, iy + oy, ix + ox, e0, e1, b0, b1);
      else
        pair_entries<false>(d, it + ot, iz + oz, iy + oy, ix + ox, e0, e1, b0, b1);
      w0 = e0;
      if (a == 0 && e1 != e0) w1 = e1;
    }
    out_dir[o] = w0;
    out_dir[o + 1] = w1;
    out_slot[o] = v0 ? s0 : -1;
    out_slot[o + 1] = v1 ? s1 : -1;
  }
}

// Samples of one launch with `per` threads to a sample.  A launch holds fewer than
// 2^32 threads (2^28 samples of 16 levels have as many); larger batches go in pieces.
inline int64_t launch_piece(int per) { return ((int64_t)1 << 31) / per; }

template <int F, typename T>
void launch_fwd_tt(const GridDev& g, const float* pos, int64_t n, const T* table, float* enc,
                   hipStream_t st) {
  const Walk walk = fwd_walk(g, n, F * sizeof(T));
  const dim3 grid(walk.blocks(n, g.L));
  const float4* p = reinterpret_cast<const float4*>(pos);
  auto kern = !g.lv[0].brick  ? encode_fwd_kernel<F, T, false, false>
              : walk.chunk < 0 ? encode_fwd_kernel<F, T, true, true>
                               : encode_fwd_kernel<F, T, true, false>;
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, g, walk, p, n, table, enc);
}

template <int F>
hipError_t launch_fwd_t(const GridDev& g, const float* pos, int64_t n, const void* table,
                        fhash_dtype dt, float* enc, hipStream_t st) {
  const int64_t piece = launch_piece(g.L);
  for (int64_t s = 0; s < n; s += piece) {
    const int64_t m = n - s < piece ? n - s : piece;
    float* e = enc + s * g.L * F;
    if (dt == FHASH_F32)
      launch_fwd_tt<F>(g, pos + 4 * s, m, reinterpret_cast<const float*>(table), e, st);
    else
      launch_fwd_tt<F>(g, pos + 4 * s, m, reinterpret_cast<const __half*>(table), e, st);
    if (const hipError_t err = hipGetLastError()) return err;
  }
  return hipSuccess;
}

template <int F>
hipError_t launch_bwd_t(const GridDev& g, const float* pos, int64_t n, const float* d_enc,
                        float* d_table, hipStream_t st) {
  const bool brick = g.lv[0].brick;
  const int per = brick ? 2 * F : g.L;
  const int64_t piece = launch_piece(per);
  for (int64_t s = 0; s < n; s += piece) {
    const int64_t m = n - s < piece ? n - s : piece;
    const float4* p = reinterpret_cast<const float4*>(pos) + s;
    const float* de = d_enc + s * g.L * F;
    const Walk walk = bwd_walk(g, m);
    const dim3 grid(brick ? (unsigned)((m * per + 255) / 256) : walk.blocks(m, g.L));
    if (brick)
      hipLaunchKernelGGL((encode_bwd_kernel<F, true>), grid, dim3(256), 0, st, g, walk, p, m, de,
                         d_table);
    else
      hipLaunchKernelGGL((encode_bwd_kernel<F, false>), grid, dim3(256), 0, st, g, walk, p, m, de,
                         d_table);
    if (const hipError_t err = hipGetLastError()) return err;
  }
  if (g.coarse == 0) return hipSuccess;
  return launch_coarse_scatter(g, pos, n, d_enc, F, (int64_t)g.L * F, d_table, st);
}

}  // namespace

hipError_t launch_encode_fwd(const GridDev& g, const float* pos, int64_t n, const void* table,
                             fhash_dtype dt, float* enc, hipStream_t st) {
  if (n == 0) return hipSuccess;
  switch (g.F) {
    case 1: return launch_fwd_t<1>(g, pos, n, table, dt, enc, st);
    case 2: return launch_fwd_t<2>(g, pos, n, table, dt, enc, st);
    case 4: return launch_fwd_t<4>(g, pos, n, table, dt, enc, st);
    case 8: return launch_fwd_t<8>(g, pos, n, table, dt, enc, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_corner_rows(const GridDev& g, const float* pos, int64_t n, int64_t* out_dir,
                              int64_t* out_slot, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int64_t blocks = (n * g.L + 255) / 256;
  hipLaunchKernelGGL(corner_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, g,
                     reinterpret_cast<const float4*>(pos), n,
                     reinterpret_cast<long long*>(out_dir), reinterpret_cast<long long*>(out_slot));
  return hipGetLastError();
}

hipError_t launch_encode_bwd(const GridDev& g, const float* pos, int64_t n, const float* d_enc,
                             float* d_table, hipStream_t st) {
  if (n == 0) return hipSuccess;
  switch (g.F) {
    case 1: return launch_bwd_t<1>(g, pos, n, d_enc, d_table, st);
    case 2: return launch_bwd_t<2>(g, pos, n, d_enc, d_table, st);
    case 4: return launch_bwd_t<4>(g, pos, n, d_enc, d_table, st);
    case 8: return launch_bwd_t<8>(g, pos, n, d_enc, d_table, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace fh
