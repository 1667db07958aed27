// Index build: voxel feature mask -> per-level active vertices -> rank directory
// (the collision-free per-level hash, Sec. 3.2.3 / Sec. 3.1).
//
// Voxel i of a dimension sits at u = i (R-1)/(S-1) on a level, a cell is active
// iff its closed box contains a masked voxel, and a vertex iff one of its cells
// is: iff some masked voxel lies within one vertex spacing of it along every
// axis.  That is separable, so a level's vertex bits come from one OR over
// voxel ranges per axis: along y (usually the axis a level shrinks most, so the
// later passes have the least to read), along z and t (vertex v = cell v-1 OR
// cell v, each voxel read once per thread), and along x inside the words.  Where the
// workspace is not to hold the whole mask transposed, it goes through the first three
// a slab of frames at a time, and the pass along t adds each slab's frames to the
// vertices they reach.
//
// The mask is first transposed to [t][z][word][y], the store order of the
// directory, so that neighbouring threads of every pass hold neighbouring y:
// coalesced loads and stores, and the word index and the x ranges of its 64
// vertices are the same in every lane (scalar arithmetic).  The directory
// stores, for every 64-vertex word of a row-padded vertex bitmap, the bits and
// the number of active vertices before the word (exclusive prefix sum of
// popcounts in F-Hash linearisation order).  Row padding bits are zero, so ranks
// equal ranks in the unpadded order.  Levels small enough to share the
// workspace of the largest go through each pass in one launch.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace fh {

namespace {

// Voxels i with c <= i(R-1)/(S-1) <= c+1 (closed cell box): ceil(c (S-1)/(R-1))
// .. floor((c+1)(S-1)/(R-1)).
// (S - 1) R below 2^31 (every volume of thousands of voxels a side): 32-bit
// divisions, a quarter of the 64-bit ones' instructions.
__device__ __forceinline__ int64_t range_lo(int64_t c, int64_t S, int64_t R) {
  if ((S - 1) * R < ((int64_t)1 << 31))
    return ((uint32_t)c * (uint32_t)(S - 1) + (uint32_t)(R - 2)) / (uint32_t)(R - 1);
  return (c * (S - 1) + R - 2) / (R - 1);
}
__device__ __forceinline__ int64_t range_hi(int64_t c, int64_t S, int64_t R) {
  const int64_t hi = (S - 1) * R < ((int64_t)1 << 31)
                         ? (uint32_t)(c + 1) * (uint32_t)(S - 1) / (uint32_t)(R - 1)
                         : ((c + 1) * (S - 1)) / (R - 1);
  return hi > S - 1 ? S - 1 : hi;
}

// floor(k (S-1)/(R-1)) for k, k+1, ... without a division per step.
struct Steps {
  int32_t q, dq, r, dr, n;  // S <= 2^31 and k < R: every quotient fits
  __device__ __forceinline__ Steps(int64_t k, int64_t S, int64_t R) {
    n = (int32_t)(R - 1);
    const int64_t p = k * (S - 1);
    q = (int32_t)(p / n);
    r = (int32_t)(p - (int64_t)q * n);
    dq = (int32_t)((S - 1) / n);
    dr = (int32_t)((S - 1) - (int64_t)dq * n);
  }
  __device__ __forceinline__ void next() {
    q += dq;
    r += dr;
    if (r >= n) {
      r -= n;
      ++q;
    }
  }
};

// One level of a launch: vertex counts, words per vertex row, and where its
// part of each workspace array begins (64-bit words; row counts; row blocks).
struct LevelBuild {
  int32_t rx, ry, rz, rt, wv, y0;  // y0: ry of the group's levels before this one
  int32_t v0, v1;                  // the t vertices that the slab's frames reach
  int64_t a, b, c, bits;           // a, b: words per frame of the slab
  int64_t row, blk, dir;
};
constexpr int kMaxGroup = FHASH_MAX_LEVELS;
struct GroupBuild {
  LevelBuild lv[kMaxGroup];
  int64_t Sx, Sy, Sz, St, Wm;
  int64_t f0, nf;  // the slab: frames f0 .. f0 + nf - 1
};

// Mask rows [t][z][y][w] -> [t][z][w][y], 64 y by up to 32 words at a time
// through LDS, so that both sides are read and written in runs.
constexpr int kTileW = 32;
__global__ void __launch_bounds__(256)
    transpose_kernel(const uint64_t* __restrict__ in, uint64_t* __restrict__ out, int64_t slabs,
                     int64_t Sy, int64_t W) {
  __shared__ uint64_t tile[kTileW][65];
  const int64_t ty = (Sy + 63) / 64, tw = (W + kTileW - 1) / kTileW, tiles = slabs * ty * tw;
  for (int64_t e = blockIdx.x; e < tiles; e += gridDim.x) {
    const int64_t slab = e / (ty * tw), rest = e - slab * ty * tw;
    const int64_t y0 = rest / tw * 64, w0 = rest % tw * kTileW;
    const int ny = Sy - y0 < 64 ? (int)(Sy - y0) : 64;
    const int nw = W - w0 < kTileW ? (int)(W - w0) : kTileW;
    const uint64_t* src = in + slab * Sy * W + y0 * W + w0;
    uint64_t* dst = out + slab * Sy * W + w0 * Sy + y0;
    for (int i = threadIdx.x; i < ny * nw; i += 256) {
      const int y = i / nw, w = i - y * nw;
      tile[w][y] = src[y * W + w];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * nw; i += 256)
      if ((i & 63) < ny) dst[(i >> 6) * Sy + (i & 63)] = tile[i >> 6][i & 63];
    __syncthreads();
  }
}

// out[o][v][q] = OR over the voxels s of cells v-1 and v of in[o][s][q]: a
// thread walks `per` vertices of one (o, q), so a voxel is read once (twice on
// a cell face).  inner: words that share an (o, s).  A walk is a chain of
// loads, so lines are cut into chunks of vertices (at least 4, each chunk reads
// one cell of its neighbour's again) until 2^20 threads share the work: the z
// pass of the 480x720x120x24 volume's levels took 427 us at 2^18 and 332 us so.
constexpr int64_t kLineThreads = 1 << 20;
__host__ __device__ inline int64_t line_chunks(int64_t lines, int64_t R) {
  const int64_t chunks = lines >= kLineThreads ? 1 : (kLineThreads + lines - 1) / lines;
  return chunks < (R + 3) / 4 ? chunks : (R + 3) / 4;
}
__device__ __forceinline__ void or_axis(const uint64_t* __restrict__ in,
                                        uint64_t* __restrict__ out, int64_t outer, int64_t S,
                                        int64_t R, int64_t inner) {
  // vertices per thread: fewer where (outer, inner) alone leaves the chip idle
  const int64_t lines = outer * inner;
  const int64_t chunks = line_chunks(lines, R);
  const int64_t per = (R + chunks - 1) / chunks, total = lines * chunks;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = e % inner, rest = e / inner;
    const int64_t v0 = (rest % chunks) * per, o = rest / chunks;
    const int64_t v1 = v0 + per < R ? v0 + per : R;
    const uint64_t* src = in + o * S * inner + q;
    uint64_t* dst = out + o * R * inner + q;
    int64_t c = v0 > 0 ? v0 - 1 : 0;
    Steps top(c, S, R);
    int64_t lo = top.q + (top.r > 0 ? 1 : 0);
    uint64_t prev = 0;
    for (; c < v1; ++c) {
      uint64_t cell = 0;
      if (c < R - 1) {
        top.next();
        const int64_t hi = top.q < S - 1 ? top.q : S - 1;
#pragma unroll 4
        for (int64_t s = lo; s <= hi; ++s) cell |= src[s * inner];
        lo = top.q + (top.r > 0 ? 1 : 0);
      }
      if (c >= v0) dst[c * inner] = prev | cell;
      prev = cell;
    }
  }
}

// Along y: [line][Sy] -> [line][ry] for every level of the group, line = (t, z,
// word).  A workgroup takes a line through all the levels (items: their
// vertices, numbered through), so that it is read from memory once.
__global__ void __launch_bounds__(256)
    or_y_kernel(GroupBuild G, int32_t items, const uint64_t* __restrict__ mask,
                uint64_t* __restrict__ A) {
  const int64_t lines = G.nf * G.Sz * G.Wm;
  for (int64_t line = blockIdx.x; line < lines; line += gridDim.x) {
    const uint64_t* src = mask + line * G.Sy;
    int j = 0;
    for (int32_t e = threadIdx.x; e < items; e += 256) {
      while (e >= G.lv[j].y0 + G.lv[j].ry) ++j;
      const int32_t R = G.lv[j].ry, v = e - G.lv[j].y0;
      const int64_t lo = v > 0 ? range_lo(v - 1, G.Sy, R) : 0;
      const int64_t hi = v < R - 1 ? range_hi(v, G.Sy, R) : G.Sy - 1;
      uint64_t acc = 0;
#pragma unroll 4
      for (int64_t s = lo; s <= hi; ++s) acc |= src[s];
      A[G.lv[j].a * G.nf + line * R + v] = acc;
    }
  }
}

__global__ void __launch_bounds__(256)
    or_z_kernel(GroupBuild G, const uint64_t* __restrict__ A, uint64_t* __restrict__ B) {
  const LevelBuild& d = G.lv[blockIdx.y];
  or_axis(A + d.a * G.nf, B + d.b * G.nf, G.nf, G.Sz, d.rz, G.Wm * d.ry);
}

__global__ void __launch_bounds__(256)
    or_t_kernel(GroupBuild G, const uint64_t* __restrict__ B, uint64_t* __restrict__ C) {
  // Along t: the slab's part of vertices v0 .. v1 - 1, walked as or_axis does.  The
  // slab that holds the first voxel of a vertex's range writes its word, later ones
  // add to it.
  const LevelBuild& d = G.lv[blockIdx.y];
  const int64_t inner = d.rz * G.Wm * d.ry, S = G.St, R = d.rt, nv = d.v1 - d.v0;
  const int64_t f1 = G.f0 + G.nf;
  const int64_t chunks = line_chunks(inner, nv);
  const int64_t per = (nv + chunks - 1) / chunks, total = inner * chunks;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = e % inner, va = d.v0 + e / inner * per;
    const int64_t vb = va + per < d.v1 ? va + per : d.v1;
    const uint64_t* src = B + d.b * G.nf + q;
    uint64_t* dst = C + d.c + q;
    int64_t c = va > 0 ? va - 1 : 0;
    Steps top(c, S, R);
    int64_t lo = top.q + (top.r > 0 ? 1 : 0), first = 0;  // first voxel of vertex c
    uint64_t prev = 0;
    for (; c < vb; ++c) {
      uint64_t cell = 0;
      const int64_t lo_c = lo;
      if (c < R - 1) {
        top.next();
        int64_t hi = top.q < S - 1 ? top.q : S - 1;
        if (hi > f1 - 1) hi = f1 - 1;
#pragma unroll 4
        for (int64_t s = lo_c > G.f0 ? lo_c : G.f0; s <= hi; ++s)
          cell |= src[(s - G.f0) * inner];
        lo = top.q + (top.r > 0 ? 1 : 0);
      }
      if (c >= va) {
        const uint64_t w = prev | cell;
        dst[c * inner] = first >= G.f0 ? w : dst[c * inner] | w;
      }
      prev = cell;
      first = lo_c;
    }
  }
}

constexpr int kScanThreads = 256;
constexpr int kScanPerThread = 8;
constexpr int64_t kScanBlockWords = kScanThreads * kScanPerThread;

__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t* sh,
                                                         uint64_t& total) {
  // Inclusive scan inside each wave, then across waves (<= 16 waves).
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint64_t x = v;
  for (int off = 1; off < 64; off <<= 1) {
    uint64_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t run = 0;
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) {
      uint64_t t = sh[i];
      sh[i] = run;
      run += t;
    }
    sh[16] = run;
  }
  __syncthreads();
  total = sh[16];
  const uint64_t res = sh[wid] + x - v;
  __syncthreads();
  return res;
}

// Along x and the row counts: a workgroup takes kRows vertex rows (t, z, y), a
// lane per row, and each of its waves every fourth word, so that a wave's word
// and the voxel ranges of its vertices are the same in every lane.  Output word
// w holds vertices 64w .. 64w + 63; a vertex is set iff the row has a voxel bit
// in its range.  Writes the bits in [tz][w][y] order, each row's count, and the
// block's total.
constexpr int kRows = 64;
__global__ void __launch_bounds__(256)
    rows_kernel(GroupBuild G, int64_t first, const uint64_t* __restrict__ C,
                uint64_t* __restrict__ bits, uint32_t* __restrict__ row_count,
                uint64_t* __restrict__ partial) {
  __shared__ uint32_t sh[4][kRows];
  const LevelBuild& d = G.lv[blockIdx.y];
  const int64_t rows = (int64_t)d.rt * d.rz * d.ry;
  const int64_t block = first + blockIdx.x;  // first: blocks of rows before this launch's
  if (block * kRows >= rows) return;  // uniform: a smaller level
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = block * kRows + lane;
  const bool valid = row < rows;
  const int64_t mine = valid ? row : rows - 1;  // every lane stays with its wave
  const int64_t tz = mine / d.ry, y = mine - tz * d.ry;
  const uint64_t* src = C + d.c + tz * G.Wm * d.ry + y;
  uint64_t* dst = bits + d.bits + tz * d.wv * d.ry + y;
  const int32_t Wm = (int32_t)G.Wm;
  uint32_t count = 0;
  for (int32_t w = wid; w < d.wv; w += 4) {
    uint64_t o = 0;
    const int nb = d.rx - 64 * w < 64 ? d.rx - 64 * w : 64;
    if (d.rx == G.Sx) {
      // one vertex per voxel: the voxel, its left and its right neighbour
      const uint64_t prev = w > 0 ? src[(int64_t)(w - 1) * d.ry] : 0ull;
      const uint64_t cur = src[(int64_t)w * d.ry];
      const uint64_t next = w + 1 < Wm ? src[(int64_t)(w + 1) * d.ry] : 0ull;
      o = cur | (cur << 1) | (prev >> 63) | (cur >> 1) | (next << 63);
      if (nb < 64) o &= (1ull << nb) - 1ull;
    } else {
      // voxels lo .. hi of vertex v (cells v - 1 and v): lane b works out those
      // of vertex 64 w + b, from where they are read back as scalars
      const int64_t v = 64 * (int64_t)w + lane;
      const int32_t lo_b = v > 0 ? (int32_t)range_lo(v - 1, G.Sx, d.rx) : 0;
      const int32_t hi_b = (int32_t)(v < d.rx - 1 ? range_hi(v, G.Sx, d.rx) : G.Sx - 1);
      int32_t have = -2;  // the word held in cur; prev holds the one before it
      uint64_t prev = 0, cur = 0;
      for (int b = 0; b < nb; ++b) {
        const int32_t lo = __builtin_amdgcn_readlane(lo_b, b);
        const int32_t hi = __builtin_amdgcn_readlane(hi_b, b);
        if (lo > hi) continue;  // no voxel near this vertex (a level finer than the volume)
        const int32_t w0 = lo >> 6, w1 = hi >> 6;
        if (w1 != have) {
          prev = w1 == have + 1 ? cur : w1 > 0 ? src[(int64_t)(w1 - 1) * d.ry] : 0ull;
          cur = src[(int64_t)w1 * d.ry];
          have = w1;
        }
        const uint64_t from = ~0ull << (lo & 63), upto = ~0ull >> (63 - (hi & 63));
        uint64_t any;
        if (w0 == w1) {
          any = cur & (from & upto);
        } else {
          any = cur & upto;
          if (w0 == w1 - 1) {
            any |= prev & from;
          } else {
            any |= prev | (src[(int64_t)w0 * d.ry] & from);
            for (int32_t wi = w0 + 1; wi < w1 - 1; ++wi) any |= src[(int64_t)wi * d.ry];
          }
        }
        o |= (any != 0 ? 1ull : 0ull) << b;
      }
    }
    if (valid) dst[(int64_t)w * d.ry] = o;
    count += valid ? __popcll(o) : 0;
  }
  sh[wid][lane] = count;
  __syncthreads();
  if (wid == 0) {
    const uint32_t c = sh[0][lane] + sh[1][lane] + sh[2][lane] + sh[3][lane];
    if (valid) row_count[d.row + row] = c;
    uint64_t total = c;
    for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
    if (lane == 0) partial[d.blk + block] = total;
  }
}

// The directory: {bits, active vertices before the word} of every word, from
// the row counts' prefix sum; kScanThreads rows per workgroup (kRows divides it).
__global__ void __launch_bounds__(kScanThreads)
    entries_kernel(GroupBuild G, const uint64_t* __restrict__ bits,
                   const uint32_t* __restrict__ row_count, const uint64_t* __restrict__ partial,
                   ulonglong2* __restrict__ dir) {
  __shared__ uint64_t sh[17];
  const LevelBuild& d = G.lv[blockIdx.y];
  const int64_t rows = (int64_t)d.rt * d.rz * d.ry;
  if (blockIdx.x * (int64_t)kScanThreads >= rows) return;  // uniform: a smaller level
  const int64_t row = blockIdx.x * (int64_t)kScanThreads + threadIdx.x;
  const bool valid = row < rows;
  uint64_t total;
  uint64_t run = block_exclusive_scan(valid ? row_count[d.row + row] : 0u, sh, total) +
                 partial[d.blk + blockIdx.x * (int64_t)(kScanThreads / kRows)];
  if (!valid) return;
  const int64_t tz = row / d.ry, y = row - tz * d.ry;
  const int64_t at = tz * d.wv * d.ry + y;
  for (int64_t w = 0; w < d.wv; ++w) {
    const uint64_t o = bits[d.bits + at + w * d.ry];
    ulonglong2 ent;
    ent.x = o;
    ent.y = run;
    dir[d.dir + at + w * d.ry] = ent;
    run += __popcll(o);
  }
}

// Store order of a brick directory: the entries of one word index for all
// brick rows of a (t, z) block are adjacent, so that the brick rows y and y+1
// of a cell read neighbouring entries.  Ranks are computed row-major first.
__global__ void dir_interleave_kernel(const ulonglong2* __restrict__ src,
                                      ulonglong2* __restrict__ dst, int64_t rows, int64_t ry,
                                      int64_t wv) {
  const int64_t total = rows * wv;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t w = e % wv, row = e / wv;
    const int64_t tz = row / ry, y = row % ry;
    dst[(tz * wv + w) * ry + y] = src[e];
  }
}

// Brick order (layout FHASH_LAYOUT_BRICKS): word w of brick row (bt, bz, by)
// holds bricks bx = 4w .. 4w+3, brick q at bits 16q .. 16q+15, vertex inner
// index (x%2) | (y%2)<<1 | (z%2)<<2 | (t%2)<<3.  Built from the vertex bits in
// [tz][word][y] order: the 8 x bits 8w .. 8w+7 of each of the brick row's 8
// vertex rows lie in one word.  Output in brick-linear
// order (((bt*Bz + bz)*By + by)*Wb + w), ranks still to be written.
__global__ void brickify_kernel(const uint64_t* __restrict__ rows, ulonglong2* __restrict__ out,
                                int64_t rx, int64_t ry, int64_t rz, int64_t rt, int64_t wv,
                                int64_t wb, int64_t by_n, int64_t bz_n, int64_t total) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t w = e % wb, row = e / wb;
    const int64_t by = row % by_n, bz = (row / by_n) % bz_n, bt = row / (by_n * bz_n);
    uint64_t bits = 0;
    for (int c = 0; c < 8; ++c) {  // (y%2, z%2, t%2) of the vertex row
      const int64_t y = 2 * by + (c & 1), z = 2 * bz + ((c >> 1) & 1), t = 2 * bt + (c >> 2);
      if (y >= ry || z >= rz || t >= rt) continue;
      const int64_t x0 = 8 * w;  // x bits 8w .. 8w+7 (x >= rx reads the row's zero padding)
      if (x0 >= rx) continue;
      const uint64_t xb = (rows[((t * rz + z) * wv + (x0 >> 6)) * ry + y] >> (x0 & 63)) & 0xFFull;
      for (int q = 0; q < 4; ++q)
        for (int ix = 0; ix < 2; ++ix)
          if ((xb >> (2 * q + ix)) & 1ull) bits |= 1ull << (16 * q + (ix | (c << 1)));
    }
    ulonglong2 ent;
    ent.x = bits;
    ent.y = 0;
    out[e] = ent;
  }
}

__global__ void __launch_bounds__(kScanThreads)
    popc_block_sums_kernel(const ulonglong2* __restrict__ dir, int64_t words,
                           uint64_t* __restrict__ partial) {
  __shared__ uint64_t sh[17];
  const int64_t base = blockIdx.x * kScanBlockWords + threadIdx.x * (int64_t)kScanPerThread;
  uint64_t s = 0;
  for (int i = 0; i < kScanPerThread; ++i)
    if (base + i < words) s += __popcll(dir[base + i].x);
  uint64_t total;
  block_exclusive_scan(s, sh, total);
  if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// Exclusive scan of the block partials of one level (blockIdx.x) in one
// workgroup: 4 per thread and round; count = total.
__device__ __forceinline__ void scan_partials(uint64_t* __restrict__ partial, int64_t nb,
                                              uint64_t* __restrict__ count) {
  __shared__ uint64_t sh[17];
  uint64_t carry = 0;
  for (int64_t r0 = 0; r0 < nb; r0 += 4096) {
    const int64_t i0 = r0 + 4 * (int64_t)threadIdx.x;
    uint64_t v[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = i0 + k < nb ? partial[i0 + k] : 0ull;
      s += v[k];
    }
    uint64_t total;
    uint64_t run = carry + block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k < nb) {
        partial[i0 + k] = run;
        run += v[k];
      }
    carry += total;
  }
  if (threadIdx.x == 0) *count = carry;
}

__global__ void __launch_bounds__(1024)
    scan_partials_kernel(uint64_t* __restrict__ partial, int64_t nb, uint64_t* __restrict__ count) {
  scan_partials(partial, nb, count);
}

__global__ void __launch_bounds__(1024)
    scan_rows_kernel(GroupBuild G, uint64_t* __restrict__ partial, uint64_t* __restrict__ counts) {
  const LevelBuild& d = G.lv[blockIdx.x];
  const int64_t rows = (int64_t)d.rt * d.rz * d.ry;
  scan_partials(partial + d.blk, (rows + kRows - 1) / kRows, counts + blockIdx.x);
}

__global__ void __launch_bounds__(kScanThreads)
    write_ranks_kernel(ulonglong2* __restrict__ dir, int64_t words,
                       const uint64_t* __restrict__ partial) {
  __shared__ uint64_t sh[17];
  const int64_t base = blockIdx.x * kScanBlockWords + threadIdx.x * (int64_t)kScanPerThread;
  uint64_t pc[kScanPerThread];
  uint64_t s = 0;
  for (int i = 0; i < kScanPerThread; ++i) {
    pc[i] = (base + i < words) ? (uint64_t)__popcll(dir[base + i].x) : 0ull;
    s += pc[i];
  }
  uint64_t total;
  uint64_t run = block_exclusive_scan(s, sh, total) + partial[blockIdx.x];
  for (int i = 0; i < kScanPerThread; ++i)
    if (base + i < words) {
      dir[base + i].y = run;
      run += pc[i];
    }
}

inline int grid_for(int64_t total, int threads) {
  int64_t b = (total + threads - 1) / threads;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

// Sizes of one level's parts of the workspace: a, b, c and bits in words (the
// outputs of the passes along y and z, per frame, along t and along x), rows, row
// blocks, and the brick directory.
struct LevelSizes {
  int64_t a, b, c, bits, rows, blk;
  int64_t Bx, By, Bz, Bt, Wb, bwords, bnb;  // brick layout
};

LevelSizes level_sizes(const int32_t* r, const int64_t* dims) {
  LevelSizes s;
  const int64_t Wm = (dims[0] + 63) / 64, Wv = ((int64_t)r[0] + 63) / 64;
  s.a = dims[2] * Wm * r[1];
  s.b = r[2] * Wm * r[1];
  s.c = (int64_t)r[3] * r[2] * Wm * r[1];
  s.rows = (int64_t)r[3] * r[2] * r[1];
  s.bits = s.rows * Wv;
  s.blk = (s.rows + kRows - 1) / kRows;
  s.Bx = ((int64_t)r[0] + 1) / 2;
  s.By = ((int64_t)r[1] + 1) / 2;
  s.Bz = ((int64_t)r[2] + 1) / 2;
  s.Bt = ((int64_t)r[3] + 1) / 2;
  s.Wb = (s.Bx + 3) / 4;
  s.bwords = s.Bt * s.Bz * s.By * s.Wb;
  s.bnb = (s.bwords + kScanBlockWords - 1) / kScanBlockWords;
  return s;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

int64_t index_dir_words(const fhash_grid_desc* g, int l) {
  const int32_t* r = g->res[l];
  if (g->layout == FHASH_LAYOUT_BRICKS)
    return (((int64_t)r[3] + 1) / 2) * (((int64_t)r[2] + 1) / 2) * (((int64_t)r[1] + 1) / 2) *
           ((((int64_t)r[0] + 1) / 2 + 3) / 4);
  return (int64_t)r[3] * r[2] * r[1] * (((int64_t)r[0] + 63) / 64);
}

namespace {

// The plan of a build.  Levels go through the passes in groups, coarsest first: the
// next levels that fit the arrays together (a brick level has them to itself), which
// hold the largest level and up to as much again (share), so that the finest level
// goes alone and the others in a few groups: each group reads the mask once.
//
// The workspace has row counts, block totals, level counts, the brick directory
// before its reordering, and either
//  - the whole mask transposed and two arrays that the passes alternate between (y ->
//    X, z -> Y, t -> X, x -> Y), or
//  - the words reduced along t (C) and one region for a slab of frames, transposed and
//    reduced along y and z, and then for the vertex bits,
// the second where the first would take more than a pass per axis over the whole mask
// does for the largest level (its cells along t, along t and z, and the directory's
// words twice) and more than kSmallBytes: levels much coarser than the volume, whose
// transposed mask is most of it.  A slab is then as large as that bound leaves, at
// least a frame.  480x720x120x100, 12 levels of up to 120x180x30x50: 2,874 us and 340
// MB in slabs, 2,316 us and 899 MB whole (2,690 us and 473 MB a pass per axis).  With
// arrays of twice the largest level throughout, 432x432x432x60 at its own resolution
// took 8,110 us and 3,228 MB; within the bound 8,471 us and 2,415 MB.
struct BuildPlan {
  bool whole;
  int groups;
  int first[FHASH_MAX_LEVELS + 1];
  int64_t frames;                             // of a slab
  int64_t X, Y, rows, blk, bricks;            // words; rows in 4 bytes; bricks in 16
  size_t bytes;                               // X, Y: C and the slab's region in slabs
};
constexpr size_t kSmallBytes = (size_t)256 << 20;

BuildPlan build_plan(const fhash_grid_desc* g, const int64_t* dims) {
  const bool brick = g->layout == FHASH_LAYOUT_BRICKS;
  const int64_t Wm = (dims[0] + 63) / 64, T = dims[3];
  const int64_t mask = dims[2] * dims[1] * Wm;  // words of a frame
  LevelSizes most{}, sizes[FHASH_MAX_LEVELS];
  int64_t bound = 0;
  for (int l = 0; l < g->n_levels; ++l) {
    const int32_t* r = g->res[l];
    const LevelSizes s = sizes[l] = level_sizes(r, dims);
    most.a = std::max(most.a, s.a);
    most.b = std::max(most.b, s.b);
    most.c = std::max(most.c, s.c);
    most.bits = std::max(most.bits, s.bits);
    most.rows = std::max(most.rows, s.rows);
    most.blk = std::max(most.blk, std::max(s.blk, brick ? s.bnb : 0));
    most.bwords = std::max(most.bwords, brick ? s.bwords : 0);
    bound = std::max(bound, (r[3] - 1) * mask + (int64_t)(r[3] - 1) * (r[2] - 1) * dims[1] * Wm +
                                2 * s.bits);
  }
  BuildPlan p{};
  p.bricks = most.bwords;
  // capacities and groups with the arrays at share sixteenths of the largest level;
  // returns the words per frame of the group that takes most of them
  auto group = [&](bool whole, int share) {
    const int64_t a = most.a * T * share / 16, b = most.b * T * share / 16;
    const int64_t c = most.c * share / 16, bits = most.bits * share / 16;
    p.whole = whole;
    p.X = whole ? std::max(a, c) : c;
    p.Y = whole ? std::max(b, bits) : bits;
    p.rows = most.rows * share / 16;
    p.blk = most.blk * share / 16;
    p.groups = 0;
    int64_t frame = 0;
    for (int l = 0; l < g->n_levels;) {
      LevelSizes t{};
      p.first[p.groups++] = l;
      for (int n = 0; l < g->n_levels; ++l, ++n) {
        const LevelSizes& s = sizes[l];
        if (n > 0 && (brick || t.c + s.c > p.X || t.bits + s.bits > p.Y ||
                      t.rows + s.rows > p.rows || t.blk + s.blk > p.blk ||
                      (whole && ((t.a + s.a) * T > p.X || (t.b + s.b) * T > p.Y))))
          break;
        t.a += s.a;
        t.b += s.b;
        t.c += s.c;
        t.bits += s.bits;
        t.rows += s.rows;
        t.blk += s.blk;
      }
      frame = std::max(frame, mask + t.a + t.b);
    }
    p.first[p.groups] = g->n_levels;
    return frame;
  };
  auto total = [&] {
    return align256((p.whole ? mask * T : 0) * 8) + align256(p.X * 8) + align256(p.Y * 8) +
           align256(p.rows * 4) + align256(p.blk * 8) + align256(8 * FHASH_MAX_LEVELS) +
           align256(p.bricks * 16);
  };
  const bool one = brick || g->n_levels == 1;
  const size_t most_bytes = std::max((size_t)bound * 8 + p.bricks * 16, kSmallBytes);
  for (int share = one ? 16 : 32; share >= 16; --share) {
    group(true, share);
    p.frames = T;
    p.bytes = total();
    if (p.bytes <= most_bytes) return p;
  }
  for (int share = one ? 16 : 20; share >= 16; share -= 4) {
    const int64_t frame = group(false, share);
    const int64_t left = bound - p.X - p.rows / 2 - p.blk;
    p.frames = std::max(std::min(left / frame, T), (int64_t)1);
    p.Y = std::max(p.frames * frame, p.Y);
    p.bytes = total();
    if (p.Y <= left) break;
  }
  return p;
}

// The t vertices v0 .. v1 - 1 of a level that frames f0 .. f1 - 1 reach: those whose
// voxel range (of the cells on either side) meets the slab, and those without a voxel
// whose range would begin in it.
void slab_vertices(int64_t S, int64_t R, int64_t f0, int64_t f1, int32_t* v0, int32_t* v1) {
  auto first = [&](int64_t v) { return v > 0 ? ((v - 1) * (S - 1) + R - 2) / (R - 1) : 0; };
  auto last = [&](int64_t v) {
    return std::max(first(v), v < R - 1 ? std::min((v + 1) * (S - 1) / (R - 1), S - 1) : S - 1);
  };
  auto lower = [&](auto reached) {  // first v in [0, R] for which reached(v) holds
    int64_t lo = 0, hi = R;
    while (lo < hi) {
      const int64_t m = (lo + hi) / 2;
      if (reached(m)) hi = m;
      else lo = m + 1;
    }
    return (int32_t)lo;
  };
  *v0 = lower([&](int64_t v) { return last(v) >= f0; });
  *v1 = lower([&](int64_t v) { return first(v) >= f1; });
}

}  // namespace

size_t index_workspace_bytes(const fhash_grid_desc* g, const int64_t* dims) {
  return build_plan(g, dims).bytes;
}

hipError_t launch_build_index(const fhash_grid_desc* g, const uint64_t* mask,
                              const int64_t* dims, ulonglong2* dir, const int64_t* dir_off,
                              void* ws, uint64_t* counts_host, hipStream_t st) {
  const bool bricks = g->layout == FHASH_LAYOUT_BRICKS;
  const BuildPlan w = build_plan(g, dims);
  char* p = static_cast<char*>(ws);
  auto take = [&p](size_t bytes) {
    char* q = p;
    p += align256(bytes);
    return q;
  };
  const int64_t frame = dims[2] * dims[1] * ((dims[0] + 63) / 64);  // words of the mask
  uint64_t* whole = reinterpret_cast<uint64_t*>(take(w.whole ? frame * dims[3] * 8 : 0));
  uint64_t* X = reinterpret_cast<uint64_t*>(take(w.X * 8));
  uint64_t* Y = reinterpret_cast<uint64_t*>(take(w.Y * 8));
  uint32_t* row_count = reinterpret_cast<uint32_t*>(take(w.rows * 4));
  uint64_t* partial = reinterpret_cast<uint64_t*>(take(w.blk * 8));
  uint64_t* counts = reinterpret_cast<uint64_t*>(take(8 * FHASH_MAX_LEVELS));
  ulonglong2* bricked = reinterpret_cast<ulonglong2*>(take(w.bricks * 16));
  uint64_t *C = X, *bits = Y;  // the passes along t and x write over what they no longer need

  const int T = 256;
  GroupBuild G{};
  G.Sx = dims[0];
  G.Sy = dims[1];
  G.Sz = dims[2];
  G.St = dims[3];
  G.Wm = (dims[0] + 63) / 64;
  for (int k = 0; k < w.groups; ++k) {
    const int l0 = w.first[k], n = w.first[k + 1] - l0;
    int64_t a = 0, b = 0, c = 0, nbits = 0, rows = 0, maxrows = 0, blk = 0;
    for (int j = 0; j < n; ++j) {
      const int32_t* r = g->res[l0 + j];
      const LevelSizes s = level_sizes(r, dims);
      LevelBuild& d = G.lv[j];
      d.rx = r[0];
      d.ry = r[1];
      d.rz = r[2];
      d.rt = r[3];
      d.wv = (r[0] + 63) / 64;
      d.y0 = j == 0 ? 0 : G.lv[j - 1].y0 + G.lv[j - 1].ry;
      d.a = a;
      d.b = b;
      d.c = c;
      d.bits = nbits;
      d.row = rows;
      d.blk = blk;
      d.dir = dir_off[l0 + j];
      a += s.a;
      b += s.b;
      c += s.c;
      nbits += s.bits;
      rows += s.rows;
      blk += s.blk;
      maxrows = std::max(maxrows, s.blk);
    }
    for (G.f0 = 0; G.f0 < G.St; G.f0 += G.nf) {
      G.nf = std::min(w.frames, G.St - G.f0);
      uint64_t* tmask = w.whole ? whole : Y;
      uint64_t* A = w.whole ? X : tmask + G.nf * frame;
      uint64_t* B = w.whole ? Y : A + G.nf * a;
      int64_t zt = 1, tt = 1;  // threads of the passes along z and t, of the level with most
      for (int j = 0; j < n; ++j) {
        LevelBuild& d = G.lv[j];
        slab_vertices(G.St, d.rt, G.f0, G.f0 + G.nf, &d.v0, &d.v1);
        const int64_t zl = G.nf * G.Wm * d.ry, tl = d.rz * G.Wm * d.ry;
        zt = std::max(zt, zl * line_chunks(zl, d.rz));
        tt = std::max(tt, tl * line_chunks(tl, d.v1 - d.v0));
      }
      const int64_t tiles = G.nf * G.Sz * ((G.Sy + 63) / 64) * ((G.Wm + kTileW - 1) / kTileW);
      if (!w.whole || k == 0)
        hipLaunchKernelGGL(transpose_kernel, dim3(grid_for(tiles, 1)), dim3(T), 0, st,
                           mask + G.f0 * frame, tmask, G.nf * G.Sz, G.Sy, G.Wm);
      hipLaunchKernelGGL(or_y_kernel, dim3(grid_for(G.nf * G.Sz * G.Wm, 1)), dim3(T), 0, st, G,
                         G.lv[n - 1].y0 + G.lv[n - 1].ry, tmask, A);
      hipLaunchKernelGGL(or_z_kernel, dim3(grid_for(zt, T), n), dim3(T), 0, st, G, A, B);
      hipLaunchKernelGGL(or_t_kernel, dim3(grid_for(tt, T), n), dim3(T), 0, st, G, B, C);
    }
    // four threads to a row: 2^30 rows are 2^32 threads, which no launch holds
    constexpr int64_t kRowBlocks = (int64_t)1 << 23;
    for (int64_t first = 0; first < maxrows; first += kRowBlocks)
      hipLaunchKernelGGL(rows_kernel, dim3((unsigned)std::min(kRowBlocks, maxrows - first), n),
                         dim3(256), 0, st, G, first, C, bits, row_count, partial);
    if (!bricks) {
      hipLaunchKernelGGL(scan_rows_kernel, dim3(n), dim3(1024), 0, st, G, partial, counts + l0);
      hipLaunchKernelGGL(entries_kernel,
                         dim3((unsigned)((maxrows + kScanThreads / kRows - 1) /
                                         (kScanThreads / kRows)), n),
                         dim3(kScanThreads), 0, st, G, bits, row_count, partial, dir);
    } else {
      const int32_t* r = g->res[l0];
      const LevelSizes s = level_sizes(r, dims);
      hipLaunchKernelGGL(brickify_kernel, dim3(grid_for(s.bwords, T)), dim3(T), 0, st, bits, bricked,
                         (int64_t)r[0], (int64_t)r[1], (int64_t)r[2], (int64_t)r[3],
                         (int64_t)G.lv[0].wv, s.Wb, s.By, s.Bz, s.bwords);
      hipLaunchKernelGGL(popc_block_sums_kernel, dim3((unsigned)s.bnb), dim3(kScanThreads), 0, st,
                         bricked, s.bwords, partial);
      hipLaunchKernelGGL(scan_partials_kernel, dim3(1), dim3(1024), 0, st, partial, s.bnb,
                         counts + l0);
      hipLaunchKernelGGL(write_ranks_kernel, dim3((unsigned)s.bnb), dim3(kScanThreads), 0, st,
                         bricked, s.bwords, partial);
      hipLaunchKernelGGL(dir_interleave_kernel, dim3(grid_for(s.bwords, T)), dim3(T), 0, st,
                         bricked, dir + dir_off[l0], s.Bt * s.Bz * s.By, s.By, s.Wb);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(counts_host, counts, sizeof(uint64_t) * g->n_levels, hipMemcpyDeviceToHost,
                     st);
  if (e != hipSuccess) return e;
  return hipStreamSynchronize(st);
}

}  // namespace fh
