// Fused tesseract encoding + MLP decoder (forward, backward, and forward + MSE
// + backward in one pass).
//
// A wave processes blocks of 16 samples.  Lane l = 16 g + s owns sample s of
// the block and the embedding features 16 a + 4 g + i of it -- exactly the
// features its MFMA B-operand registers carry -- so each lane gathers the
// levels behind those features itself (4/F levels per 16-feature block), the
// encoding lands directly in MLP input registers, and the encoding gradient
// that the MLP backward leaves in the same registers is scattered by the same
// lane for the same levels.  Corner weights are recomputed, never stored.
#pragma once
#include <type_traits>

#include "encode_dev.h"
#include "kernels.h"
#include "mlp_dev.h"
#include "mlp_train_dev.h"

namespace fh {

namespace fused_detail {

// Waves per workgroup: eight in every mode; in a small batch fewer of them take
// blocks (fused_launch), so that it spreads over more CUs.  The forward keeps only
// the decoder weights in LDS; the backward modes also hold the workgroup's
// gradient image and per-wave tiles.  MODE_FWD16: the forward with a 16-bit
// MFMA decoder (inference).
enum { MODE_FWD = 0, MODE_BWD = 1, MODE_TRAIN = 2, MODE_FWD16 = 3 };
constexpr bool is_forward(int mode) { return mode == MODE_FWD || mode == MODE_FWD16; }
constexpr int waves_per_block(int mode) { return (void)mode, 8; }

struct FusedArgs {
  const float4* pos;
  const float* target;  // MODE_TRAIN
  const float* dy;      // MODE_BWD
  int64_t n;
  const int32_t* n_dev;  // forward: NULL, or the sample count (at most n) on the device
  const void* table;
  const float* params;
  float* y;        // MODE_FWD
  float* d_table;  // MODE_BWD / TRAIN
  float* part;     // per-workgroup parameter-gradient partials
  double* loss_sum;
  int64_t P;
  int waves;   // of a workgroup that take blocks (FusedLaunch)
  float coef;  // dL/dy = coef * (y - target)
  int in_w;    // L * F
};

template <int NLMAX, int F, typename T, int INP, bool BRICK>
__device__ __forceinline__ void gather_block(const GridDev& g, const LevelDev* lv, float4 p,
                                             bool valid, const T* table,
                                             float (&xb)[INP / 16][4]) {
  const int lane = threadIdx.x & 63, grp = lane >> 4;
  constexpr int LPB = 4 / F;  // levels per lane per 16-feature block
  if constexpr (BRICK) {
#pragma unroll
    for (int a = 0; a < INP / 16; ++a)
#pragma unroll
      for (int j = 0; j < LPB; ++j) {
        const int l = (16 * a + 4 * grp) / F + j;
        float e[F];
        if (valid && l < g.L) {
          encode_brick_level<F, T>(lv[l], g.dir, g.active != 0, p, table, e, g.tmask);
        } else {
#pragma unroll
          for (int k = 0; k < F; ++k) e[k] = 0.0f;
        }
#pragma unroll
        for (int k = 0; k < F; ++k) xb[a][j * F + k] = e[k];
      }
  } else {
    // the lane's levels two at a time (one more would double the registers of
    // the loads in flight); a level past the last repeats the last one's loads
    constexpr int NLV = (INP / 16) * LPB, NL = NLV < NLMAX ? NLV : NLMAX;
#pragma unroll
    for (int i = 0; i < NLV; i += NL) {
      int l[NL];
      float e[NL][F];
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        l[j] = (16 * ((i + j) / LPB) + 4 * grp) / F + (i + j) % LPB;
#pragma unroll
        for (int k = 0; k < F; ++k) e[j][k] = 0.0f;
      }
      if (valid && l[0] < g.L) {
        int m[NL];
#pragma unroll
        for (int j = 0; j < NL; ++j) m[j] = l[j] < g.L ? l[j] : g.L - 1;
        encode_rows<NL, F, T>(g, lv, m, p, table, e);
      }
#pragma unroll
      for (int j = 0; j < NL; ++j)
#pragma unroll
        for (int k = 0; k < F; ++k)
          xb[(i + j) / LPB][((i + j) % LPB) * F + k] = l[j] < g.L ? e[j][k] : 0.0f;
    }
  }
}

// Scatter of a block's encoding gradient, one level of the lane at a time
// (scatter_rows).  Levels below g.coarse are not added here: their gradient goes
// to g.dxc for the LDS scatter (coarse.hip).  Brick order: 2F consecutive lanes
// own one (sample, level); pass k of 2F gives lane q the sample-level held by
// lane k * (64 / 2F) + q / 2F, whose position and gradient arrive by shuffles.
template <int F, int INP, bool BRICK>
__device__ __forceinline__ void scatter_block(const GridDev& g, const LevelDev* lv, float4 p,
                                              bool valid, int64_t smp,
                                              const float (&dx)[INP / 16][4], float* d_table) {
  const int lane = threadIdx.x & 63, grp = lane >> 4;
  constexpr int LPB = 4 / F;
  if constexpr (!BRICK) {
#pragma unroll
    for (int a = 0; a < INP / 16; ++a)
#pragma unroll
      for (int j = 0; j < LPB; ++j) {
        const int l = (16 * a + 4 * grp) / F + j;  // this lane group's level
        float gr[F];
#pragma unroll
        for (int q = 0; q < F; ++q) gr[q] = dx[a][j * F + q];
        if (valid && l < g.coarse)
#pragma unroll
          for (int q = 0; q < F; ++q) g.dxc[((int64_t)l * g.nsamp + smp) * F + q] = gr[q];
        const bool own = valid && l >= g.coarse && l < g.L;
        if (__ballot(own) != 0) scatter_rows<F>(g, lv[l], p, own, gr, d_table);
      }
    return;
  }
  constexpr int Q = 2 * F, PER = 64 / Q;
  const int r = lane % Q, e = r / F, f = r % F;
#pragma unroll
  for (int a = 0; a < INP / 16; ++a)
#pragma unroll
    for (int j = 0; j < LPB; ++j) {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int m = k * PER + lane / Q;  // source lane (= sample-level)
        const int src_grp = m >> 4;
        const int ls = (16 * a + 4 * src_grp) / F + j;
        float gsrc[F];
#pragma unroll
        for (int q = 0; q < F; ++q) gsrc[q] = __shfl(dx[a][j * F + q], m, 64);
        float4 ps;
        ps.x = __shfl(p.x, m, 64);
        ps.y = __shfl(p.y, m, 64);
        ps.z = __shfl(p.z, m, 64);
        ps.w = __shfl(p.w, m, 64);
        const bool vs = __shfl((int)valid, m, 64) != 0;
        float gval = gsrc[0];
#pragma unroll
        for (int q = 1; q < F; ++q)
          if (f == q) gval = gsrc[q];
        if (ls < g.L && vs)
          scatter_brick_lane<F>(lv[ls], g.dir, g.active != 0, ps, e, f, gval, d_table, g.touch,
                                g.touch_begin, g.gmask);
      }
    }
}

// One workgroup per CU in the backward modes: the decoder weights, the FP32
// gradient image of the workgroup (mlp_train_dev.h) and eight waves' tiles
// share its LDS.  D is the decoder arithmetic: float (FP32 MFMA) or a 16-bit
// type (_Float16 / __bf16 MFMA with FP32 accumulation); the FP32-decoder
// forward is MODE_FWD, the 16-bit one MODE_FWD16.
template <int MODE, int F, typename T, int INP, int H, int NH, typename D, bool BRICK>
__global__ void __launch_bounds__(64 * waves_per_block(MODE))
    __attribute__((amdgpu_waves_per_eu(is_forward(MODE) ? 1 : 2)))
    fused_kernel(GridDev g, FusedArgs A) {
  constexpr int kWaves = waves_per_block(MODE);  // every workgroup's, nw of them take blocks
  const int nw = A.waves;
  constexpr bool FWD = is_forward(MODE);
  if constexpr (FWD) {
    if (A.n_dev != nullptr) {
      A.n = *A.n_dev;
      if (blockIdx.x * (int64_t)(nw * 16) >= A.n) return;  // uniform: nothing to stage for
    }
  }
  constexpr bool D32 = std::is_same<D, float>::value;
  using S = MlpShape<INP, H, NH>;
  using G = GradLds<INP, H, NH>;
  constexpr int WFL = (MODE == MODE_FWD16) ? MlpShapeH<INP, H, NH>::TOTAL_FLOATS
                      : D32               ? S::WFLOATS
                                          : MlpShapeT<INP, H, NH>::TOTAL_FLOATS;
  constexpr int GFL = FWD ? 0 : G::FLOATS;
  constexpr int WS = FWD ? 0
                     : D32 ? train_wave_scratch_f32<INP, H, NH>()
                           : train_wave_scratch_t<INP, H, NH>();
  __shared__ __attribute__((aligned(16))) float lds[WFL + GFL + kWaves * WS + 1];
  __shared__ LevelDev lv[FHASH_MAX_LEVELS];
  if constexpr (MODE == MODE_FWD16)
    load_weights_lds_h<INP, H, NH, D, 64 * kWaves>(lds, A.params, A.in_w);
  else if constexpr (D32)
    load_weights_lds<INP, H, NH, 64 * kWaves>(lds, A.params, A.in_w);
  else
    load_weights_lds_t<INP, H, NH, D, 64 * kWaves>(lds, A.params, A.in_w);
  static_assert(WFL % 4 == 0, "the gradient image is read 16 bytes at a time");
  float* grad = lds + WFL;
  if constexpr (!FWD) grad_lds_zero<INP, H, NH>(grad);
  for (int e = threadIdx.x; e < FHASH_MAX_LEVELS; e += blockDim.x) lv[e] = g.lv[e];
  __syncthreads();
  const T* table = reinterpret_cast<const T*>(A.table);
  const int lane = threadIdx.x & 63, grp = lane >> 4, s = lane & 15;
  const int wib = threadIdx.x >> 6;
  float* scratch = lds + WFL + GFL + wib * WS;
  const int64_t nblk = (A.n + 15) / 16;
  const int64_t nwav = (int64_t)gridDim.x * nw;
  const int64_t wave = (int64_t)blockIdx.x * nw + wib;
  double loss = 0.0;
  for (int64_t b = wib < nw ? wave : nblk; b < nblk; b += nwav) {
    // Keep the decoder weights in LDS rather than in registers across blocks:
    // the compiler would otherwise hoist every layer's weight fragments out of
    // this loop (64 registers per 64x64 layer) and cut the waves per SIMD.
    __asm__ volatile("" ::: "memory");
    const int64_t smp = b * 16 + s;
    const bool valid = smp < A.n;
    const float4 p = valid ? A.pos[smp] : make_float4(0.f, 0.f, 0.f, 0.f);
    float xb[S::INB][4];
    gather_block<FWD ? 1 : 2, F, T, INP, BRICK>(g, lv, p, valid, table, xb);
    float hs[NH][S::HB][4];
    float yv;
    if constexpr (MODE == MODE_FWD16)
      yv = mlp_block_fwd_h<INP, H, NH, D>(lds, xb);
    else if constexpr (D32)
      yv = mlp_block_fwd<INP, H, NH>(lds, xb, hs);
    else
      yv = mlp_block_fwd_t<INP, H, NH, D>(lds, xb, hs);
    if constexpr (FWD) {
      if (grp == 0 && valid) A.y[smp] = yv;
      continue;
    } else {
      float dyv = 0.0f;
      if (MODE == MODE_BWD) {
        dyv = valid ? A.dy[smp] : 0.0f;
      } else {
        const float r = valid ? yv - A.target[smp] : 0.0f;
        dyv = A.coef * r;
        if (grp == 0) loss += (double)r * (double)r;
      }
      float dxb[S::INB][4];
      if constexpr (D32)
        mlp_block_bwd_lds<INP, H, NH>(lds, grad, scratch, xb, hs, dyv, dxb);
      else
        mlp_block_bwd_t<INP, H, NH, D>(lds, grad, reinterpret_cast<D*>(scratch), xb, hs, dyv,
                                       dxb);
      scatter_block<F, INP, BRICK>(g, lv, p, valid, smp, dxb, A.d_table);
    }
  }
  if constexpr (!FWD) {
    __syncthreads();
    grad_lds_write<INP, H, NH>(grad, A.in_w, A.part + (int64_t)blockIdx.x * A.P);
    if (MODE == MODE_TRAIN && A.loss_sum != nullptr) {
      for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off, 64);
      if (lane == 0 && wib < nw) unsafeAtomicAdd(A.loss_sum, loss);
    }
  }
}

// Workgroups of a launch (= decoder-gradient partials of a backward launch) and
// waves of each.  A wave takes one block of 16 samples where the waves allow
// (8192 in the forward, 2048 in the backward).  Eight waves share a workgroup's
// weights and gradient image; a batch of fewer than 2048 blocks spreads over 256
// workgroups first, a CU each: the lookups of 16 samples are about 4,000 line
// requests, one per cycle and CU, so eight waves on one CU and 248 CUs idle
// waited for each other.  1000 points, 8 waves on 8 CUs / a wave on each of 63:
// 33.1 / 23.2 us, 19.1 with the weights staged in one latency.  Every workgroup is
// launched with eight waves all the same, and those without a block only help to
// stage: a workgroup of one wave held the whole decoder in its registers on the
// way to LDS, which set the kernel's register count for every batch (forward of
// 32-64-64-64-1: 234 registers, now 100, two workgroups to a CU).  1000 points
// 19.1 -> 12.8 us, the decodes of four 512 x 512 renders and three point queries
// 9.38 -> 7.22 ms, the training kernel of 20,011 samples 143 -> 132 us.
struct FusedLaunch {
  int64_t blocks;
  int waves;
};
inline FusedLaunch fused_launch(int64_t n, int mode) {
  const int64_t nblk = n > 0 ? (n + 15) / 16 : 1, cap = is_forward(mode) ? 8192 : 2048;
  const int64_t w = nblk < cap ? nblk : cap;
  const int64_t most = waves_per_block(mode), each = (w + 255) / 256;
  const int64_t waves = each < most ? each : most;
  return {(w + waves - 1) / waves, (int)waves};
}

// The most partials that a backward launch of n samples or fewer writes: what a
// workspace is sized for.  The launch's own count falls wherever another wave
// joins each workgroup (256 at 4,096 samples, 129 at 4,097), and a workspace that
// holds a batch has to hold every smaller one.
inline int64_t fused_most_partials(int64_t n) {
  const int64_t nblk = n > 0 ? (n + 15) / 16 : 1;
  return nblk < 256 ? nblk : 256;
}

// The brick slot order is built for the production decoder shapes only
// (32 inputs, hidden width 64, 2 or 3 hidden layers, F = 2 or 4); the host
// rejects other shapes on a brick-ordered index.
template <int F, int INP, int H, int NH>
constexpr bool brick_shape() {
  return (F == 2 || F == 4) && INP == 32 && H == 64 && (NH == 2 || NH == 3);
}

template <int MODE, int F, typename T, int INP, int H, int NH, typename D>
hipError_t fused_t(const GridDev& g, FusedArgs A, float* d_params, hipStream_t st) {
  const FusedLaunch fl = fused_launch(A.n, MODE);
  A.waves = fl.waves;
  const dim3 grid((unsigned)fl.blocks), block(64 * waves_per_block(MODE));
  if (g.lv[0].brick) {
    if constexpr (brick_shape<F, INP, H, NH>())
      hipLaunchKernelGGL((fused_kernel<MODE, F, T, INP, H, NH, D, true>), grid, block, 0, st, g, A);
    else
      return hipErrorNotSupported;
  } else {
    hipLaunchKernelGGL((fused_kernel<MODE, F, T, INP, H, NH, D, false>), grid, block, 0, st, g, A);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || is_forward(MODE)) return e;
  if (g.coarse > 0) {
    e = launch_coarse_scatter(g, reinterpret_cast<const float*>(A.pos), A.n, g.dxc, A.n * F, F,
                              A.d_table, st);
    if (e != hipSuccess) return e;
  }
  return launch_reduce_partials(A.part, fl.blocks, A.P, d_params, st);
}

template <int MODE, int F, typename T, typename D>
hipError_t fused_shape(const GridDev& g, int H, int NH, FusedArgs A, float* d_params,
                       hipStream_t st) {
  const int inp = ((A.in_w + 15) / 16) * 16;
  switch (inp * 1000 + H * 10 + NH) {
#define FH_C(I, HH, N) \
  case I * 1000 + HH * 10 + N: return fused_t<MODE, F, T, I, HH, N, D>(g, A, d_params, st);
    FH_C(16, 32, 1) FH_C(16, 32, 2) FH_C(16, 32, 3)
    FH_C(16, 64, 1) FH_C(16, 64, 2) FH_C(16, 64, 3)
    FH_C(32, 32, 1) FH_C(32, 32, 2) FH_C(32, 32, 3)
    FH_C(32, 64, 1) FH_C(32, 64, 2) FH_C(32, 64, 3)
#undef FH_C
  }
  return hipErrorInvalidValue;
}

// Every feature count, FP32 or FP16 table, decoder arithmetic D.
template <int MODE, typename D>
hipError_t fused_dispatch(const GridDev& g, int H, int NH, fhash_dtype tdt, FusedArgs A,
                          float* d_params, hipStream_t st) {
  if (A.n == 0) return hipSuccess;
  if (tdt == FHASH_F32) {
    switch (g.F) {
      case 1: return fused_shape<MODE, 1, float, D>(g, H, NH, A, d_params, st);
      case 2: return fused_shape<MODE, 2, float, D>(g, H, NH, A, d_params, st);
      case 4: return fused_shape<MODE, 4, float, D>(g, H, NH, A, d_params, st);
    }
  } else {
    switch (g.F) {
      case 1: return fused_shape<MODE, 1, __half, D>(g, H, NH, A, d_params, st);
      case 2: return fused_shape<MODE, 2, __half, D>(g, H, NH, A, d_params, st);
      case 4: return fused_shape<MODE, 4, __half, D>(g, H, NH, A, d_params, st);
    }
  }
  return hipErrorInvalidValue;
}

// Two features per level only (the production configurations).
template <int MODE, typename D>
hipError_t fused_dispatch_f2(const GridDev& g, int H, int NH, fhash_dtype tdt, FusedArgs A,
                             float* d_params, hipStream_t st) {
  if (A.n == 0) return hipSuccess;
  if (g.F != 2) return hipErrorInvalidValue;
  if (tdt == FHASH_F32) return fused_shape<MODE, 2, float, D>(g, H, NH, A, d_params, st);
  return fused_shape<MODE, 2, __half, D>(g, H, NH, A, d_params, st);
}

}  // namespace fused_detail

}  // namespace fh
