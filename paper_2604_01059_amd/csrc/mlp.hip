// Training kernels of the scoring network (learned rewrite proposal):
// forward, per-state softmax cross-entropy, backward with a deterministic
// reduction, Adam.  Network and numerics: mlp_dev.h.
#include <algorithm>
#include "zx_internal.h"
#include "mlp_dev.h"

using namespace zxmlp;

namespace {

constexpr int FBS = 64;       // forward block: one wavefront, so that few rows still spread over the CUs
constexpr int BW = 4;         // wavefronts of a backward block, one hidden tile each
constexpr int MAX_PARTS = 1024;  // partial gradients kept per backward call
constexpr int RW = 16;        // wavefronts of a reduction block
constexpr int RCH = 128;      // partials staged at a time

__global__ void mlp_sync_kernel(const float* param, uint16_t* wbf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < IN * HID) {
    const int k = i / HID, n = i - k * HID;
    wbf[Q_W1T + n * IN + k] = to_bf16(param[P_W1 + i]);
  } else if (i < IN * HID + HID) {
    const int n = i - IN * HID;
    wbf[Q_W2 + n] = to_bf16(param[P_W2 + n]);
  }
}

// A operand for rows row0..row0+31 of x; rows >= rows read as zero.
__device__ inline bf16x8 load_a_global(const uint16_t* x, int64_t row0, int64_t rows) {
  const int lane = threadIdx.x & 63;
  const int64_t r = row0 + (lane & 31);
  uint4 q = {0, 0, 0, 0};
  if (r < rows) q = *(const uint4*)(x + r * IN + 8 * (lane >> 5));
  return __builtin_bit_cast(bf16x8, q);
}

__global__ __launch_bounds__(FBS) void mlp_forward_kernel(const uint16_t* wbf, const float* param,
                                                          const uint16_t* x, int64_t rows, float* score) {
  const int lane = threadIdx.x & 63;
  const int64_t row0 = ((int64_t)blockIdx.x * (FBS / 64) + (threadIdx.x >> 6)) * 32;
  if (row0 >= rows) return;
  float s[16];
  hidden32<TILES>(load_a_global(x, row0, rows), wbf, param, s);
  const float sc = sum_hidden(s, param[P_B2]);
  const int64_t r = row0 + acc_row(lane & 15, lane);
  if ((lane & 16) == 0 && r < rows) score[r] = sc;
}

// One wavefront per segment.
__global__ void mlp_loss_kernel(const float* score, const int64_t* cost, const int32_t* seg_off,
                                int32_t n_seg, float* dscore, float* loss) {
  const int lane = threadIdx.x & 63;
  const int seg = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (seg >= n_seg) return;
  const int a = seg_off[seg], b = seg_off[seg + 1];
  // target: even over the present rows of least cost
  int64_t bc = INT64_MAX;
  float mx = -INFINITY;
  for (int r = a + lane; r < b; r += 64) {
    const int64_t cr = cost[r];
    if (cr < 0) continue;
    bc = cr < bc ? cr : bc;
    mx = fmaxf(mx, score[r]);
  }
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t oc = __shfl_xor(bc, o);
    bc = oc < bc ? oc : bc;
    mx = fmaxf(mx, __shfl_xor(mx, o));
  }
  if (bc == INT64_MAX) {  // no present row
    for (int r = a + lane; r < b; r += 64) dscore[r] = 0.f;
    if (lane == 0) loss[seg] = 0.f;
    return;
  }
  float se = 0.f, st = 0.f;
  int nt = 0;
  for (int r = a + lane; r < b; r += 64) {
    if (cost[r] < 0) continue;
    se += expf(score[r] - mx);
    if (cost[r] == bc) {
      st += score[r];
      ++nt;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    se += __shfl_xor(se, o);
    st += __shfl_xor(st, o);
    nt += __shfl_xor(nt, o);
  }
  const float inv = 1.0f / (float)n_seg, tw = 1.0f / (float)nt;
  for (int r = a + lane; r < b; r += 64) {
    float d = 0.f;
    if (cost[r] >= 0) d = (expf(score[r] - mx) / se - (cost[r] == bc ? tw : 0.f)) * inv;
    dscore[r] = d;
  }
  if (lane == 0) loss[seg] = logf(se) + mx - st * tw;
}

// Backward.  Part p of np covers the 32-row chunks p, p + np, ... in order; a
// wavefront does one part of one 32-unit tile of the hidden layer, with its
// partial gradient in registers; the parts are added in order by
// mlp_reduce_kernel.  Every sum runs in one fixed order (over a lane half's
// rows, the two halves, a part's chunks, the parts): the same inputs give the
// same bits, which the optimiser needs, since a gradient that is zero up to
// rounding (b2's always is) still moves its weight by up to the learning rate.
//
// Bound: latency of one chunk and tile (a product on the matrix cores, 16 rows
// of 16 fp32 multiply-adds a lane) for few rows, the fp32 VALU rate for many.
// 2048 rows: 20 us with one wavefront walking all eight tiles of its part and
// a branch around each load, now 13 us; 131072 rows: 59 us.
__global__ __launch_bounds__(64 * BW) void mlp_backward_kernel(const uint16_t* wbf, const float* param,
                                                               const uint16_t* x, const float* dscore,
                                                               int64_t rows, int np, float* ws) {
  __shared__ __align__(16) uint16_t xs[BW][32 * IN];
  constexpr int BPP = TILES / BW;  // blocks per part
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 5, l32 = lane & 31;
  const int p = blockIdx.x / BPP, t = (blockIdx.x % BPP) * BW + wv;
  const int n = 32 * t + l32;
  const bf16x8 w1 = __builtin_bit_cast(bf16x8, *(const uint4*)(wbf + Q_W1T + n * IN + 8 * g));
  const float b1 = param[P_B1 + n];
  const float w2 = from_bf16(wbf[Q_W2 + n]);
  float aw1[IN], ab1 = 0.f, aw2 = 0.f, ab2 = 0.f;
#pragma unroll
  for (int k = 0; k < IN; ++k) aw1[k] = 0.f;
  const int64_t nchunks = (rows + 31) / 32;
  for (int64_t ch = p; ch < nchunks; ch += np) {
    const int64_t row0 = ch * 32;
    const bf16x8 a = load_a_global(x, row0, rows);
    float ds[16], dsum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      // clamped, then selected: a branch would wait for each load in turn
      const int64_t r = row0 + acc_row(i, lane);
      const float v = dscore[r < rows ? r : rows - 1];
      ds[i] = r < rows ? v : 0.f;
    }
    *(uint4*)(&xs[wv][l32 * IN + 8 * g]) = __builtin_bit_cast(uint4, a);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    f32x16 z = {};
    const f32x16 pre = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w1, z, 0, 0, 0);
    float gw2 = 0.f, gb1 = 0.f, gw1[IN];
#pragma unroll
    for (int k = 0; k < IN; ++k) gw1[k] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      dsum += ds[i];
      const float v = pre[i] + b1;
      gw2 += fmaxf(v, 0.f) * ds[i];
      const float dp = v > 0.f ? ds[i] * w2 : 0.f;
      gb1 += dp;
      const uint16_t* xr = &xs[wv][acc_row(i, lane) * IN];
      const uint4 q0 = *(const uint4*)xr, q1 = *(const uint4*)(xr + 8);
      const uint32_t qq[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
      for (int k = 0; k < IN; ++k) gw1[k] += from_bf16((uint16_t)(qq[k >> 1] >> (16 * (k & 1)))) * dp;
    }
    // the two half-waves hold the same hidden unit for different rows
    aw2 += gw2 + __shfl_xor(gw2, 32);
    ab1 += gb1 + __shfl_xor(gb1, 32);
#pragma unroll
    for (int k = 0; k < IN; ++k) aw1[k] += gw1[k] + __shfl_xor(gw1[k], 32);
    ab2 += dsum + __shfl_xor(dsum, 32);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // every lane has read xs before the next chunk's
  }
  float* out = ws + (int64_t)p * NPARAM;
  if (g == 0) {
    out[P_W2 + n] = aw2;
    out[P_B1 + n] = ab1;
  }
#pragma unroll
  for (int k = 0; k < IN / 2; ++k) out[P_W1 + (k + IN / 2 * g) * HID + n] = g ? aw1[k + IN / 2] : aw1[k];
  if (t == 0 && lane == 0) out[P_B2] = ab2;
}

// grad = the parts added in order.  A block owns 64 parameters: one wavefront
// adds the 128 parts in one LDS buffer while the others bring the next 128
// into the other (a thread that loads and adds part after part waits on
// memory for each few: 16 us for 64 parts; now 3.7, and 24 for 1024).
__global__ __launch_bounds__(64 * RW) void mlp_reduce_kernel(const float* ws, int np, float* grad) {
  __shared__ float st[2][RCH][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane, j = i < NPARAM ? i : NPARAM - 1;
  auto bring = [&](int buf, int p0, int w, int nw) {
    const int c = np - p0 < RCH ? np - p0 : RCH;
#pragma unroll 9
    for (int r = w; r < c; r += nw) st[buf][r][lane] = ws[(int64_t)(p0 + r) * NPARAM + j];
  };
  bring(0, 0, wv, RW);
  __syncthreads();
  float s = 0.f;
  for (int p0 = 0, buf = 0; p0 < np; p0 += RCH, buf ^= 1) {
    const int c = np - p0 < RCH ? np - p0 : RCH;
    if (wv == 0) {
#pragma unroll 32
      for (int r = 0; r < c; ++r) s += st[buf][r][lane];
    } else {
      bring(buf ^ 1, p0 + RCH, wv - 1, RW - 1);
    }
    __syncthreads();
  }
  if (wv == 0 && i < NPARAM) grad[i] = s;
}

__global__ void mlp_adam_kernel(float* param, uint16_t* wbf, const float* grad, float* m, float* v,
                                float lr, float b1, float b2, float eps, float bc1, float bc2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= NPARAM) return;
  const float gi = grad[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float p = param[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
  param[i] = p;
  if (i < IN * HID) {
    const int k = i / HID, n = i - k * HID;
    wbf[Q_W1T + n * IN + k] = to_bf16(p);
  } else if (i >= P_W2 && i < P_W2 + HID) {
    wbf[Q_W2 + (i - P_W2)] = to_bf16(p);
  }
}

int bwd_parts(int64_t rows) {
  const int64_t c = (rows + 31) / 32;
  return (int)std::min<int64_t>(std::max<int64_t>(c, 1), MAX_PARTS);
}

}  // namespace

extern "C" zx_status zx_mlp_sync(const zx_mlp* w, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(w && w->param && w->wbf16, "null network");
  hipLaunchKernelGGL(mlp_sync_kernel, dim3((NBF16 + 255) / 256), dim3(256), 0, s, w->param, w->wbf16);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

extern "C" zx_status zx_mlp_forward(const zx_mlp* w, const uint16_t* x, int64_t rows, float* score,
                                    hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(w && w->param && w->wbf16, "null network");
  ZX_CHECK_ARG(rows >= 0, "negative rows");
  if (rows == 0) return ZX_OK;
  ZX_CHECK_ARG(x && score, "null buffer");
  const int64_t waves = (rows + 31) / 32;
  const int64_t blocks = (waves + FBS / 64 - 1) / (FBS / 64);
  ZX_CHECK_ARG(blocks <= INT32_MAX, "too many rows");
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((uint32_t)blocks), dim3(FBS), 0, s, w->wbf16, w->param, x,
                     rows, score);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

extern "C" zx_status zx_mlp_loss(const float* score, const int64_t* cost, const int32_t* seg_off,
                                 int32_t n_seg, float* dscore, float* loss, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(n_seg >= 0, "negative segment count");
  if (n_seg == 0) return ZX_OK;
  ZX_CHECK_ARG(score && cost && seg_off && dscore && loss, "null buffer");
  const int per = 4;
  hipLaunchKernelGGL(mlp_loss_kernel, dim3((n_seg + per - 1) / per), dim3(64 * per), 0, s, score, cost,
                     seg_off, n_seg, dscore, loss);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

extern "C" size_t zx_mlp_workspace_bytes(int64_t rows) {
  if (rows < 0) return 0;
  return (size_t)bwd_parts(rows) * NPARAM * sizeof(float);
}

extern "C" zx_status zx_mlp_backward(const zx_mlp* w, const uint16_t* x, const float* dscore, int64_t rows,
                                     float* grad, void* ws, size_t ws_bytes, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(w && w->param && w->wbf16, "null network");
  ZX_CHECK_ARG(rows >= 0 && grad && ws, "bad argument");
  ZX_CHECK_ARG(rows == 0 || (x && dscore), "null buffer");
  if (ws_bytes < zx_mlp_workspace_bytes(rows)) {
    zx_set_error("workspace too small");
    return ZX_ECAPACITY;
  }
  const int np = bwd_parts(rows);
  hipLaunchKernelGGL(mlp_backward_kernel, dim3(np * (TILES / BW)), dim3(64 * BW), 0, s, w->wbf16, w->param, x, dscore,
                     rows, np, (float*)ws);
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3((NPARAM + 63) / 64), dim3(64 * RW), 0, s, (const float*)ws, np, grad);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

extern "C" zx_status zx_mlp_adam(const zx_mlp* w, const float* grad, float* m, float* v, float lr,
                                 float beta1, float beta2, float eps, int32_t step, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(w && w->param && w->wbf16 && grad && m && v, "null buffer");
  ZX_CHECK_ARG(step >= 1, "step counts from 1");
  ZX_CHECK_ARG(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps > 0.f, "bad Adam constants");
  const float bc1 = (float)(1.0 - std::pow((double)beta1, (double)step));
  const float bc2 = (float)(1.0 - std::pow((double)beta2, (double)step));
  hipLaunchKernelGGL(mlp_adam_kernel, dim3((NPARAM + 63) / 64), dim3(64), 0, s, w->param, w->wbf16, grad,
                     m, v, lr, beta1, beta2, eps, bc1, bc2);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}
