// Detector sampling f = T e (section on the repetition-code example,
// equation detector_sampling; the sampling paragraph after equation
// dets-only): per shot, the error mechanisms that fire are found by
// geometric gaps (drawn for the largest firing probability pmax, then
// thinned to each mechanism's own probability), and every firing
// mechanism's column of T is XORed into the shot's f bits.
//
// A wavefront samples a chunk of consecutive shots, a lane one shot at a
// time; the f rows (fw <= 32 words) of the chunk live in LDS and are written
// out as one contiguous block when ld_out = fw.  Random numbers are
// counter-based SplitMix64 (Steele, Lea, Flood, OOPSLA 2014): draw t of shot s is mix64(seed + (s 2^32 + t + 1)
// GAMMA).  Per candidate: one draw for the gap, G = floor(ln U / ln(1 -
// pmax)), U = ((u >> 11) + 1) 2^-53 (no gap draw when pmax = 1), and one draw
// v for thinning: fire iff (v >> 11) < floor(p_j / pmax 2^53).  The values are
// those of fp64; gap_of decides most gaps in fp32 where that gives the same.
#include "zx_internal.h"

namespace {

constexpr int DS_PREP = 1024;     // threads of the preparation
constexpr int DS_BS = 512;        // threads of the sampler
constexpr int DS_TAB_MAX = 4096;  // mechanisms whose records go into LDS (64 KiB)
// CUs of the card and LDS bytes a CU, for the launch's shape: asking the runtime
// for them takes 0.3 of the 11 us of a small call.  With fewer CUs the chunks
// wait their turn.
constexpr int DS_CUS = 256;
constexpr int DS_LDS = 160 * 1024;
constexpr int DS_CHUNK_WORDS = 1024;  // f words of a wavefront's chunk in LDS (at least a row per lane)
constexpr int DS_MAX_FW = 32;

struct DetWs {
  ZxWsHeader hdr;      // status
  double pmax, log1m;  // largest probability, ln(1 - pmax)
  int32_t valid;
  int32_t pad[59];
  // followed by uint64_t thr[n_err]
};
static_assert(sizeof(DetWs) % 256 == 0, "workspace header size");

__device__ __forceinline__ uint64_t sm_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// largest probability, its log, the thinning thresholds; one workgroup
// Also validates the model: col_ptr non-decreasing from 0 to nnz, every
// col_idx entry in [0, n_f), every probability in [0, 1]; otherwise the
// status becomes ZX_EINVAL and no shot is sampled (rows are written as zero).
__global__ __launch_bounds__(DS_PREP) void det_prep_kernel(const int32_t* __restrict__ col_ptr,
                                                         const int32_t* __restrict__ col_idx, int64_t nnz,
                                                         const double* __restrict__ prob, int32_t n_err,
                                                         int32_t n_f, DetWs* ws, uint64_t* __restrict__ thr) {
  __shared__ double red[DS_PREP / 64];
  double mx = 0.0;
  int b = 0;
  for (int j = threadIdx.x; j < n_err; j += DS_PREP) {
    const double p = prob[j];
    if (!(p >= 0.0 && p <= 1.0)) b = 1;
    else mx = fmax(mx, p);
    if (col_ptr[j] > col_ptr[j + 1]) b = 1;
  }
  if (threadIdx.x == 0 && (col_ptr[0] != 0 || (int64_t)col_ptr[n_err] != nnz)) b = 1;
  for (int64_t q = threadIdx.x; q < nnz; q += DS_PREP)
    if (col_idx[q] < 0 || col_idx[q] >= n_f) b = 1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  const bool bad = __syncthreads_or(b);
  double pmax = red[0];
#pragma unroll
  for (int w = 1; w < DS_PREP / 64; ++w) pmax = fmax(pmax, red[w]);
  const double two53 = 9007199254740992.0;
  if (bad) {
    if (threadIdx.x == 0) {
      ws->hdr.status = ZX_EINVAL;
      ws->valid = 0;
    }
    return;
  }
  for (int j = threadIdx.x; j < n_err; j += DS_PREP)
    thr[j] = pmax > 0.0 ? (uint64_t)(prob[j] / pmax * two53) : 0ull;
  if (threadIdx.x == 0) {
    ws->hdr.status = 0;
    ws->pmax = pmax;
    ws->log1m = log1p(-pmax);  // log(1 - pmax) would round to 0 below pmax = 2^-53
    ws->valid = 1;
  }
}

// Gap to the next candidate, exactly floor(log(U) / log1m) of the fp64
// functions for U = u 2^-53, or `rem` when that leaves the `rem` mechanisms
// that are left.  fp32 decides where it can: with x = fp32(U) and the
// hardware log2 (relative error below 2^-23 over all fp32 of [2^-53, 1],
// compared value by value), q = log2(x) / log2(1 - pmax) is within
// 2 2^-23 q + 2^-23.4 / |log2(1 - pmax)| of the true quotient, of which eps
// takes 3 2^-23 and 2^-23; the fp64 result's own error is far below the rest.
// Only where q +- eps holds a whole number (4 lanes in 10^4 at most at
// pmax = 1.5e-3), or where something is not finite, does fp64 run.
__device__ __forceinline__ int gap_of(uint64_t u, float inv, double log1m, int rem) {
  const double U = (double)u / 9007199254740992.0;
  const float q = __builtin_amdgcn_logf((float)U) * inv;
  const float eps = fmaf(q, 0x1.8p-22f, -inv * 0x1p-23f);
  const float lo = q - eps, hi = q + eps;
  if (lo > (float)rem) return rem;
  const float fl = floorf(lo);
  if (fl == floorf(hi) && fl >= 0.f) return fl < 0x1p31f && (int)fl < rem ? (int)fl : rem;
  const double g = floor(log(U) / log1m);
  return g < (double)rem ? (int)g : rem;  // a NaN quotient ends the shot too
}

// Bound: the arithmetic of the walk (two 64-bit mixes a candidate), so the
// kernel keeps lanes busy and cheap.  A wavefront takes `chunk` shots; a lane
// whose shot has ended takes the chunk's next one, so a wavefront runs for
// the mean number of candidates and not for the largest of 64.  The gap is
// decided in fp32 (gap_of).  A mechanism is one 16-byte record (threshold, number
// of f bits, up to four of them), built in LDS once per workgroup where all
// fit (TAB), so a candidate costs one load and no chain of three.  16.8 M
// shots of 193 bits, 641 mechanisms, 0.96 candidates a shot: 497 us under the
// profiler with a shot per lane, fp64 logarithms and the chain of loads; now
// 176 (whole calls without it 445 and 168).
template <bool TAB>
__global__ __launch_bounds__(DS_BS) void det_sample_kernel(const int32_t* __restrict__ col_ptr,
                                                           const int32_t* __restrict__ col_idx,
                                                           const DetWs* __restrict__ ws,
                                                           const uint64_t* __restrict__ thr, int32_t n_err,
                                                           int32_t fw, int32_t chunk, uint64_t seed, int64_t shot0,
                                                           int64_t n_shots, uint64_t* __restrict__ out,
                                                           int64_t ld_out) {
  extern __shared__ __attribute__((aligned(16))) uint64_t lds[];  // records, then [waves][chunk][fw]
  constexpr uint32_t MORE = 7;  // more f bits than a record holds
  uint4* const tab = (uint4*)lds;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t* const rows = lds + (TAB ? 2 * n_err : 0) + (size_t)wv * chunk * fw;
  for (int x = lane; x < chunk * fw; x += 64) rows[x] = 0;
  const bool valid = ws->valid != 0;
  if (TAB && valid) {
    for (int j = threadIdx.x; j < n_err; j += DS_BS) {
      const int q0 = col_ptr[j], cnt = col_ptr[j + 1] - q0;
      uint64_t bits = 0;
      if (cnt > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) bits |= (uint64_t)(uint32_t)col_idx[q0 + (q < cnt ? q : cnt - 1)] << (16 * q);
      }
      const uint64_t t = thr[j] | (uint64_t)(cnt <= 4 ? (uint32_t)cnt : MORE) << 54;  // thr <= 2^53
      tab[j] = make_uint4((uint32_t)t, (uint32_t)(t >> 32), (uint32_t)bits, (uint32_t)(bits >> 32));
    }
  }
  __syncthreads();
  const double pmax = ws->pmax, log1m = ws->log1m;
  const bool run = valid && pmax > 0.0;
  const float inv = (float)(0.6931471805599453 / log1m);  // 1 / log2(1 - pmax)
  const uint64_t gamma = 0x9E3779B97F4A7C15ull;
  const int64_t n_chunks = (n_shots + chunk - 1) / chunk;
  const int64_t stride = (int64_t)gridDim.x * (DS_BS / 64);
  for (int64_t ch = (int64_t)blockIdx.x * (DS_BS / 64) + wv; ch < n_chunks; ch += stride) {
    const int64_t first = ch * chunk;
    const int cnt = (int)(n_shots - first < chunk ? n_shots - first : chunk);
    const uint64_t base = seed + ((uint64_t)(shot0 + first) << 32) * gamma;  // draw t of shot i: base + (2^32 i + t + 1) gamma
    int shot = lane, next = 64;
    bool act = run && shot < cnt;
    uint64_t state = base + ((uint64_t)shot << 32) * gamma;
    int pos = 0;
    while (__ballot(act)) {
      if (pmax < 1.0) {
        state += gamma;
        pos += gap_of((sm_mix(state) >> 11) + 1, inv, log1m, n_err - pos);
      }
      const bool end = act && pos >= n_err;
      if (act && !end) {
        state += gamma;
        const uint64_t v = sm_mix(state) >> 11;
        uint32_t* const row = (uint32_t*)(rows + (size_t)shot * fw);
        uint64_t t;
        uint32_t nb = MORE;
        uint2 bits = {0, 0};
        if (TAB) {
          const uint4 r = tab[pos];
          t = r.x | (uint64_t)(r.y & 0x3fffffu) << 32;
          nb = r.y >> 22;
          bits = {r.z, r.w};
        } else {
          t = thr[pos];
        }
        if (v < t) {
          if (nb != MORE) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint32_t bi = ((q < 2 ? bits.x : bits.y) >> (16 * (q & 1))) & 0xffffu;
              if (q < (int)nb) atomicXor(row + (bi >> 5), 1u << (bi & 31));
            }
          } else {
            const int q1 = col_ptr[pos + 1];
            for (int q = col_ptr[pos]; q < q1; ++q) {
              const int bi = col_idx[q];
              atomicXor(row + (bi >> 5), 1u << (bi & 31));
            }
          }
        }
        pos += 1;
      }
      const uint64_t m = __ballot(end);
      if (end) {
        shot = next + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        act = shot < cnt;
        state = base + ((uint64_t)shot << 32) * gamma;
        pos = 0;
      }
      next += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int words = cnt * fw;
    if (ld_out == fw) {
      uint64_t* const o = out + first * fw;
      for (int x = lane; x < words; x += 64) {
        o[x] = rows[x];
        rows[x] = 0;
      }
    } else {
      for (int x = lane; x < words; x += 64) {
        const int r = x / fw;
        out[(first + r) * ld_out + (x - r * fw)] = rows[x];
        rows[x] = 0;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

}  // namespace

extern "C" size_t zx_detector_workspace_bytes(int32_t n_err) {
  if (n_err < 0) return 0;
  return sizeof(DetWs) + (((size_t)n_err * 8 + 255) & ~size_t(255));
}

extern "C" zx_status zx_detector_sample(const int32_t* col_ptr, const int32_t* col_idx, int64_t nnz,
                                        const double* prob, int32_t n_err, int32_t n_f, uint64_t seed,
                                        int64_t shot0, int64_t n_shots, uint64_t* out, int64_t ld_out, void* ws,
                                        size_t ws_bytes, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(out && ws && col_ptr, "null argument");
  ZX_CHECK_ARG(n_err >= 0 && n_f > 0 && n_shots > 0 && shot0 >= 0 && nnz >= 0, "bad sizes");
  ZX_CHECK_ARG(n_err == 0 || prob, "null probabilities");
  ZX_CHECK_ARG(nnz == 0 || col_idx, "null col_idx");
  const int fw = (n_f + 63) / 64;
  ZX_CHECK_ARG(ld_out >= fw, "ld_out %lld < %d", (long long)ld_out, fw);
  ZX_CHECK_ARG(((uintptr_t)ws & 255) == 0, "workspace must be 256-byte aligned");
  ZX_CHECK_ARG(shot0 + n_shots <= (1ll << 31), "shot index beyond 2^31");
  if (fw > DS_MAX_FW) {
    zx_set_error("n_f=%d beyond %d f bits per shot", n_f, 64 * DS_MAX_FW);
    return ZX_ECAPACITY;
  }
  if (ws_bytes < zx_detector_workspace_bytes(n_err)) {
    zx_set_error("workspace %zu < %zu bytes", ws_bytes, zx_detector_workspace_bytes(n_err));
    return ZX_ECAPACITY;
  }
  DetWs* W = (DetWs*)ws;
  uint64_t* thr = (uint64_t*)((uint8_t*)ws + sizeof(DetWs));
  hipLaunchKernelGGL(det_prep_kernel, dim3(1), dim3(DS_PREP), 0, s, col_ptr, col_idx, nnz, prob, n_err, n_f, W, thr);
  ZX_HIP(hipGetLastError());
  // shots per chunk: at least one a lane; more where the rows are short, as
  // long as a chunk for each wavefront of two workgroups a CU is left
  constexpr int waves = DS_BS / 64;
  const int64_t per_wave = n_shots / ((int64_t)DS_CUS * 2 * waves);
  int64_t chunk = DS_CHUNK_WORDS / fw;
  if (chunk > per_wave) chunk = per_wave;
  chunk = chunk < 64 ? 64 : chunk / 64 * 64;
  const bool tab = n_err <= DS_TAB_MAX && 16 * n_err + waves * chunk * fw * 8 <= DS_LDS;
  const size_t lds = (tab ? 16 * (size_t)n_err : 0) + (size_t)waves * chunk * fw * 8;
  const int64_t want = (n_shots + waves * chunk - 1) / (waves * chunk);
  const int64_t held = (int64_t)DS_CUS * (lds <= (size_t)DS_LDS / 4 ? 4 : (size_t)DS_LDS / lds);
  const int64_t blocks = want < held ? want : held;
  const void* fn = tab ? (const void*)det_sample_kernel<true> : (const void*)det_sample_kernel<false>;
  if (lds > 64 * 1024) ZX_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, DS_LDS));
  if (tab)
    hipLaunchKernelGGL(det_sample_kernel<true>, dim3((unsigned)blocks), dim3(DS_BS), lds, s, col_ptr, col_idx, W, thr,
                       n_err, fw, (int)chunk, seed, shot0, n_shots, out, ld_out);
  else
    hipLaunchKernelGGL(det_sample_kernel<false>, dim3((unsigned)blocks), dim3(DS_BS), lds, s, col_ptr, col_idx, W, thr,
                       n_err, fw, (int)chunk, seed, shot0, n_shots, out, ld_out);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

extern "C" zx_status zx_detector_status(const void* ws, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(ws, "null workspace");
  ZX_HIP(hipStreamSynchronize(s));
  int32_t st = 0;
  ZX_HIP(hipMemcpy(&st, ws, 4, hipMemcpyDeviceToHost));
  return st;
}
