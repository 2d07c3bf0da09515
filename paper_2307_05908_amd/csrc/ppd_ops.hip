// Stand-alone early prediction (Sec. 3: the LM classifier applied to an intermediate hidden state, then the
// top-k of its output): one call outside any decoding context, for callers that run the transformer layers
// themselves.  One launch (early_kernel) for rows that fit a wave's registers; longer ones go through gemm_kernel (final norm fused
// into its prologue, every workgroup leaves its own top-k) and a small kernel that merges the lists.
#include "../../include/ppd.h"
#include "ppd_kernels.h"
#include "ppd_launch.h"

#include <string.h>

#include <mutex>
#include <type_traits>

using namespace ppd;

namespace ppd {

template <int T>
__global__ __launch_bounds__(T) void topk_merge_kernel(TopkMergeArgs a) {
  __shared__ float wv[T / WAVE];
  __shared__ int wi[T / WAVE];
  __shared__ int win[MAXM];
  __shared__ float winv[MAXM];
  merge_block_lists<T>(a.pk_val, a.pk_idx, a.nblk, a.kk, a.k, wv, wi, win, winv);
  if ((int)threadIdx.x < a.k) {
    a.ids[threadIdx.x] = win[threadIdx.x];
    if (a.vals) a.vals[threadIdx.x] = winv[threadIdx.x];
  }
}

// ---- the whole early prediction in one launch: norm, classifier, every workgroup's top-k, and the last workgroup's merge of them
struct EarlyArgs {
  const float* h; const void* g; const void* b; const void* W;   // row, gain, bias or null, classifier [V][K]
  float* logits;
  uint2* lists;          // [gridDim.x][MAXM] (value, id) of every workgroup
  int* cnt;              // workgroups done; zero between launches of one grid
  int32_t* ids; float* vals;     // [k]; vals may be null
  int K, V, k, norm, wide;       // wide: gains and biases may be read 16 bytes at a time
  float eps;
};

// arg max by (value descending, id ascending) over a wave, in every lane: rows of 16 lanes by lane-permuting moves, then the four rows
__device__ __forceinline__ void early_best(float& v, int& i) {
  auto take = [&](float ov, int oi) { if (better(ov, oi, v, i)) { v = ov; i = oi; } };
  auto step = [&](auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
    take(dpp_f32<C>(v), __builtin_amdgcn_update_dpp(0, i, C, 0xf, 0xf, false));
  };
  step(std::integral_constant<int, 0xB1>()); step(std::integral_constant<int, 0x4E>());
  step(std::integral_constant<int, 0x141>()); step(std::integral_constant<int, 0x140>());
  const float v0 = v; const int i0 = i;
#pragma unroll
  for (int r = 0; r < 64; r += 16) take(lane_f32(v0, r), __builtin_amdgcn_readlane(i0, r));
}

// A wave owns a run of consecutive classifier rows (gridDim.x * 4 runs of equal length, at most 64 rows) and has the normalised row in
// its registers: lane l the VEC elements 64 VEC j + VEC l .. of every block j.  R rows are requested ahead, a row's blocks each as the
// one before it in the register is consumed.  Nothing waits at a barrier or goes through LDS before the logits are there.
// What bounds it: the stream of the classifier, 5.7 TB/s over the whole call at 32000 x 4096 bf16, on top of some 8 us of launch,
// ramp, top-k and merge.  Few bytes in flight are the faster way: about 8 KiB a wave and four waves a compute unit (32000 x 4096: 46.1 us
// with one row ahead and 256 workgroups, 57.5 with two rows, 47.3 with 512 workgroups).  The logits' order of additions is gemm_kernel's.
// Measured, the whole call, us, two launches (norm and rows through LDS, sets of four rows strided over the grid, a merge launch) / this one: bf16
// 32000 x 4096 59.8 / 45.7, 4000 x 4096 22.7 / 14.8, 32000 x 5120 66.8 / 56.5, 32000 x 2048 42.2 / 27.1, 50272 x 768 38.9 / 20.9, 50272 x 64 34.4 /
// 14.7; fp32 20000 x 2560 47.4 / 37.5, 30000 x 1024 42.0 / 25.8, 50272 x 256 35.5 / 17.2, 1024 x 256 14.8 / 11.5 (the host's part of a call).
template <typename WT, int NB, int R>
__global__ __launch_bounds__(256, 2) void early_kernel(EarlyArgs a) {
  constexpr int VEC = WTr<WT>::VEC, BK = WAVE * VEC, ESZ = 16 / VEC;
  constexpr int SURE = NB <= 4 ? NB - 1 : NB - 2;          // blocks that every K of this instance fills
  __shared__ float hlog[4 * WAVE];
  __shared__ float mv[4 * MAXM]; __shared__ int mi[4 * MAXM];
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K, nw = gridDim.x * 4, gw = blockIdx.x * 4 + wave;
  const int r0 = (int)((int64_t)a.V * gw / nw), r1 = (int)((int64_t)a.V * (gw + 1) / nw);
  float x[NB][VEC];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int k = j * BK + lane * VEC, kc = j < SURE || k < K ? k : 0;
#pragma unroll
    for (int q = 0; q < VEC / 4; ++q) {
      const float4 v = *(const float4*)(a.h + kc + 4 * q);
      x[j][4 * q] = v.x; x[j][4 * q + 1] = v.y; x[j][4 * q + 2] = v.z; x[j][4 * q + 3] = v.w;
    }
  }
  u32x4 w[R][NB];
  // the run as a buffer of its own: what is asked for past its end is not read and comes as zeros
  const unsigned row_bytes = (unsigned)K * ESZ, run_bytes = (unsigned)(r1 - r0) * row_bytes;
  const __amdgpu_buffer_rsrc_t run = __builtin_amdgcn_make_buffer_rsrc((char*)a.W + (size_t)r0 * row_bytes, 0, (int)run_bytes, 0x00020000);
  auto request = [&](int slot, int j, unsigned row) {      // row: its byte offset in the run
    const int k = j * BK + lane * VEC;
    w[slot][j] = __builtin_amdgcn_raw_buffer_load_b128(run, row + (j < SURE || k < K ? (unsigned)(j * 1024 + lane * 16) : 0u), 0, 2);   // 2: non-temporal
  };
  u32x4 gq[NB], bq[NB];
  auto piece = [&](const void* p, int k) -> u32x4 {        // VEC elements as they lie in memory
    if (a.wide) return *(const u32x4*)((const char*)p + (size_t)k * ESZ);
    uint32_t u[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (VEC == 4) u[e] = ((const uint32_t*)p)[k + e];
      else u[e] = ((const uint16_t*)p)[k + 2 * e] | (uint32_t)((const uint16_t*)p)[k + 2 * e + 1] << 16;
    }
    return (u32x4){u[0], u[1], u[2], u[3]};
  };
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int k = j * BK + lane * VEC, kc = j < SURE || k < K ? k : 0;
    gq[j] = piece(a.g, kc);
    bq[j] = a.b ? piece(a.b, kc) : (u32x4){0u, 0u, 0u, 0u};
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) request(i, j, (unsigned)i * row_bytes);
  // statistics: a lane's elements block by block, the blocks' sums one after the other, then the lanes
  float mu = 0.f;
  if (a.norm == 0) {
    float t = 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float u = 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) u += x[j][e];
      t += j < SURE || j * BK + lane * VEC < K ? u : 0.f;
    }
    mu = wave_sum(t) / (float)K;
  }
  float t2 = 0.f;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    float u = 0.f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) { const float d = x[j][e] - mu; u = fmaf(d, d, u); }
    t2 += j < SURE || j * BK + lane * VEC < K ? u : 0.f;
  }
  const float rs = 1.0f / sqrtf(wave_sum(t2) / (float)K + a.eps);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int k = j * BK + lane * VEC;
    const bool in = j < SURE || k < K;
    float gf[VEC], bf[VEC];
    WTr<WT>::unpack(gq[j], gf);
    WTr<WT>::unpack(bq[j], bf);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      float t = (x[j][e] - mu) * rs * gf[e];
      if (a.b) t += bf[e];
      x[j][e] = in ? t : 0.f;
    }
  }
  float mine = -INFINITY;                                  // lane i: the logit of the run's row i
  unsigned ahead = R * row_bytes;
  for (int row = r0; row < r1; row += R) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      float y = 0.f;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        u32x4 q = w[i][j];
        if (j >= SURE && j * BK + lane * VEC >= K) q = (u32x4){0u, 0u, 0u, 0u};
        float wf[VEC];
        WTr<WT>::unpack(q, wf);
#pragma unroll
        for (int e = 0; e < VEC; ++e) y = fmaf(x[j][e], wf[e], y);
        request(i, j, ahead);
      }
      ahead += row_bytes;
      y = wave_sum(y);
      if (lane == row + i - r0) mine = y;
    }
  }
  const int n = r1 - r0;
  if (lane < n) a.logits[r0 + lane] = mine;
  hlog[wave * WAVE + lane] = lane < n ? mine : -INFINITY;
  __syncthreads();
  // this workgroup's top-k, past the L2
  if (wave == 0) {
    float ev[4]; int ei[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int rw = (int)((int64_t)a.V * (blockIdx.x * 4 + u) / nw), re = (int)((int64_t)a.V * (blockIdx.x * 4 + u + 1) / nw);
      ev[u] = hlog[u * WAVE + lane]; ei[u] = rw + lane < re ? rw + lane : 0x7fffffff;
    }
    float lv = -INFINITY; int li = 0x7fffffff;             // lane r keeps the r-th
    for (int r = 0; r < a.k; ++r) {
      float v = -INFINITY; int i = 0x7fffffff;
#pragma unroll
      for (int u = 0; u < 4; ++u) if (better(ev[u], ei[u], v, i)) { v = ev[u]; i = ei[u]; }
      early_best(v, i);
#pragma unroll
      for (int u = 0; u < 4; ++u) if (ei[u] == i) { ev[u] = -INFINITY; ei[u] = 0x7fffffff; }
      if (lane == r) { lv = v; li = i; }
    }
    if (lane < a.k) {
      const unsigned long long e = ((unsigned long long)(unsigned)li << 32) | __float_as_uint(lv);
      __hip_atomic_store((unsigned long long*)(a.lists + (size_t)blockIdx.x * MAXM + lane), e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the list is where every XCD finds it
    if (lane == 0) s_last = atomicInc((unsigned*)a.cnt, gridDim.x - 1) == gridDim.x - 1;     // (the last one leaves zero)
  }
  __syncthreads();
  if (!s_last) return;
  // merge: a thread keeps the heads of two lists (of more, where there are more than 512, one after the other), a wave its best k
  float best_v = -INFINITY; int best_i = 0x7fffffff;       // lane r of a wave: the r-th of its lists so far
  for (int b0 = 0; b0 < (int)gridDim.x; b0 += 512) {
    float lv[2][MAXM]; int li[2][MAXM];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int q = 0; q < MAXM; ++q) {
        lv[u][q] = -INFINITY; li[u][q] = 0x7fffffff;
        const int blk = b0 + u * 256 + tid;
        if (q < a.k && blk < (int)gridDim.x) {
          const unsigned long long e = __hip_atomic_load((unsigned long long*)(a.lists + (size_t)blk * MAXM + q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          lv[u][q] = __uint_as_float((unsigned)e); li[u][q] = (int)(e >> 32);
        }
      }
    float nv = -INFINITY; int ni = 0x7fffffff;
    for (int r = 0; r < a.k; ++r) {
      float v = best_v; int i = best_i;
#pragma unroll
      for (int u = 0; u < 2; ++u) if (better(lv[u][0], li[u][0], v, i)) { v = lv[u][0]; i = li[u][0]; }
      early_best(v, i);
      if (lane == r) { nv = v; ni = i; }
      if (best_i == i) { best_v = -INFINITY; best_i = 0x7fffffff; }
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (li[u][0] == i) {
#pragma unroll
          for (int q = 0; q + 1 < MAXM; ++q) { lv[u][q] = lv[u][q + 1]; li[u][q] = li[u][q + 1]; }
          lv[u][MAXM - 1] = -INFINITY; li[u][MAXM - 1] = 0x7fffffff;
        }
    }
    best_v = nv; best_i = ni;
  }
  if (lane < a.k) { mv[wave * MAXM + lane] = best_v; mi[wave * MAXM + lane] = best_i; }
  __syncthreads();
  if (wave != 0) return;
  float ev = -INFINITY; int ei = 0x7fffffff;
  if (lane < 4 * MAXM && (lane & (MAXM - 1)) < a.k) { ev = mv[lane]; ei = mi[lane]; }
  for (int r = 0; r < a.k; ++r) {
    float v = ev; int i = ei;
    early_best(v, i);
    if (ei == i) { ev = -INFINITY; ei = 0x7fffffff; }
    if (lane == 0) { a.ids[r] = i; if (a.vals) a.vals[r] = v; }
  }
}

}  // namespace ppd

namespace {

constexpr int OPS_GMAX = 512;   // workgroup budget of the head GEMM (as in a context)

struct EarlyTopkPlan {
  int early_grid;        // > 0: workgroups of early_kernel; 0: two launches (rows too long for a wave's registers)
  int grid, KC;
  size_t lds;
  size_t logits_bytes, pk_bytes;   // scratch: logits [vocab] (when the caller takes none), block lists [grid][MAXM] twice
};

template <typename WT, int NB, int R>
hipError_t early_go(const EarlyArgs& a, int grid, hipStream_t stream) {
  hipLaunchKernelGGL((early_kernel<WT, NB, R>), dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}
// blocks of 64 x 16 bytes of a row that an instance holds; 0: more than any does
inline int early_blocks(int d_model, int wdtype) {
  const int nb = (d_model + (wdtype ? 511 : 255)) / (wdtype ? 512 : 256);
  for (const int n : {1, 2, 3, 4, 6, 8, 10}) if (nb <= n) return n;
  return 0;
}
template <typename WT>
hipError_t early_launch(const EarlyArgs& a, int blocks, int grid, hipStream_t stream) {
  switch (blocks) {
    case 1: return early_go<WT, 1, 8>(a, grid, stream);
    case 2: return early_go<WT, 2, 4>(a, grid, stream);
    case 3: return early_go<WT, 3, 3>(a, grid, stream);
    case 4: return early_go<WT, 4, 2>(a, grid, stream);
    case 6: return early_go<WT, 6, 1>(a, grid, stream);
    case 8: return early_go<WT, 8, 1>(a, grid, stream);
    case 10: return early_go<WT, 10, 1>(a, grid, stream);
    default: return hipErrorInvalidValue;
  }
}
// Workgroups: one on a compute unit (two are 3 to 10 % slower, 192 in all up to 8 %), fewer where a wave would have under four rows
// (1000 x 4096: 21.0 us with 16 rows a wave, 13.2 with 4, 15.6 with 1), more where it would have over 64.
int early_grid(int d_model, int vocab, int wdtype) {
  if (!early_blocks(d_model, wdtype)) return 0;
  int g = (vocab + 15) / 16;
  if (g > 256) g = 256;
  if (g < (vocab + HEAD_MAX_ROWS - 1) / HEAD_MAX_ROWS) g = (vocab + HEAD_MAX_ROWS - 1) / HEAD_MAX_ROWS;
  return g;
}

// argument checks shared by the variants; fills the launch plan
int early_topk_plan(int d_model, int vocab, int norm, int wdtype, const void* norm_g, const void* norm_b,
                    const void* head, const float* h, int k, const int32_t* ids_out, EarlyTopkPlan* p) {
  if (d_model < 8 || d_model % 8 || vocab < 1 || norm < 0 || norm > 1 || wdtype < 0 || wdtype > 1) return PPD_EINVAL;
  if (!norm_g || (norm == 0 && !norm_b) || !head || !h || !ids_out) return PPD_EINVAL;
  if (k < 1 || k > PPD_MAX_K || k > vocab) return PPD_EINVAL;
  if (((uintptr_t)h | (uintptr_t)head) & 15) return PPD_EINVAL;
  // one row, four weight rows per wave: the x tile holds the whole reduction length, or chunks of it
  const int span = 1024;   // staged k elements come in multiples of this (a float4 per thread; two k-blocks of 8 bf16 x 64 lanes)
  const int kpad = (d_model + span - 1) / span * span;
  const int kc_cap = GEMM_X_FLOATS / span * span;
  p->KC = kpad < kc_cap ? kpad : kc_cap;
  p->grid = head_grid_valu(vocab, OPS_GMAX);
  p->lds = (GEMM_LDS_HDR + (size_t)p->KC + HEAD_MAX_ROWS) * sizeof(float);
  p->early_grid = early_grid(d_model, vocab, wdtype);
  if (p->early_grid > p->grid) p->grid = p->early_grid;    // (scratch for the lists of either)
  p->logits_bytes = ((size_t)vocab * sizeof(float) + 255) & ~(size_t)255;
  p->pk_bytes = (size_t)p->grid * MAXM * sizeof(float);
  return PPD_OK;
}

// The launch, or the two; logits, pk_val, pk_idx: DEVICE scratch (or the caller's logits buffer), the lists of one launch take the place of
// both pk_val and pk_idx; cnt: a word that is zero
hipError_t early_topk_launch(const EarlyTopkPlan& p, int d_model, int vocab, int norm, float norm_eps, int wdtype,
                             const void* norm_g, const void* norm_b, const void* head, const float* h, int k,
                             float* logits, float* pk_val, int32_t* pk_idx, int* cnt, int32_t* ids_out, float* vals_out,
                             hipStream_t stream) {
  if (p.early_grid > 0) {
    EarlyArgs e;
    e.h = h; e.g = norm_g; e.b = norm == 0 ? norm_b : nullptr; e.W = head; e.logits = logits; e.lists = (uint2*)pk_val; e.cnt = cnt;
    e.ids = ids_out; e.vals = vals_out; e.K = d_model; e.V = vocab; e.k = k; e.norm = norm; e.eps = norm_eps;
    e.wide = ((((uintptr_t)e.g | (uintptr_t)e.b) & 15) == 0);
    return wdtype == 0 ? early_launch<float>(e, early_blocks(d_model, 0), p.early_grid, stream) : early_launch<bf16_t>(e, early_blocks(d_model, 1), p.early_grid, stream);
  }
  GemmArgs a; memset(&a, 0, sizeof a);
  GemmGroup& G = a.g[0];
  G.X = h; G.Rsd = nullptr; G.Y = logits; G.W[0] = head;
  G.ng = norm_g; G.nb = norm == 0 ? norm_b : nullptr; G.M = 1;
  a.K = d_model; a.N[0] = vocab; a.ntot = vocab; a.ldx = d_model; a.ldy = vocab;
  a.norm = norm; a.eps = norm_eps; a.act = 0; a.KC = p.KC;
  a.topk = k; a.pk_val = pk_val; a.pk_idx = pk_idx;
  hipError_t e = wdtype == 0 ? launch_gemm_t<float, false, 4>(stream, a, 1, 0, dim3(p.grid, 1), p.lds)
                             : launch_gemm_t<bf16_t, false, 4>(stream, a, 1, 0, dim3(p.grid, 1), p.lds);
  if (e != hipSuccess) return e;
  TopkMergeArgs t;
  t.pk_val = pk_val; t.pk_idx = pk_idx; t.nblk = p.grid; t.kk = k; t.k = k; t.ids = ids_out; t.vals = vals_out;
  if (merge_threads(t.nblk) == 256) hipLaunchKernelGGL(topk_merge_kernel<256>, dim3(1), dim3(256), 0, stream, t);
  else hipLaunchKernelGGL(topk_merge_kernel<512>, dim3(1), dim3(512), 0, stream, t);
  return hipGetLastError();
}

// ---- the variant that allocates nothing: its scratch is this array (one copy per GPU, held until the process ends)
constexpr int NOALLOC_MAX_VOCAB = 65536;      // logits the array holds
constexpr int NOALLOC_MAX_GRID = 512;         // per-workgroup top-k lists it holds (OPS_GMAX workgroups at most for such vocabularies)
constexpr size_t NOALLOC_LOGITS_BYTES = (size_t)NOALLOC_MAX_VOCAB * sizeof(float);
constexpr size_t NOALLOC_PK_BYTES = (size_t)NOALLOC_MAX_GRID * MAXM * sizeof(float);
// behind them a count of workgroups that are done for every grid, zero to begin with and between launches.  (One for all grids would be
// left at a wrong value for good by calls that overlap against the rule; a grid's own is a whole number of launches' counts whatever overlaps.)
constexpr size_t NOALLOC_CNT_BYTES = (NOALLOC_MAX_GRID + 1) * sizeof(int);
constexpr size_t NOALLOC_SCRATCH_BYTES = NOALLOC_LOGITS_BYTES + 2 * NOALLOC_PK_BYTES + NOALLOC_CNT_BYTES;   // 290 KiB
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[NOALLOC_MAX_DEVICES];     // device address of `scratch` on each GPU, looked up at the first call there

// Device address of the current GPU's copy of the array (in host code the array's name is only a handle for this
// lookup, never an address to pass on).
hipError_t scratch_of_current_device(char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = (char*)g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

extern "C" {

int ppd_early_topk(int d_model, int vocab, int norm, float norm_eps, int wdtype, const void* norm_g,
                   const void* norm_b, const void* head, const float* h, int k, int32_t* ids_out,
                   float* vals_out, float* logits_out, void* hip_stream) {
  EarlyTopkPlan p;
  int rc = early_topk_plan(d_model, vocab, norm, wdtype, norm_g, norm_b, head, h, k, ids_out, &p);
  if (rc) return rc;
  hipStream_t stream = (hipStream_t)hip_stream;
  char* buf = nullptr;
  const size_t lb = logits_out ? 0 : p.logits_bytes;
  hipError_t e = hipMalloc((void**)&buf, lb + 2 * p.pk_bytes + sizeof(int));
  if (e != hipSuccess) { set_global_hip_error((int)e); (void)hipGetLastError(); return e == hipErrorOutOfMemory ? PPD_ENOMEM : PPD_EHIP; }
  float* logits = logits_out ? logits_out : (float*)buf;
  int* const cnt = (int*)(buf + lb + 2 * p.pk_bytes);
  e = hipMemsetAsync(cnt, 0, sizeof(int), stream);
  if (e == hipSuccess)
    e = early_topk_launch(p, d_model, vocab, norm, norm_eps, wdtype, norm_g, norm_b, head, h, k, logits,
                          (float*)(buf + lb), (int32_t*)(buf + lb + p.pk_bytes), cnt, ids_out, vals_out, stream);
  const hipError_t es = hipStreamSynchronize(stream);   // the buffer is freed below: the launches must be done with it
  if (e == hipSuccess) e = es;
  (void)hipFree(buf);
  if (e != hipSuccess) { set_global_hip_error((int)e); (void)hipGetLastError(); return PPD_EHIP; }
  return PPD_OK;
}

int ppd_early_topk_noalloc(int d_model, int vocab, int norm, float norm_eps, int wdtype, const void* norm_g,
                           const void* norm_b, const void* head, const float* h, int k, int32_t* ids_out,
                           float* vals_out, float* logits_out, void* hip_stream) {
  EarlyTopkPlan p;
  int rc = early_topk_plan(d_model, vocab, norm, wdtype, norm_g, norm_b, head, h, k, ids_out, &p);
  if (rc) return rc;
  if (vocab > NOALLOC_MAX_VOCAB || p.grid > NOALLOC_MAX_GRID) return PPD_ELIMIT;
  char* sp = nullptr;
  hipError_t e = scratch_of_current_device(&sp);
  if (e == hipSuccess) {
    // nothing in the array has to start at zero: the GEMM writes every logit and the first k entries of every
    // workgroup's list, and the merge reads only those
    float* logits = logits_out ? logits_out : (float*)sp;
    e = early_topk_launch(p, d_model, vocab, norm, norm_eps, wdtype, norm_g, norm_b, head, h, k, logits,
                          (float*)(sp + NOALLOC_LOGITS_BYTES), (int32_t*)(sp + NOALLOC_LOGITS_BYTES + NOALLOC_PK_BYTES),
                          (int*)(sp + NOALLOC_LOGITS_BYTES + 2 * NOALLOC_PK_BYTES) + p.early_grid, ids_out, vals_out, (hipStream_t)hip_stream);
  }
  if (e != hipSuccess) { set_global_hip_error((int)e); (void)hipGetLastError(); return PPD_EHIP; }
  return PPD_OK;
}

}  // extern "C"
