// HIP kernels of the PPD decode path for gfx950 (64-wide wavefronts).
//
// Every kernel takes up to two row groups per launch.  In a pipelined step of
// the parallel phase (Algorithm 2, the "in parallel" block) group 0 is the
// main token at layer dbar+j (one row) and group 1 holds the k candidate
// tokens at layer j (k rows): two different layers' weights, each streamed
// from HBM once for all rows of its group.
//
// Bit-reproducibility rule: the arithmetic that produces one output row
// depends only on that row's inputs, never on how many rows share the launch,
// on the group, on the grid, or on where the row's own key/value is stored.
// Each reduction has one fixed order (lane -> k mapping, butterfly across
// lanes, waves in index order, position chunks in index order), and every
// multiply-add is an explicit fmaf.  This is what makes a candidate row's
// layers 1..d-dbar equal, bit for bit, to the layers plain decoding would run
// on the same token.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ppd {

struct bf16_t { uint16_t v; };
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int WAVE = 64;
constexpr int GEMM_THREADS = 256;   // 4 waves
constexpr int GEMM_WAVES = GEMM_THREADS / WAVE;
constexpr int GEMM_X_FLOATS = 15360; // floats of the LDS x tile (60 KB): 15 float4 per thread
constexpr int GEMM_BATCH = 8;       // 16-byte loads per lane in one register batch: WR weight rows x 8/WR k-blocks
constexpr int GEMM_AHEAD = 3;       // batches requested ahead of the arithmetic (ring of four register buffers)
constexpr int GEMM_LDS_HDR = 80;    // floats in front of the x tile: norm statistics and their reduction scratch
constexpr int HEAD_MAX_ROWS = 256;  // logits one workgroup of the head GEMM may produce (block top-k buffer)
constexpr int ATT_THREADS = 256;
constexpr int ATT_WAVES = ATT_THREADS / WAVE;
constexpr int ATT_CHUNK = 64;       // positions per workgroup; chunk c covers [c*64, (c+1)*64)
constexpr int MAXM = 8;

// Round state in device memory, written by the tiny state kernel behind a prompt and by the
// selection kernels of a round; read by every kernel that needs a position or a token id.
struct DevState {
  int32_t pos;        // absolute position of the main token x_t (a round's final selection leaves the next round's)
  int32_t next_tok;   // id of x_t
  int32_t result[2];  // token x_{t+1}, match_idx of the last final selection
  int32_t cand[MAXM]; // early top-k ids
  int32_t cand_next[2][MAXM]; // candidates of the next round, predicted at the end of a matching round, in the half its position's parity selects
  int32_t sampled;    // final prediction drawn by the sampling kernel (sampling-based variants)
  uint32_t sel_done;   // workgroups of a final selection that are done (zero between launches)
  int32_t seq;         // rounds finished since the context was created (the host waits for the next value)
  int32_t aborted;     // a workgroup of the round's one-launch chain of layers gave up waiting: the round's results are void
};

__device__ __forceinline__ float bf16_to_f32(uint16_t u) { return __uint_as_float(((uint32_t)u) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <typename WT> struct WTr;
template <> struct WTr<float> {
  static constexpr int VEC = 4;
  __device__ static __forceinline__ void unpack(const u32x4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  __device__ static __forceinline__ float load1(const void* p, size_t i) { return ((const float*)p)[i]; }
  __device__ static __forceinline__ float round(float x) { return x; }
  __device__ static __forceinline__ void store1(void* p, size_t i, float x) { ((float*)p)[i] = x; }
};
template <> struct WTr<bf16_t> {
  static constexpr int VEC = 8;
  __device__ static __forceinline__ void unpack(const u32x4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
  }
  __device__ static __forceinline__ float load1(const void* p, size_t i) { return bf16_to_f32(((const uint16_t*)p)[i]); }
  __device__ static __forceinline__ float round(float x) { return bf16_to_f32(f32_to_bf16(x)); }
  __device__ static __forceinline__ void store1(void* p, size_t i, float x) { ((uint16_t*)p)[i] = f32_to_bf16(x); }
};

// weights and cached keys/values are read once per launch: stream them past the caches
__device__ __forceinline__ u32x4 ld_stream(const void* p) { return __builtin_nontemporal_load((const u32x4*)p); }

// 64 lanes x 16 bytes from per-lane global addresses to LDS at lds_dst + 16 * lane (lds_dst is the same
// for the whole wave and goes through M0).  Written as assembly so that the wait for it stays ours:
// the request counts in vmcnt like any load, and loads return in order.
// (A readfirstlane on the address kept the compiler from folding the cast's null check, three scalar instructions per request:
// the prompt GEMM's staging wave fell behind with it, 7B shape 160 rows 9.75 -> 10.4 ms.)
__device__ __forceinline__ void dma16(const void* src, void* lds_dst) {
  const unsigned la = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_dst;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(la) : "memory", "m0");
}

// Wave reductions on the data-parallel-primitive path: inside each row of 16 lanes with four
// lane-permuting adds (partner lanes compute a + b and b + a, so all 16 agree), then the four row
// results in row order.  Every lane returns the same value.
template <int CTRL> __device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_f32(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f32<0xB1>(v);     // quad_perm [1,0,3,2]
  v += dpp_f32<0x4E>(v);     // quad_perm [2,3,0,1]
  v += dpp_f32<0x141>(v);    // row_half_mirror
  v += dpp_f32<0x140>(v);    // row_mirror
  return ((lane_f32(v, 0) + lane_f32(v, 16)) + lane_f32(v, 32)) + lane_f32(v, 48);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));
  v = fmaxf(v, dpp_f32<0x4E>(v));
  v = fmaxf(v, dpp_f32<0x141>(v));
  v = fmaxf(v, dpp_f32<0x140>(v));
  return fmaxf(fmaxf(lane_f32(v, 0), lane_f32(v, 16)), fmaxf(lane_f32(v, 32), lane_f32(v, 48)));
}
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }
// arg max by (value descending, id ascending) over a wave; every lane ends with the winner
__device__ __forceinline__ void wave_best(float& v, int& i) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    float ov = __shfl_xor(v, o, WAVE); int oi = __shfl_xor(i, o, WAVE);
    if (better(ov, oi, v, i)) { v = ov; i = oi; }
  }
}

// ------------------------------------------------------------------ round state
// (plain, non-template kernels are compiled into the engine's translation unit only)
#ifdef PPD_ENGINE_TU
// streaming-read probe: every thread walks the buffer with U 16-byte non-temporal loads in flight
template <int U>
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* p, size_t n16, uint32_t* sink) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (; i + (U - 1) * stride < n16; i += U * stride) {
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = ld_stream(p + i + u * stride);
#pragma unroll
    for (int u = 0; u < U; ++u) acc ^= v[u];
  }
  for (; i < n16; i += stride) acc ^= ld_stream(p + i);
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) *sink = acc.x;   // keeps the loads alive; practically never taken
}
__global__ void set_state_kernel(DevState* ds, int pos, int tok) {
  if (threadIdx.x == 0) { ds->pos = pos; if (tok >= 0) ds->next_tok = tok; }
}
// One row of activations to another place (x_0's, from the prompt pass to the first round)
__global__ __launch_bounds__(256) void keep_row_kernel(float* to, const float* row, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) to[i] = row[i];
}
// First launch of a round with a one-launch chain of layers: the buffers of its steps' outputs are marked empty (ex), and the
// activation rows are kept (save) so that the round can be run again if the launch has to give up; restore: this is
// that second run.  (Other rounds begin with their first layer: what a round finds in the state and in row 0 the one before left there.)
struct BeginArgs {
  DevState* ds;
  u32x4* ex; size_t n16; uint32_t empty;     // 16-byte pieces to fill
  float* h; float* save; int nsave; int restore;
};
__global__ __launch_bounds__(256) void begin_round_kernel(BeginArgs a) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  if (t == 0) a.ds->aborted = 0;
  const u32x4 e = {a.empty, a.empty, a.empty, a.empty};
  for (size_t i = t; i < a.n16; i += stride) a.ex[i] = e;
  for (size_t i = t; i < (size_t)a.nsave; i += stride) { if (a.restore) a.h[i] = a.save[i]; else a.save[i] = a.h[i]; }
}
#endif

// ------------------------------------------------------------------ embedding
// Row set-up (start of the main process, start of every sub-process): h_0 = E[token] (+ P[pos]).
struct EmbedArgs {
  const void* tok_emb; const void* pos_emb;   // pos_emb null for RoPE models
  const int32_t* ids;   // DEVICE: token id of row r is ids[r]
  const DevState* ds;
  float* h;             // [rows][d_model]
  int rows, d_model, pos_off;   // the rows sit at position ds->pos + pos_off (+ r * pos_step for row r)
  int pos_step;
  int vocab;            // rows of tok_emb
};
// An id outside the vocabulary can only come out of a selection over logits that are not numbers (every comparison
// with a NaN fails, and the "nothing found" id stays): it must never become an address.
__device__ __forceinline__ int id_in_vocab(int id, int vocab) { return (unsigned)id < (unsigned)vocab ? id : 0; }
template <typename WT>
__device__ __forceinline__ void embed_rows(const EmbedArgs& a, int r, int i0, int stride) {
  const int tok = id_in_vocab(a.ids[r], a.vocab);
  int pos = a.ds->pos + a.pos_off + r * a.pos_step;
  for (int i = i0; i < a.d_model; i += stride) {
    float v = WTr<WT>::load1(a.tok_emb, (size_t)tok * a.d_model + i);
    if (a.pos_emb) v += WTr<WT>::load1(a.pos_emb, (size_t)pos * a.d_model + i);
    a.h[(size_t)r * a.d_model + i] = v;
  }
}
template <typename WT>
__global__ void embed_kernel(EmbedArgs a) {
  embed_rows<WT>(a, blockIdx.y, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// ------------------------------------------------------------------ skinny GEMM
// Y[m][n] = epilogue( sum_k norm(X)[m][k] * W[n][k] ), M <= 8 rows per group and workgroup.
// The layer forward of the main process and of the sub-processes (Algorithm 2);
// the sub-processes' k rows share one pass over their layer's weights.
//
// A workgroup requests its group's input rows, then the first three register
// batches of its weight rows, and only then normalises the rows and puts them
// in LDS: a wave's loads return in order, so the rows arrive first and the
// weights stream in behind them.  Its four waves each take sets of weight rows,
// read with 16-byte non-temporal loads three batches ahead of the arithmetic.
struct GemmGroup {
  const float* X;     // [M][ldx] input rows (before the fused norm)
  const float* Rsd;   // residual rows [M][ldy] added in the epilogue, or null
  float* Y;           // [M][ldy]
  const void* W[3];   // up to three row segments (Q,K,V); for SwiGLU W[0] = gate, W[1] = up, paired row by row
  const void* B[3];   // biases per segment or null
  const void* ng; const void* nb;  // gain / bias of the fused norm
  int M;
};
struct GemmArgs {
  GemmGroup g[2];
  int K;            // reduction length (multiple of VEC)
  int N[3];         // rows per segment
  int ntot;         // logical output rows (= N0+N1+N2, or N0 for SwiGLU)
  int ldx, ldy;
  int norm;         // -1 none, 0 LayerNorm, 1 RMSNorm
  float eps;
  int act;          // 0 none, 1 GELU, 2 ReLU, 3 SwiGLU (pairs W[0], W[1])
  int KC;           // K elements staged in LDS at a time (multiple of the batch span (8/WR)*64*VEC)
  int topk;         // > 0: LM-head launch; every workgroup also writes its own top-k (value, id)
  float* pk_val; int32_t* pk_idx;   // [gridDim.x][MAXM] block candidates (topk > 0)
};

__device__ __forceinline__ float gelu_erf(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752440f)); }
__device__ __forceinline__ float silu(float u) { return u / (1.0f + expf(-u)); }

// WR: weight rows a wave streams together (4, or 2 when the matrix has few rows per wave);
// a register batch is always 8 loads per lane: WR rows x (8 / WR) k-blocks.
// GF: one row's gains are requested with the row (see gains_first).
template <typename WT, int MT, bool PAIRED, int WR, bool GF>
__device__ __forceinline__ void gemm_body(const GemmArgs& a, const GemmGroup& G, float* lds, int r0 = 0) {
  constexpr int VEC = WTr<WT>::VEC;
  constexpr int BK = WAVE * VEC;                 // k elements per block
  constexpr int NBK = GEMM_BATCH / WR;           // k-blocks per batch
  constexpr int SPAN = NBK * BK;                 // k elements per batch
  constexpr int LR = PAIRED ? WR / 2 : WR;       // logical rows per set
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int M = MT == MAXM && G.M - r0 > MT ? MT : G.M - r0, K = a.K, KC = a.KC;
  float4* xs4 = (float4*)(lds + GEMM_LDS_HDR);  // [MT][KC/4] float4; for VEC == 8 the two halves of every 8-group are split

  const int nsets = (a.ntot + LR - 1) / LR;
  const int nwaves = gridDim.x * GEMM_WAVES;
  const int gw = blockIdx.x * GEMM_WAVES + wave;
  const int nbps = (K + SPAN - 1) / SPAN;                  // batches per set
  const int bpc = KC / SPAN;                               // batches per staged chunk
  const bool single = KC >= K;
  // Sets gw, gw + nwaves, ... belong to this wave.  When the reduction length is staged in
  // chunks the waves of a workgroup meet at barriers, so they all run the same number of sets
  // (a wave without a set left repeats its last one and drops the result).
  const int nmine = gw < nsets ? (nsets - gw + nwaves - 1) / nwaves : 0;
  const int nit = single ? nmine : (nsets + nwaves - 1) / nwaves;
  const int Q = nit * nbps;

  // ---- load side: runs GEMM_AHEAD batches ahead of the arithmetic.  Every request is issued
  // unconditionally (lanes past the end of a row re-read its last 16 bytes and zero them), so
  // the loads of one wave return in a known order and the arithmetic waits for its own batch only.
  const char* wp[WR];
  int l_it = 0, l_b = 0;
  auto set_rows = [&](int it) {
    int s = gw + it * nwaves;
    if (s >= nsets) s = nsets - 1;
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      int n = s * LR + r;
      int nc = n < a.ntot ? n : a.ntot - 1;
      if (PAIRED) {
        wp[2 * r] = (const char*)G.W[0] + (size_t)nc * K * sizeof(WT);
        wp[2 * r + 1] = (const char*)G.W[1] + (size_t)nc * K * sizeof(WT);
      } else {
        int seg = 0, loc = nc;
        if (loc >= a.N[0]) { loc -= a.N[0]; seg = 1; if (loc >= a.N[1]) { loc -= a.N[1]; seg = 2; } }
        wp[r] = (const char*)G.W[seg] + (size_t)loc * K * sizeof(WT);
      }
    }
  };
  // request batch (l_it, l_b) into buf and move on.  Once the wave has requested all its batches
  // the loads go to the start of the (cache-resident) input row instead: still issued, never used.
  const char* idle = (const char*)(G.X + (lane * 4) % K);
  bool l_done = false;
  auto issue_next = [&](u32x4 (&buf)[NBK][WR]) {
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
      const int k = l_b * SPAN + j * BK + lane * VEC;
      const int kcl = k < K ? k : K - VEC;
#pragma unroll
      for (int r = 0; r < WR; ++r) buf[j][r] = ld_stream(l_done ? idle : wp[r] + (size_t)kcl * sizeof(WT));
    }
    if (l_b + 1 < nbps) ++l_b;
    else if (l_it + 1 < nit) { l_b = 0; ++l_it; set_rows(l_it); }
    else l_done = true;
  };
  // zero what lies past the end of the row
  auto mask_tail = [&](int c_b, u32x4 (&buf)[NBK][WR]) {
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
      const bool ok = c_b * SPAN + j * BK + lane * VEC < K;
#pragma unroll
      for (int r = 0; r < WR; ++r)
        if (!ok) buf[j][r] = (u32x4){0u, 0u, 0u, 0u};
    }
  };

  float* stat = lds;                  // mu[MAXM], rstd[MAXM]
  float* redA = lds + 16;             // [MAXM][GEMM_WAVES] partial sums
  float* redB = lds + 48;             // [MAXM][GEMM_WAVES] partial sums of squared deviations
  u32x4 b0[NBK][WR], b1[NBK][WR], b2[NBK][WR], b3[NBK][WR];
  set_rows(0);

  // Norm statistics use one fixed order per row whatever the tile shape: thread t owns the
  // elements k = 4t + 1024 j (+0..3), sums them for j = 0, 1, ... in turn, then a butterfly
  // inside each wave, then the four wave sums in index order.  LayerNorm: mean first, then
  // the squared deviations.
  auto combine4 = [&](const float* r) { return ((r[0] + r[1]) + r[2]) + r[3]; };
  constexpr int XR = GEMM_X_FLOATS / (GEMM_THREADS * 4);   // float4 registers per thread that hold the whole tile
  if (single) {
    // The whole reduction length fits the tile.  Memory returns a wave's loads in order, so the
    // input rows (and gains) are requested first, the weight batches right behind them, and
    // everything up to the staged tile then only waits for the rows.
    const int spr = KC >> 10;              // float4 slots per row per thread
    float4 xr[XR];
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      xr[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      const int m = i / spr, kk = (i - m * spr) * 1024 + tid * 4;
      if (m < M && kk < K) xr[i] = *(const float4*)(G.X + (size_t)(r0 + m) * a.ldx + kk);
    }
    // One row, GF: its gains come with it (later they would wait behind the weights).  GR float4 slots of a thread, 4096 elements,
    // are what the registers take: with 8 of them a workgroup fewer fits a compute unit; the rest of a longer row's gains is
    // read behind the weights.
    constexpr int GR = MT == 1 && GF ? 4 : 0;
    float gr[GR + 1][4], br[GR + 1][4];
    if (MT == 1 && a.norm >= 0) {
#pragma unroll
      for (int i = 0; i < GR; ++i) {
        const int kk = i * 1024 + tid * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          gr[i][e] = kk < K ? WTr<WT>::load1(G.ng, kk + e) : 0.f;
          br[i][e] = kk < K && G.nb ? WTr<WT>::load1(G.nb, kk + e) : 0.f;
        }
      }
    }
    issue_next(b0);
    issue_next(b1);
    issue_next(b2);
    if (a.norm >= 0) {
      if (a.norm == 0) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          float sm = 0.f;
#pragma unroll
          for (int i = 0; i < XR; ++i)
            if (i / spr == m) { sm += xr[i].x; sm += xr[i].y; sm += xr[i].z; sm += xr[i].w; }
          sm = wave_sum(sm);
          if (lane == 0) redA[m * GEMM_WAVES + wave] = sm;
        }
        __syncthreads();
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const float mu = a.norm == 0 ? combine4(redA + m * GEMM_WAVES) / (float)K : 0.f;
        float s2 = 0.f;
#pragma unroll
        for (int i = 0; i < XR; ++i)
          if (i / spr == m && (i - m * spr) * 1024 + tid * 4 < K) {
            float d0 = xr[i].x - mu, d1 = xr[i].y - mu, d2 = xr[i].z - mu, d3 = xr[i].w - mu;
            s2 = fmaf(d0, d0, s2); s2 = fmaf(d1, d1, s2); s2 = fmaf(d2, d2, s2); s2 = fmaf(d3, d3, s2);
          }
        s2 = wave_sum(s2);
        if (lane == 0) redB[m * GEMM_WAVES + wave] = s2;
        if (tid == 0) stat[m] = mu;
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      const int m = i / spr, kk = (i - m * spr) * 1024 + tid * 4;
      if (m >= M) continue;
      float4 v = xr[i];
      if (a.norm >= 0 && kk < K) {
        const float mu = stat[m];
        const float rs = 1.0f / sqrtf(combine4(redB + m * GEMM_WAVES) / (float)K + a.eps);
        float xv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float t = (xv[e] - mu) * rs * (i < GR ? gr[i < GR ? i : 0][e] : WTr<WT>::load1(G.ng, kk + e));
          if (G.nb) t += i < GR ? br[i < GR ? i : 0][e] : WTr<WT>::load1(G.nb, kk + e);
          xv[e] = t;
        }
        v = make_float4(xv[0], xv[1], xv[2], xv[3]);
      }
      int slot = (VEC == 8) ? (((kk & 7) >> 2) * (KC >> 3) + (kk >> 3)) : (kk >> 2);
      xs4[m * (KC >> 2) + slot] = v;       // beyond K: zeros (the weights there are zero too)
    }
    __syncthreads();
  } else {
    // The reduction length is staged chunk by chunk.  Statistics first (same order as above).
    if (a.norm >= 0) {
      if (a.norm == 0) {
        for (int m = 0; m < M; ++m) {
          const float* x = G.X + (size_t)(r0 + m) * a.ldx;
          float sm = 0.f;
          for (int i = tid * 4; i < K; i += 1024) {
            float4 v = *(const float4*)(x + i);
            sm += v.x; sm += v.y; sm += v.z; sm += v.w;
          }
          sm = wave_sum(sm);
          if (lane == 0) redA[m * GEMM_WAVES + wave] = sm;
        }
        __syncthreads();
      }
      for (int m = 0; m < M; ++m) {
        const float* x = G.X + (size_t)(r0 + m) * a.ldx;
        const float mu = a.norm == 0 ? combine4(redA + m * GEMM_WAVES) / (float)K : 0.f;
        float s2 = 0.f;
        for (int i = tid * 4; i < K; i += 1024) {
          float4 v = *(const float4*)(x + i);
          float d0 = v.x - mu, d1 = v.y - mu, d2 = v.z - mu, d3 = v.w - mu;
          s2 = fmaf(d0, d0, s2); s2 = fmaf(d1, d1, s2); s2 = fmaf(d2, d2, s2); s2 = fmaf(d3, d3, s2);
        }
        s2 = wave_sum(s2);
        if (lane == 0) redB[m * GEMM_WAVES + wave] = s2;
        if (tid == 0) stat[m] = mu;
      }
      __syncthreads();
      if (tid < M) stat[MAXM + tid] = 1.0f / sqrtf(combine4(redB + tid * GEMM_WAVES) / (float)K + a.eps);
      // (the barrier in front of the first chunk's staging publishes stat[])
    }
    issue_next(b0);
    issue_next(b1);
    issue_next(b2);
  }
  // chunked mode: x rows [k0, k0 + KC) -> LDS, normalised when the launch fuses a norm
  auto stage = [&](int k0) {
    const int kc = (K - k0) < KC ? (K - k0) : KC;          // valid elements, multiple of VEC (>= 4)
    for (int idx = tid * 4; idx < M * KC; idx += GEMM_THREADS * 4) {
      int m = idx / KC, kk = idx - m * KC;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);          // zero tail: weights beyond K are zero too
      if (kk < kc) {
        v = *(const float4*)(G.X + (size_t)(r0 + m) * a.ldx + k0 + kk);
        if (a.norm >= 0) {
          float mu = stat[m], rs = stat[MAXM + m];
          float xv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float t = (xv[e] - mu) * rs * WTr<WT>::load1(G.ng, k0 + kk + e);
            if (G.nb) t += WTr<WT>::load1(G.nb, k0 + kk + e);
            xv[e] = t;
          }
          v = make_float4(xv[0], xv[1], xv[2], xv[3]);
        }
      }
      int slot = (VEC == 8) ? (((kk & 7) >> 2) * (KC >> 3) + (kk >> 3)) : (kk >> 2);
      xs4[m * (KC >> 2) + slot] = v;
    }
  };

  float acc[WR][MT];
#pragma unroll
  for (int r = 0; r < WR; ++r)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[r][m] = 0.f;
  float* hlog = lds + GEMM_LDS_HDR + (size_t)MT * KC;   // [HEAD_MAX_ROWS] logits of this workgroup (topk launches)
  float pb[WR], prs[LR][MT];                            // bias and residual of the current set

  // arithmetic of batch q (held in cur)
  auto step = [&](int q, u32x4 (&cur)[NBK][WR]) {
    const int c_it = q / nbps, c_b = q - c_it * nbps;
    if (!single && (c_b % bpc) == 0) {
      __syncthreads();
      stage(c_b * SPAN);
      __syncthreads();
    }
    if (c_b == nbps - 1) mask_tail(c_b, cur);
    if (c_b == 0) {
      // bias and residual of this set's outputs: requested now, needed after the set's last batch
      const int s0 = gw + c_it * nwaves;
#pragma unroll
      for (int r = 0; r < LR; ++r) {
        int n = s0 * LR + r;
        if (n >= a.ntot) n = a.ntot - 1;
        if (PAIRED) {
          pb[2 * r] = G.B[0] ? WTr<WT>::load1(G.B[0], n) : 0.f;
          pb[2 * r + 1] = G.B[1] ? WTr<WT>::load1(G.B[1], n) : 0.f;
        } else {
          int seg = 0, loc = n;
          if (loc >= a.N[0]) { loc -= a.N[0]; seg = 1; if (loc >= a.N[1]) { loc -= a.N[1]; seg = 2; } }
          pb[r] = G.B[seg] ? WTr<WT>::load1(G.B[seg], loc) : 0.f;
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) prs[r][m] = (G.Rsd && m < M) ? G.Rsd[(size_t)(r0 + m) * a.ldy + n] : 0.f;
      }
    }
    const int k0 = single ? 0 : (c_b / bpc) * KC;
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
      const int kl = c_b * SPAN + j * BK + lane * VEC - k0;    // < KC
      float xf[MT][VEC];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (m < M) {
          float4 lo = xs4[m * (KC >> 2) + (VEC == 8 ? (kl >> 3) : (kl >> 2))];
          xf[m][0] = lo.x; xf[m][1] = lo.y; xf[m][2] = lo.z; xf[m][3] = lo.w;
          if constexpr (VEC == 8) {
            float4 hi = xs4[m * (KC >> 2) + (KC >> 3) + (kl >> 3)];
            xf[m][4] = hi.x; xf[m][5] = hi.y; xf[m][6] = hi.z; xf[m][7] = hi.w;
          }
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) xf[m][e] = 0.f;
        }
      }
#pragma unroll
      for (int r = 0; r < WR; ++r) {
        float wf[VEC];
        WTr<WT>::unpack(cur[j][r], wf);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[r][m] = fmaf(xf[m][e], wf[e], acc[r][m]);
      }
    }
    if (c_b == nbps - 1) {
      // the set is complete: cross-lane reduction and epilogue
#pragma unroll
      for (int r = 0; r < WR; ++r)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[r][m] = wave_sum(acc[r][m]);
      const int s = gw + c_it * nwaves;
      if (lane == 0 && c_it < nmine) {
#pragma unroll
        for (int r = 0; r < LR; ++r) {
          int n = s * LR + r;
          if (n >= a.ntot) continue;
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            if (m >= M) continue;
            float y;
            if (PAIRED) {
              y = silu(acc[2 * r][m] + pb[2 * r]) * (acc[2 * r + 1][m] + pb[2 * r + 1]);
            } else {
              y = acc[r][m] + pb[r];
              if (a.act == 1) y = gelu_erf(y);
              else if (a.act == 2) y = fmaxf(y, 0.f);
            }
            y += prs[r][m];
            G.Y[(size_t)(r0 + m) * a.ldy + n] = y;
            if (a.topk > 0 && m == 0) hlog[(c_it * GEMM_WAVES + wave) * LR + r] = y;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < WR; ++r)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[r][m] = 0.f;
    }
  };
  // one request and one batch of arithmetic per step, buffers rotating
  int q = 0;
  for (; q + 4 <= Q; q += 4) {
    issue_next(b3); step(q, b0);
    issue_next(b0); step(q + 1, b1);
    issue_next(b1); step(q + 2, b2);
    issue_next(b2); step(q + 3, b3);
  }
  if (q < Q) { issue_next(b3); step(q, b0); }
  if (q + 1 < Q) { issue_next(b0); step(q + 1, b1); }
  if (q + 2 < Q) { issue_next(b1); step(q + 2, b2); }

  // ---- LM head: this workgroup's top-k by (logit descending, id ascending)
  if (a.topk > 0) {
    __syncthreads();
    if (wave == 0) {
      // entry e = (it*4 + w)*LR + r  <->  vocabulary id ((blockIdx.x*4 + w) + it*nwaves)*LR + r
      constexpr int EPL = HEAD_MAX_ROWS / WAVE;
      float ev[EPL]; int ei[EPL];
      const int nent = nit * GEMM_WAVES * LR;
#pragma unroll
      for (int u = 0; u < EPL; ++u) {
        int e = lane + u * WAVE;
        ev[u] = -INFINITY; ei[u] = 0x7fffffff;
        if (e < nent) {
          int r = e % LR, t = e / LR, w = t % GEMM_WAVES, it = t / GEMM_WAVES;
          int id = ((blockIdx.x * GEMM_WAVES + w) + it * nwaves) * LR + r;
          if (id < a.ntot) { ev[u] = hlog[e]; ei[u] = id; }
        }
      }
      for (int r = 0; r < a.topk; ++r) {
        float v = -INFINITY; int i = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < EPL; ++u) if (better(ev[u], ei[u], v, i)) { v = ev[u]; i = ei[u]; }
        wave_best(v, i);
#pragma unroll
        for (int u = 0; u < EPL; ++u) if (ei[u] == i) { ev[u] = -INFINITY; ei[u] = 0x7fffffff; }
        if (lane == 0) { a.pk_val[blockIdx.x * MAXM + r] = v; a.pk_idx[blockIdx.x * MAXM + r] = i; }
      }
    }
  }
}

// MA rows in group 0, MB rows in group 1 (MB == 0: single-group launch; of 8 rows, blockIdx.z counts eights of rows of a prompt chunk)
template <typename WT, int MA, int MB, bool PAIRED, int WR, bool GF = true>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_kernel(GemmArgs a) {
  extern __shared__ float4 lds4[];
  float* lds = (float*)lds4;
  if (MB == 0 || blockIdx.y == 0) gemm_body<WT, MA, PAIRED, WR, GF>(a, a.g[0], lds, MA == MAXM ? (int)blockIdx.z * MAXM : 0);
  else gemm_body<WT, (MB < 1 ? 1 : MB), PAIRED, WR, GF>(a, a.g[1], lds);
}

// Reduction lengths of at most 1024, fp32 weights: a launch is a chain of latencies, not a stream.  Every operand of an output
// (rows, gains, weight row, bias, residual) is requested at once; one row is normalised by every wave for itself, so that
// nothing waits at a barrier or goes through LDS; a wave owns LR outputs (4 in head launches, whose lists are per workgroup).
// The additions are gemm_body's, in its order: block j of 256 elements is wave j's share of a row's statistics there,
// and lane l's products 4 l .. 4 l + 3 of blocks 0, 1, ... are its products here.
// Several rows behind a norm are normalised by one wave of the workgroup each and shared through LDS (every wave for itself: a PPD
// round of 12 layers, k = 3 / 8, us, before / now: 256 wide 179 / 170 and 219 / 198, 512 248 / 236 and 363 / 325, 1024 454 / 425 and 674 / 550).
// A prompt chunk of more than 8 rows is so many workgroups more, 8 rows each: the weights of such models come from L2, and 32 rows take as long as 8.
// Measured (K = 256, one row / one and three rows): norm-fused projections of 768 / 1024
// outputs 11.1 / 11.9 -> 3.8 / 4.3 us with one and three rows, 7.5 -> 2.5 us with one; 1024 logits 8.7 -> 4.0 us.
constexpr int GEMM_SMALL_K = 1024;
constexpr int GEMM_SMALL_ROWS = 4096;     // outputs of a launch: 1024 workgroups, all resident at once
template <int MT, int NB, bool PAIRED, int LR>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_small_kernel(GemmArgs a) {
  __shared__ float hlog[GEMM_WAVES * LR];
  const GemmGroup& G = a.g[blockIdx.y];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = MT == MAXM ? (int)blockIdx.z * MAXM : 0;      // (the next rows of a prompt chunk)
  const int M = MT == MAXM && G.M - r0 > MT ? MT : G.M - r0, K = a.K;
  constexpr int WROWS = PAIRED ? 2 * LR : LR;
  const int n0 = ((int)blockIdx.x * GEMM_WAVES + wave) * LR;
  // several rows behind a norm: a wave normalises rows wave, wave + 4 only, and has the others' from LDS
  constexpr bool SHARE = MT > 1;
  constexpr int OWN = SHARE ? MT / GEMM_WAVES : 1;
  __shared__ float4 xsh[SHARE ? MT : 1][SHARE ? NB * WAVE : 1];
  const bool share = SHARE && a.norm >= 0;
  float4 x[MT][NB], xo[OWN][NB], gn[NB], bs[NB], w[WROWS][NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int k = 256 * j + 4 * lane, kc = k < K ? k : 0;
    if (share) {
#pragma unroll
      for (int i = 0; i < OWN; ++i) { const int m = wave + i * GEMM_WAVES; xo[i][j] = *(const float4*)(G.X + (size_t)(r0 + (m < M ? m : 0)) * a.ldx + kc); }
    } else {
#pragma unroll
      for (int m = 0; m < MT; ++m) x[m][j] = m < M ? *(const float4*)(G.X + (size_t)(r0 + m) * a.ldx + kc) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (a.norm >= 0) {
      const float* g = (const float*)G.ng + kc;
      gn[j] = make_float4(g[0], g[1], g[2], g[3]);
      const float* b = (const float*)G.nb + kc;
      bs[j] = G.nb ? make_float4(b[0], b[1], b[2], b[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  float pb[WROWS], prs[LR][MT];
#pragma unroll
  for (int r = 0; r < LR; ++r) {
    const int n = n0 + r < a.ntot ? n0 + r : a.ntot - 1;
    int seg = 0, loc = n;
    if (!PAIRED && loc >= a.N[0]) { loc -= a.N[0]; seg = 1; if (loc >= a.N[1]) { loc -= a.N[1]; seg = 2; } }
#pragma unroll
    for (int p = 0; p < WROWS / LR; ++p) {
      const int s = PAIRED ? p : seg, i = PAIRED ? 2 * r + p : r;
      const float* row = (const float*)G.W[s] + (size_t)loc * K;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int k = 256 * j + 4 * lane;
        w[i][j] = *(const float4*)(row + (k < K ? k : 0));
      }
      pb[i] = G.B[s] ? ((const float*)G.B[s])[loc] : 0.f;
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) prs[r][m] = (G.Rsd && m < M) ? G.Rsd[(size_t)(r0 + m) * a.ldy + n] : 0.f;
  }
  // past the end of the row: zeros on both sides
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (256 * j + 4 * lane >= K) {
#pragma unroll
      for (int m = 0; m < MT; ++m) x[m][j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int i = 0; i < OWN; ++i) xo[i][j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int i = 0; i < WROWS; ++i) w[i][j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  auto normalise = [&](float4 (&v)[NB]) {
    auto combine4 = [&](const float (&r)[4]) { return ((r[0] + r[1]) + r[2]) + r[3]; };
    float mu = 0.f, r[4] = {0.f, 0.f, 0.f, 0.f};
    if (a.norm == 0) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        float s = 0.f;
        s += v[j].x; s += v[j].y; s += v[j].z; s += v[j].w;
        r[j] = wave_sum(s);
      }
      mu = combine4(r) / (float)K;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float s2 = 0.f;
      if (256 * j + 4 * lane < K) {
        const float d0 = v[j].x - mu, d1 = v[j].y - mu, d2 = v[j].z - mu, d3 = v[j].w - mu;
        s2 = fmaf(d0, d0, s2); s2 = fmaf(d1, d1, s2); s2 = fmaf(d2, d2, s2); s2 = fmaf(d3, d3, s2);
      }
      r[j] = wave_sum(s2);
    }
    const float rs = 1.0f / sqrtf(combine4(r) / (float)K + a.eps);
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (256 * j + 4 * lane < K) {
        float4 u = v[j];
        u.x = (u.x - mu) * rs * gn[j].x; u.y = (u.y - mu) * rs * gn[j].y; u.z = (u.z - mu) * rs * gn[j].z; u.w = (u.w - mu) * rs * gn[j].w;
        if (G.nb) { u.x += bs[j].x; u.y += bs[j].y; u.z += bs[j].z; u.w += bs[j].w; }
        v[j] = u;
      }
  };
  if constexpr (SHARE) {
    if (share) {
#pragma unroll
      for (int i = 0; i < OWN; ++i) {
        const int m = wave + i * GEMM_WAVES;
        if (m < M) {
          normalise(xo[i]);
#pragma unroll
          for (int j = 0; j < NB; ++j) xsh[m][j * WAVE + lane] = xo[i][j];
        }
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j) x[m][j] = m < M ? xsh[m][j * WAVE + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  } else if (a.norm >= 0) normalise(x[0]);
  float acc[WROWS][MT];
#pragma unroll
  for (int i = 0; i < WROWS; ++i)
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        s = fmaf(x[m][j].x, w[i][j].x, s); s = fmaf(x[m][j].y, w[i][j].y, s);
        s = fmaf(x[m][j].z, w[i][j].z, s); s = fmaf(x[m][j].w, w[i][j].w, s);
      }
      acc[i][m] = s;
    }
#pragma unroll
  for (int r = 0; r < LR; ++r)
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (m >= M) continue;
      float y;
      if (PAIRED) {
        y = silu(wave_sum(acc[2 * r][m]) + pb[2 * r]) * (wave_sum(acc[2 * r + 1][m]) + pb[2 * r + 1]);
      } else {
        y = wave_sum(acc[r][m]) + pb[r];
        if (a.act == 1) y = gelu_erf(y);
        else if (a.act == 2) y = fmaxf(y, 0.f);
      }
      y += prs[r][m];
      if (lane == 0 && n0 + r < a.ntot) {
        G.Y[(size_t)(r0 + m) * a.ldy + n0 + r] = y;
        if (LR > 1 && m == 0) hlog[wave * LR + r] = y;
      }
    }
  if (LR > 1 && a.topk > 0) {       // this workgroup's top-k by (logit descending, id ascending)
    __syncthreads();
    if (wave == 0) {
      int ei = (int)blockIdx.x * GEMM_WAVES * LR + lane;
      float ev = -INFINITY;
      if (lane < GEMM_WAVES * LR && ei < a.ntot) ev = hlog[lane];
      else ei = 0x7fffffff;
      for (int r = 0; r < a.topk; ++r) {
        float v = ev; int i = ei;
        wave_best(v, i);
        if (ei == i) { ev = -INFINITY; ei = 0x7fffffff; }
        if (lane == 0) { a.pk_val[blockIdx.x * MAXM + r] = v; a.pk_idx[blockIdx.x * MAXM + r] = i; }
      }
    }
  }
}

// ------------------------------------------------------------------ attention
// Decode attention of one token per row over the layer's cached positions
// [0, p) plus the row's own position p.  The rows of a group share p and the
// cached prefix (the sub-processes all extend x_<=t by one candidate); each
// row has its own key/value for position p, which this kernel also rotates
// (RoPE) and stores: at cache position p for the main token, in the row's
// tail slot for a candidate.
//
// Keys and values are cached in fp32, in blocks that are operands of
// v_mfma_f32_16x16x4_f32 as they lie in memory.  A block holds 16 positions of
// one head; inside it, for each group s of 16 components, 64 lanes x 4 floats:
//   keys:   lane i + 16 c, float u = K[position i]        [component 16 s + 4 c + u]
//   values: lane i + 16 c, float u = V[position 4 c + u]  [component 16 s + i]
// so a wave reads one kilobyte per load, and one such register quadruple feeds
// four MFMAs: scores = K q (rows: positions, columns: the group's token rows,
// reduction over components) and outputs = V^T p (rows: components, reduction
// over positions).  No shuffles, and up to 16 rows cost what one costs.
//
// A workgroup takes one head and one chunk of 64 positions, one block per
// wave.  Request order (a wave's loads return in order): the rows' own q, k, v
// (direct to LDS) and the rotation table first, then the block's keys, then
// its values.
constexpr int KV_BLOCK = 16;
__host__ __device__ inline size_t kv_blocks(int max_ctx) { return (size_t)((max_ctx + ATT_CHUNK - 1) / ATT_CHUNK) * (ATT_CHUNK / KV_BLOCK); }
// float index inside one head's cache
__host__ __device__ inline size_t k_index(int pos, int comp, int HD) {
  return (((size_t)(pos >> 4) * (HD / 16) + (comp >> 4)) * 64 + (pos & 15) + 16 * ((comp >> 2) & 3)) * 4 + (comp & 3);
}
__host__ __device__ inline size_t v_index(int pos, int comp, int HD) {
  return (((size_t)(pos >> 4) * (HD / 16) + (comp >> 4)) * 64 + (comp & 15) + 16 * ((pos >> 2) & 3)) * 4 + (pos & 3);
}

// one value of row m, column n of packed rows
__device__ __forceinline__ void put_packed1(uint16_t* out, size_t plane_elems, int KT, int m, int n, float y) {
  const uint32_t hp = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){y, 0.f}, bf16x2));
  const uint32_t lp = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){y - __uint_as_float(hp << 16), 0.f}, bf16x2));
  const size_t o = (((size_t)(m >> 4) * KT + (n >> 5)) * 64 + (m & 15) + 16 * ((n >> 3) & 3)) * 8 + (n & 7);
  out[o] = (uint16_t)hp;
  out[plane_elems + o] = (uint16_t)lp;
}

struct AttnGroup {
  const float* qkv;     // [M][3*d_model]: q | k | v as produced by the QKV projection
  float* Kc; float* Vc; // this layer's cache: [H][blocks][HD/16][64][4]
  float* tailK; float* tailV;   // own_cache == 0: destination of the rows' own key/value, [M][H][HD]
  float* part;          // [M][H][nchunk_max][hd+2] partial (unnormalised o, max, sum)
  int pos_off;          // the rows sit at position p = ds->pos + pos_off and attend to cached positions [0, p)
  int own_cache;        // the row's own key/value go to cache position p (one row only)
  int M;                // rows, 1..16
  int causal;           // prompt chunk (M up to 32): row m sits at position p + m and attends to [0, p + m); the keys and
                        // values of all rows are in the cache already (chunk_kv_kernel), nothing is stored here
};
// Rows of a prompt chunk per workgroup (grid z): its work is a chain of short phases, and the rows are what can be spread over the
// machine.  Measured (7B shape, 26 rows, one chunk of positions): 16 rows per workgroup 11.6 us, 4 rows 5.9 us.
constexpr int ATT_CAUSAL_ROWS = 4;
struct AttnArgs {
  AttnGroup g[2];
  const DevState* ds;
  const float2* rope;   // [max_ctx][hd/2] (cos, sin) or null
  int H, d_model, max_ctx, nchunk_max;
  float scale;
  uint16_t* outp;       // prompt chunk whose positions all lie in the first chunk: the finished rows in packed form (see PackArgs),
                        // in place of partials (there is nothing to merge)
};

template <int HD> __host__ __device__ constexpr int attn_lds_floats(int M) {
  // raw q|k|v and, later, the wave partials in the same place (the raw rows are done with after the rotation),
  // then q (scaled), own k, own v, scores, statistics (max, sum, own weight, -)
  return M * (ATT_WAVES * HD + 3 * HD + ATT_CHUNK + 4);
}

template <int HD, bool CAUSAL = false>
__global__ __launch_bounds__(ATT_THREADS) void attn_kernel(AttnArgs a) {
  extern __shared__ float4 lds4[];
  float* lds = (float*)lds4;
  const AttnGroup& G = a.g[CAUSAL ? 0 : blockIdx.z];
  const int r0 = CAUSAL ? (int)blockIdx.z * ATT_CAUSAL_ROWS : 0;
  constexpr int NS = HD / 16, half = HD / 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.y, c = blockIdx.x;
  const int p = a.ds->pos + G.pos_off + r0, M = CAUSAL && G.M - r0 > ATT_CAUSAL_ROWS ? ATT_CAUSAL_ROWS : G.M - r0;
  const int j0 = c * ATT_CHUNK;
  if (j0 > p + (CAUSAL ? M - 1 : 0)) return;
  // position of row m; whether this chunk holds it; whether the chunk lies before or at it at all
  auto pos_of = [&](int m) { return CAUSAL ? p + m : p; };
  auto owns = [&](int m) { const int pm = pos_of(m); return pm >= j0 && pm < j0 + ATT_CHUNK; };
  auto live = [&](int m) { return !CAUSAL || j0 <= pos_of(m); };
  static_assert(ATT_WAVES >= 3, "the wave partials reuse the raw rows' place");
  float* raw = lds;                   // [M][3][HD]
  float* ored = lds;                  // [ATT_WAVES][M][HD], written only after the barriers that follow the rotation
  float* qs = lds + M * ATT_WAVES * HD;   // [M][HD]
  float* ko = qs + M * HD;            // [M][HD]
  float* vo = ko + M * HD;            // [M][HD]
  float* sc = vo + M * HD;            // [M][ATT_CHUNK]
  float* st = sc + M * ATT_CHUNK;     // [M][4]

  // own q, k, v of every row, as they are: kilobyte pieces of the [M][3][HD] image
  {
    const int nfl = M * 3 * HD;
    for (int f0 = wave * 256; f0 < nfl; f0 += ATT_WAVES * 256) {
      const int f = f0 + lane * 4;
      if (f < nfl) {
        const int m = f / (3 * HD), r = f - m * (3 * HD), sec = r / HD, i = r - sec * HD;
        dma16(G.qkv + (size_t)(r0 + m) * 3 * a.d_model + (size_t)sec * a.d_model + (size_t)h * HD + i, raw + f0);
      }
    }
  }
  // rotation pair of this thread's component (the same for every row)
  const int ci = tid % HD;
  float2 cz = make_float2(1.f, 0.f);
  if (a.rope) cz = a.rope[(size_t)p * half + (ci < half ? ci : ci - half)];
  // this wave's block: keys, then values
  const size_t hb = (size_t)h * kv_blocks(a.max_ctx) + (size_t)(c * (ATT_CHUNK / KV_BLOCK) + wave);
  const char* kb = (const char*)G.Kc + hb * (NS * 1024) + lane * 16;
  const char* vb = (const char*)G.Vc + hb * (NS * 1024) + lane * 16;
  f32x4_t kreg[NS], vreg[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) kreg[s] = __builtin_nontemporal_load((const f32x4_t*)(kb + s * 1024));
#pragma unroll
  for (int s = 0; s < NS; ++s) vreg[s] = __builtin_nontemporal_load((const f32x4_t*)(vb + s * 1024));

  // the rows' own loads have arrived once only the 2 NS block loads are outstanding
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NS) : "memory");
  // rotate, scale, store the rows' own key and value
  for (int idx = tid; idx < M * HD; idx += ATT_THREADS) {
    const int m = idx / HD, i = idx - m * HD;     // i == ci: ATT_THREADS is a multiple of HD
    const float* r = raw + m * 3 * HD;
    float q = r[i], k = r[HD + i];
    const float v = r[2 * HD + i];
    if (CAUSAL && a.rope) cz = a.rope[(size_t)pos_of(m) * half + (i < half ? i : i - half)];
    if (a.rope) {
      const int ip = i < half ? i + half : i - half;
      const float qo = r[ip], kk = r[HD + ip];
      if (i < half) { q = fmaf(q, cz.x, -(qo * cz.y)); k = fmaf(k, cz.x, -(kk * cz.y)); }
      else          { q = fmaf(q, cz.x, qo * cz.y);    k = fmaf(k, cz.x, kk * cz.y); }
    }
    qs[m * HD + i] = q * a.scale;
    ko[m * HD + i] = k;
    vo[m * HD + i] = v;
  }
  __syncthreads();

  // scores of the block's 16 positions: lane l = n + 16 c feeds column n (row n of the group; lanes
  // past M repeat row 0, their columns are never read) and components 16 s + 4 c + u
  const int bn = lane & 15, bc = lane >> 4;
  const int bm = bn < M ? bn : 0;
  {
    f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const f32x4_t q4 = *(const f32x4_t*)(qs + bm * HD + 16 * s + 4 * bc);
#pragma unroll
      for (int u = 0; u < 4; ++u) sacc = __builtin_amdgcn_mfma_f32_16x16x4f32(kreg[s][u], q4[u], sacc, 0, 0, 0);
    }
    // sacc[jj]: position 16 wave + 4 bc + jj of the chunk, row bn.  Cached positions keep their score,
    // later ones get -inf, the rows' own position is filled in below.
    if (bn < M) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int jl = 16 * wave + 4 * bc + jj, j = j0 + jl, pm = pos_of(bn);
        if (j != pm) sc[bn * ATT_CHUNK + jl] = j < pm ? sacc[jj] : -INFINITY;
      }
    }
  }
  {
    for (int m = wave; m < M; m += ATT_WAVES) {
      if (!owns(m)) continue;
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < HD / WAVE; ++e) s = fmaf(qs[m * HD + lane + e * WAVE], ko[m * HD + lane + e * WAVE], s);
      s = wave_sum(s);
      if (lane == 0) sc[m * ATT_CHUNK + (pos_of(m) - j0)] = s;
    }
  }
  __syncthreads();
  // chunk-local softmax numerators: one wave per row, one position per lane
  for (int m = wave; m < M; m += ATT_WAVES) {
    if (!live(m)) continue;      // (the chunk lies past this row: its scores are not used and nothing is written for it)
    const float v = sc[m * ATT_CHUNK + lane];
    const float mx = wave_max(v);
    const float e = expf(v - mx);
    const float sum = wave_sum(e);
    const bool own = owns(m) && lane == pos_of(m) - j0;
    sc[m * ATT_CHUNK + lane] = own ? 0.f : e;       // the own position is added outside the MFMAs
    if (own) st[m * 4 + 2] = e;
    if (lane == 0) { st[m * 4] = mx; st[m * 4 + 1] = sum; }
  }
  __syncthreads();
  // weighted values of the block: rows = components 16 s + i, reduction over its 16 positions 4 c + u
  {
    const f32x4_t p4 = *(const f32x4_t*)(sc + bm * ATT_CHUNK + 16 * wave + 4 * bc);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      f32x4_t oacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 4; ++u) oacc = __builtin_amdgcn_mfma_f32_16x16x4f32(vreg[s][u], p4[u], oacc, 0, 0, 0);
      // oacc[jj]: component 16 s + 4 bc + jj, row bn
      if (bn < M) *(f32x4_t*)(ored + (wave * M + bn) * HD + 16 * s + 4 * bc) = oacc;
    }
  }
  __syncthreads();
  // the four blocks in wave order, then the rows' own position
  for (int idx = tid; idx < M * HD; idx += ATT_THREADS) {
    const int m = idx / HD, i = idx - m * HD;
    if (!live(m)) continue;
    const bool owns_p = owns(m);
    float o = ored[(0 * M + m) * HD + i];
#pragma unroll
    for (int w = 1; w < ATT_WAVES; ++w) o += ored[(w * M + m) * HD + i];
    if (owns_p) o = fmaf(st[m * 4 + 2], vo[m * HD + i], o);
    if (CAUSAL && a.outp) {       // (as attn_merge_kernel on one chunk: weight 1, added to 0)
      put_packed1(a.outp, (size_t)a.d_model * 32, a.d_model / 32, r0 + m, h * HD + i, (o + 0.f) / st[m * 4 + 1]);
      continue;
    }
    float* dst = G.part + (((size_t)(r0 + m) * a.H + h) * a.nchunk_max + c) * (HD + 2);
    dst[i] = o;
    if (i == 0) { dst[HD] = st[m * 4]; dst[HD + 1] = st[m * 4 + 1]; }
    // the row's own key and value (stored last: no store waits in the request queue behind the block loads)
    if (owns_p && !CAUSAL) {
      if (G.own_cache) {
        const size_t base = (size_t)h * kv_blocks(a.max_ctx) * (KV_BLOCK * HD);
        G.Kc[base + k_index(p, i, HD)] = ko[m * HD + i];
        G.Vc[base + v_index(p, i, HD)] = vo[m * HD + i];
      } else {
        const size_t d = ((size_t)m * a.H + h) * HD + i;
        G.tailK[d] = ko[m * HD + i];
        G.tailV[d] = vo[m * HD + i];
      }
    }
  }
}

// Short sequences (at most ATT_WHOLE chunks of positions): a head of a group is one workgroup's, four waves for every chunk, and the
// chunks are merged where they are, so that the launch of attn_merge_kernel goes.  The arithmetic of a chunk, and of the merge
// of one chunk per slice, is those kernels'.  Bound by its chain of latencies (the rows, the cached blocks, four barriers).
// Measured (a PPD round of a 12-layer model, us, both kernels / this one): fp32 256 wide, k = 3, position 20 196 / 171, 105 214 / 197; OPT-like 768 347 / 329, 362 / 353; LLaMA-like 1024 327 / 311,
// 389 / 380; 4096 1354 / 1341, 1270 / 1256.  With four chunks to a workgroup the larger one loses what the launch costs: OPT-like
// 768 at 100 362 / 353, at 200 364 / 365; LLaMA-like 1024 at 200 324 / 340 (and 343 where its idle waves loaded, too).
constexpr int ATT_WHOLE = 2;
constexpr int ATT_WHOLE_THREADS = ATT_WHOLE * ATT_THREADS;
template <int HD> __host__ __device__ constexpr int attn_whole_lds_floats(int M) {
  return M * (ATT_WHOLE * ATT_WAVES * HD + 3 * HD + ATT_WHOLE * ATT_CHUNK + 2 * ATT_WHOLE + 1);
}
struct AttnWholeArgs { AttnArgs a; float* out[2]; };      // out: [M][d_model] of either group
template <int HD>
__global__ __launch_bounds__(ATT_WHOLE_THREADS) void attn_whole_kernel(AttnWholeArgs w) {
  extern __shared__ float4 lds4[];
  float* lds = (float*)lds4;
  const AttnArgs& a = w.a;
  const AttnGroup& G = a.g[blockIdx.y];
  constexpr int NS = HD / 16, half = HD / 2, WAVES = ATT_WHOLE * ATT_WAVES, POS = ATT_WHOLE * ATT_CHUNK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x, p = a.ds->pos + G.pos_off, M = G.M, nc = p / ATT_CHUNK + 1;
  if (nc > ATT_WHOLE) return;         // (its launcher refuses such a position, and run_round_once a graph captured for fewer chunks)
  float* raw = lds;                   // [M][3][HD]
  float* ored = lds;                  // [WAVES][M][HD], written only after the barriers that follow the rotation
  float* qs = lds + M * WAVES * HD;   // [M][HD]
  float* ko = qs + M * HD;            // [M][HD]
  float* vo = ko + M * HD;            // [M][HD]
  float* sc = vo + M * HD;            // [M][POS]
  float* st = sc + M * POS;           // [M][ATT_WHOLE][2]: largest score, sum of a chunk
  float* so = st + M * 2 * ATT_WHOLE; // [M] weight of the own position
  {
    const int nfl = M * 3 * HD;
    for (int f0 = wave * 256; f0 < nfl; f0 += WAVES * 256) {
      const int f = f0 + lane * 4;
      if (f < nfl) {
        const int m = f / (3 * HD), r = f - m * (3 * HD), sec = r / HD, i = r - sec * HD;
        dma16(G.qkv + (size_t)m * 3 * a.d_model + (size_t)sec * a.d_model + (size_t)h * HD + i, raw + f0);
      }
    }
  }
  const int ci = tid % HD;
  float2 cz = make_float2(1.f, 0.f);
  if (a.rope) cz = a.rope[(size_t)p * half + (ci < half ? ci : ci - half)];
  // this wave's block, keys, then values; nothing for a chunk past the position
  const bool mine = wave / ATT_WAVES < nc;
  const size_t hb = (size_t)h * kv_blocks(a.max_ctx) + (size_t)wave;
  const char* kb = (const char*)G.Kc + hb * (NS * 1024) + lane * 16;
  const char* vb = (const char*)G.Vc + hb * (NS * 1024) + lane * 16;
  f32x4_t kreg[NS], vreg[NS];
  if (mine) {
#pragma unroll
    for (int s = 0; s < NS; ++s) kreg[s] = __builtin_nontemporal_load((const f32x4_t*)(kb + s * 1024));
#pragma unroll
    for (int s = 0; s < NS; ++s) vreg[s] = __builtin_nontemporal_load((const f32x4_t*)(vb + s * 1024));
    // the rows' own loads have arrived once only the 2 NS block loads are outstanding
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NS) : "memory");
  } else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  asm volatile("s_barrier" ::: "memory");
  for (int idx = tid; idx < M * HD; idx += ATT_WHOLE_THREADS) {
    const int m = idx / HD, i = idx - m * HD;     // i == ci: ATT_WHOLE_THREADS is a multiple of HD
    const float* r = raw + m * 3 * HD;
    float q = r[i], k = r[HD + i];
    const float v = r[2 * HD + i];
    if (a.rope) {
      const int ip = i < half ? i + half : i - half;
      const float qo = r[ip], kk = r[HD + ip];
      if (i < half) { q = fmaf(q, cz.x, -(qo * cz.y)); k = fmaf(k, cz.x, -(kk * cz.y)); }
      else          { q = fmaf(q, cz.x, qo * cz.y);    k = fmaf(k, cz.x, kk * cz.y); }
    }
    qs[m * HD + i] = q * a.scale;
    ko[m * HD + i] = k;
    vo[m * HD + i] = v;
  }
  __syncthreads();
  // scores of the wave's 16 positions (see attn_kernel)
  const int bn = lane & 15, bc = lane >> 4;
  const int bm = bn < M ? bn : 0;
  if (mine) {
    f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const f32x4_t q4 = *(const f32x4_t*)(qs + bm * HD + 16 * s + 4 * bc);
#pragma unroll
      for (int u = 0; u < 4; ++u) sacc = __builtin_amdgcn_mfma_f32_16x16x4f32(kreg[s][u], q4[u], sacc, 0, 0, 0);
    }
    if (bn < M) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int j = 16 * wave + 4 * bc + jj;
        if (j != p) sc[bn * POS + j] = j < p ? sacc[jj] : -INFINITY;
      }
    }
  }
  for (int m = wave; m < M; m += WAVES) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < HD / WAVE; ++e) s = fmaf(qs[m * HD + lane + e * WAVE], ko[m * HD + lane + e * WAVE], s);
    s = wave_sum(s);
    if (lane == 0) sc[m * POS + p] = s;
  }
  __syncthreads();
  // softmax numerators of a chunk: one wave per row and chunk, one position per lane
  for (int u = wave; u < M * nc; u += WAVES) {
    const int m = u / nc, c = u - m * nc, j = c * ATT_CHUNK + lane;
    const float v = sc[m * POS + j];
    const float mx = wave_max(v);
    const float e = expf(v - mx);
    const float sum = wave_sum(e);
    sc[m * POS + j] = j == p ? 0.f : e;             // the own position is added outside the MFMAs
    if (j == p) so[m] = e;
    if (lane == 0) { st[(m * ATT_WHOLE + c) * 2] = mx; st[(m * ATT_WHOLE + c) * 2 + 1] = sum; }
  }
  __syncthreads();
  // weighted values of the wave's block
  if (mine) {
    const f32x4_t p4 = *(const f32x4_t*)(sc + bm * POS + 16 * wave + 4 * bc);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      f32x4_t oacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 4; ++u) oacc = __builtin_amdgcn_mfma_f32_16x16x4f32(vreg[s][u], p4[u], oacc, 0, 0, 0);
      if (bn < M) *(f32x4_t*)(ored + (wave * M + bn) * HD + 16 * s + 4 * bc) = oacc;
    }
  }
  __syncthreads();
  // of every chunk the four blocks in wave order and the rows' own position, then the chunks in their order
  for (int idx = tid; idx < M * HD; idx += ATT_WHOLE_THREADS) {
    const int m = idx / HD, i = idx - m * HD;
    const float* const sm = st + m * ATT_WHOLE * 2;
    float gm = -INFINITY, oo = 0.f, ll = 0.f;
    for (int c = 0; c < nc; ++c) gm = fmaxf(gm, sm[2 * c]);
    for (int c = 0; c < nc; ++c) {
      const float* const oc = ored + ((size_t)c * ATT_WAVES * M + m) * HD + i;
      float o = oc[0];
#pragma unroll
      for (int v = 1; v < ATT_WAVES; ++v) o += oc[(size_t)v * M * HD];
      if (c == nc - 1) o = fmaf(so[m], vo[m * HD + i], o);
      const float wgt = expf(sm[2 * c] - gm);
      oo = fmaf(wgt, o, oo);
      ll = fmaf(wgt, sm[2 * c + 1], ll);
    }
    w.out[blockIdx.y][(size_t)m * a.d_model + (size_t)h * HD + i] = oo / ll;
    if (G.own_cache) {
      const size_t base = (size_t)h * kv_blocks(a.max_ctx) * (KV_BLOCK * HD);
      G.Kc[base + k_index(p, i, HD)] = ko[m * HD + i];
      G.Vc[base + v_index(p, i, HD)] = vo[m * HD + i];
    } else {
      const size_t d = ((size_t)m * a.H + h) * HD + i;
      G.tailK[d] = ko[m * HD + i];
      G.tailV[d] = vo[m * HD + i];
    }
  }
}

// Prompt chunk: rows m = 0..M-1 sit at consecutive positions p + m.  Their keys (rotated exactly as the
// attention kernel rotates a row's own key) and values go into the cache before the chunk's attention runs,
// so that every row finds the rows before it there.  One workgroup per (row, head), one thread per component.
struct ChunkKvArgs {
  const float* qkv;     // [M][3*d_model]
  float* Kc; float* Vc; // this layer's cache
  const float2* rope;
  const DevState* ds;
  int HD, d_model, max_ctx;
};
#ifdef PPD_ENGINE_TU
__global__ void chunk_kv_kernel(ChunkKvArgs a) {
  const int m = blockIdx.x, h = blockIdx.y, i = threadIdx.x, HD = a.HD, half = HD / 2;
  const int pos = a.ds->pos + m;
  const float* r = a.qkv + (size_t)m * 3 * a.d_model + (size_t)h * HD;
  float k = r[a.d_model + i];
  const float v = r[2 * a.d_model + i];
  if (a.rope) {
    const float2 cz = a.rope[(size_t)pos * half + (i < half ? i : i - half)];
    const float kk = r[a.d_model + (i < half ? i + half : i - half)];
    if (i < half) k = fmaf(k, cz.x, -(kk * cz.y));
    else          k = fmaf(k, cz.x, kk * cz.y);
  }
  const size_t base = (size_t)h * kv_blocks(a.max_ctx) * (KV_BLOCK * HD);
  a.Kc[base + k_index(pos, i, HD)] = k;
  a.Vc[base + v_index(pos, i, HD)] = v;
}
#endif

// A round that is run again: what its first run left at the pending position of the caches may be no number, and the MFMAs
// read whole blocks (weight 0 times NaN is NaN), so the position is cleared in the layers that the round goes through, from
// layer0 on.  (After a match the layers below hold the matching candidate's keys and values there: the round does not
// compute them again.)  One workgroup per (head, layer).
struct ClearKvArgs { float* Kc; float* Vc; const DevState* ds; int H, HD, max_ctx, layer0; };
#ifdef PPD_ENGINE_TU
__global__ void clear_kv_kernel(ClearKvArgs a) {
  const int i = threadIdx.x, pos = a.ds->pos;
  const size_t base = ((size_t)(a.layer0 + blockIdx.y) * a.H + blockIdx.x) * kv_blocks(a.max_ctx) * (KV_BLOCK * a.HD);
  a.Kc[base + k_index(pos, i, a.HD)] = 0.f;
  a.Vc[base + v_index(pos, i, a.HD)] = 0.f;
}
#endif

// merge of the chunk partials, chunks in index order
struct MergeArgs {
  const float* part[2]; float* out[2];   // out: [M][d_model]
  uint16_t* outp;      // prompt chunks of bf16 models: the rows as packed two-term operands instead (see PackArgs)
  int pos_off[2]; int M[2];
  int causal[2];       // row m sits m positions further on (prompt chunk)
  const DevState* ds;
  int H, HD, d_model, nchunk_max;
};
#ifdef PPD_ENGINE_TU
constexpr int MERGE_THREADS = 512;
// One workgroup per (row, head, group): thread t = component t % HD, slice t / HD.  Slice s merges the
// chunks s, s + S, s + 2S, ... (S = MERGE_THREADS / HD slices) in that order with a running maximum,
// 16 chunks' loads in flight together; then the slices are merged in slice order.
__global__ __launch_bounds__(MERGE_THREADS) void attn_merge_kernel(MergeArgs a) {
  __shared__ float sm_o[MERGE_THREADS], sl_m[8], sl_l[8];
  const int g = blockIdx.z, h = blockIdx.y, m = blockIdx.x;
  if (m >= a.M[g]) return;
  const int nc = (a.ds->pos + a.pos_off[g] + (a.causal[g] ? m : 0)) / ATT_CHUNK + 1;
  const int S = MERGE_THREADS / a.HD;          // 4 (head_dim 128) or 8 (64)
  const int i = threadIdx.x % a.HD, sl = threadIdx.x / a.HD;
  const float* base = a.part[g] + (((size_t)m * a.H + h) * a.nchunk_max) * (a.HD + 2);
  const size_t cs = a.HD + 2;
  constexpr int UB = 16;    // chunks whose loads are in flight together
  float mx = -INFINITY, o = 0.f, l = 0.f;
  for (int c0 = sl; c0 < nc; c0 += UB * S) {
    float tm[UB], ts[UB], to[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int c = c0 + u * S;
      const float* pc = base + (size_t)(c < nc ? c : c0) * cs;
      tm[u] = pc[a.HD]; ts[u] = pc[a.HD + 1]; to[u] = pc[i];
    }
    float bm = mx;
#pragma unroll
    for (int u = 0; u < UB; ++u) if (c0 + u * S < nc) bm = fmaxf(bm, tm[u]);
    const float rescale = expf(mx - bm);     // 0 for the first batch (mx = -inf), 1 when the maximum stays
    o *= rescale; l *= rescale; mx = bm;
#pragma unroll
    for (int u = 0; u < UB; ++u)
      if (c0 + u * S < nc) {
        const float w = expf(tm[u] - mx);
        o = fmaf(w, to[u], o);
        l = fmaf(w, ts[u], l);
      }
  }
  // slices in order; a slice without chunks has mx = -inf and weight 0
  sm_o[threadIdx.x] = o;
  if (i == 0) { sl_m[sl] = mx; sl_l[sl] = l; }
  __syncthreads();
  if (sl == 0) {
    float gm = -INFINITY;
    for (int q = 0; q < S; ++q) gm = fmaxf(gm, sl_m[q]);
    float oo = 0.f, ll = 0.f;
    for (int q = 0; q < S; ++q) {
      const float w = expf(sl_m[q] - gm);     // exp(-inf) = 0 for an empty slice
      oo = fmaf(w, sm_o[q * a.HD + i], oo);
      ll = fmaf(w, sl_l[q], ll);
    }
    const float y = oo / ll;
    if (a.outp) put_packed1(a.outp, (size_t)a.d_model * 32, a.d_model / 32, m, h * a.HD + i, y);
    else a.out[g][(size_t)m * a.d_model + (size_t)h * a.HD + i] = y;
  }
}
#endif

// ------------------------------------------------------------------ selection
// Early prediction: top-k of the early logits by (logit descending, id ascending); the head GEMM
// leaves every workgroup's own top-k, this kernel merges them and sets up the k candidate rows
// (Algorithm 2: the early top-k and its hand-out to the sub-processes -- here: their embedding rows).
// Final prediction: arg max of the final logits (ties to the lowest id), verification against the
// early candidates (Algorithm 2's comparison of each candidate with the final token), then adoption:
// on a match the matching candidate's hidden row becomes the main row and its key/value tails of layers
// 1..d-dbar become cache position t+1; without a match the tails are overwritten by the next round, and
// the main row becomes the token's embedding.  The workgroup that is done last leaves the next position.
// Appendix B's sampling-based variants replace only the arg max: the token verified here is then the one
// drawn by top-k sampling (inside this kernel, from the merged lists) or by the sampling kernel (top-p).
struct SelectArgs {
  const float* pk_val; const int32_t* pk_idx;   // [nblk][MAXM] block candidates, first kk of each valid
  int nblk; int kk;     // kk = k (early) or 1 (final)
  int k;
  int mode;             // 0: early top-k -> cand[0..k) + embed; 1: final arg max + verify + adopt
  DevState* ds;
  int32_t* host_result; // device-visible pinned host memory: [0] token, [1] match_idx (mode 1), [2..2+k) candidates (mode 0, or
                        // mode 1 where the round before predicted them), [2 + MAXM] number of finished rounds, written after the rest (mode 1): the host polls it
  EmbedArgs emb;        // candidate rows (mode 0; mode 1 with spec)
  EmbedArgs next;       // mode 1: row 0 of the next round, unless that one begins with an adopted row
  int take_next;        // mode 1: the round's candidates are those that the round before predicted (cand_next)
  // adoption (mode 1)
  float* h;                 // [1+k][d_model]: row 0 main, rows 1.. candidates
  const float* tailK; const float* tailV;   // [nb][k][H][hd]
  float* Kc; float* Vc;     // [L][H][blocks][hd/16][64][4]
  size_t head_floats;       // floats of one head's cache
  int nb, H, hd, d_model, max_ctx;
  // speculative early prediction (mode 1, exit layer d/2, early head = LM head): the head pass that made the
  // final logits of row 0 also made, for every candidate row, the early logits of the next round (the
  // candidate's state after d/2 layers is that round's exit-layer state).  On a match the matching row's
  // top-k become the next candidates here and now, and the next round starts with its parallel phase.
  int spec;
  int pk_stride;            // block lists of row m start at (m * pk_stride) * MAXM
  const float* spec_logits; // [k][vocab] logits of the candidate rows
  float* early_spec;        // [2][vocab]: the matching row's logits are kept as the early logits of the round at
                            // the next position, in the half that position's parity selects
  int vocab;
  int sampled;              // mode 1: the final prediction is ds->sampled (drawn by sample_kernel), not the arg max
  // mode 1, top-k sampling with samp_topk <= kk kept tokens: they are the head of the merged block lists, so the
  // draw happens here (fp64 inversion over the samp_topk best in ranking order, same uniform as sample_kernel)
  int samp_topk;
  uint64_t samp_seed;
};
// ------------------------------------------------------------------ sampling-based final prediction
// Appendix B: the final prediction is drawn by top-k or top-p sampling instead of the arg max; the rest of a
// round is unchanged.  One workgroup draws the token by inversion from the fp32 logits, in fp64: tokens are
// ranked by (logit descending, id ascending), w_i = exp(z_i - z_max); top-k sampling keeps the ks first of the
// ranking, top-p the shortest prefix whose mass reaches p times the total; with W the kept mass, the token is
// the first of the ranking whose cumulative mass exceeds u W.  u comes from Philox-4x32-10 (Salmon et al.,
// SC 2011) keyed by the seed, counter = sequence position of the token being chosen: decoding with and
// without PPD draws the same numbers.
// No sort: each of the two questions ("where does the kept prefix end", "where does the cumulative mass pass
// u W") asks for the largest key kappa whose mass-at-or-above G(kappa) meets a bound; kappa is fixed bit by bit
// from the top of an order-preserving 32-bit image of the logit, G always being added up in one fixed order.
// ten rounds: two 32x32->64 products, halves crossed over and mixed with counter and key; key steps by the Weyl constants
__device__ inline uint32_t philox4x32_10_word0(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1) {
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t h0 = __umulhi(0xD2511F53u, c0), l0 = 0xD2511F53u * c0;
    const uint32_t h1 = __umulhi(0xCD9E8D57u, c2), l1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
    c0 = n0; c1 = l1; c2 = n2; c3 = l0;
  }
  return c0;
}

#ifdef PPD_ENGINE_TU
constexpr int SAMP_THREADS = 1024;
constexpr int SAMP_MEMU = 8;     // loads in flight per thread when keys and weights are re-read from memory
constexpr int SAMP_NT = 64;      // thresholds at which sample_weights_kernel leaves mass and count: 1/8 apart down to 4 below the
                                 // largest logit, then 1/4 apart to 12 below
constexpr int SAMP_CAP = 6144;   // tokens between two thresholds that are searched in LDS
constexpr int SAMP_SOLO = 512;   // of those, what one wave searches alone
constexpr int SAMP_KEEP = 64;    // keys of a thread of sample_kernel that stay in its registers
struct SampleArgs {
  const float* z; int n;     // logits [n]
  int mode, ks;              // 1 top-k sampling (ks kept), 2 top-p sampling
  double p;
  uint64_t seed;
  DevState* ds;              // reads pos, writes sampled
  const float* pk_val; int nblk;   // [nblk][MAXM] block candidates of the head launch: the first of each is the block's largest logit
  double* w; uint32_t* keys; // scratch [npad] each: weights and keys, zero beyond n; npad = n rounded up to a multiple of
  int npad;                  // SAMP_THREADS * SAMP_MEMU
  double* pm; int* pc;       // scratch [npad / SAMP_THREADS][SAMP_NT + 1]: mass and count of a workgroup's tokens at or above a threshold
};

// larger logit <-> larger key; -0 and +0 are one value; no finite or infinite logit has key 0
__device__ inline uint32_t samp_key(float z) {
  const uint32_t b = __float_as_uint(z == 0.f ? 0.f : z);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float samp_unkey(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k); }

template <int CTRL> __device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double lane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double wave_sum_f64(double v) {     // same scheme as wave_sum
  v += dpp_f64<0xB1>(v);
  v += dpp_f64<0x4E>(v);
  v += dpp_f64<0x141>(v);
  v += dpp_f64<0x140>(v);
  return ((lane_f64(v, 0) + lane_f64(v, 16)) + lane_f64(v, 32)) + lane_f64(v, 48);
}


__device__ inline uint32_t samp_threshold(float zmax, int j) { return samp_key(zmax - (j <= 32 ? 0.125f * (float)j : 4.f + 0.25f * (float)(j - 32))); }

// Keys and weights of all tokens, one per thread, and how much lies at or above each threshold (in one fixed order: token by
// token, wave by wave, then workgroup by workgroup).  In the sampling kernel, one workgroup, the exponentials alone took 30 us
// at 50272 tokens and every look at them another 5.  A sum over the wave's lanes for each threshold was four thousand
// instructions of every wave: 19 us, 5 now (50272 tokens, logits of standard deviation 4).
__global__ __launch_bounds__(SAMP_THREADS) void sample_weights_kernel(SampleArgs a) {
  constexpr int NW = SAMP_THREADS / WAVE;
  __shared__ float s_red[NW];
  __shared__ double s_m[NW][SAMP_NT + 1];
  __shared__ int s_c[NW][SAMP_NT + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = blockIdx.x * SAMP_THREADS + tid;
  const bool in = i < a.n;
  const float z = in ? a.z[i] : 0.f;
  float mx = -INFINITY;
  for (int b = tid; b < a.nblk; b += SAMP_THREADS) mx = fmaxf(mx, a.pk_val[(size_t)b * MAXM]);
  mx = wave_max(mx);
  if (lane == 0) s_red[wave] = mx;
  __syncthreads();
  mx = s_red[0];
  for (int v = 1; v < NW; ++v) mx = fmaxf(mx, s_red[v]);
  const uint32_t key = in ? samp_key(z) : 0u;
  const double w = in ? exp((double)z - (double)mx) : 0.0;
  a.keys[i] = key;
  a.w[i] = w;
  // lane j has threshold j, and the wave's tokens come by in turn, those below the last threshold left out
  static_assert(SAMP_NT == WAVE, "a threshold per lane");
  const uint32_t thr = samp_threshold(mx, lane);
  double m = 0.0; int c = 0;
  const bool counts = key >= samp_threshold(mx, SAMP_NT - 1);
  for (unsigned long long todo = __ballot(counts); todo; todo &= todo - 1) {
    const int l = __builtin_ctzll(todo);
    const double wl = lane_f64(w, l);
    const bool ge = (uint32_t)__builtin_amdgcn_readlane((int)key, l) >= thr;
    m += ge ? wl : 0.0;
    c += ge ? 1 : 0;
  }
  s_m[wave][lane] = m; s_c[wave][lane] = c;
  // All tokens: what the last threshold has and, on top, what lies below it.  (Where nothing does, the two are one sum to the last
  // bit: a mass that all tokens together reach is reached at the last threshold, too, and no search goes below it for nothing.)
  m = lane_f64(m, SAMP_NT - 1) + wave_sum_f64(counts ? 0.0 : w);
  const int all = __popcll(__ballot(key != 0u));
  if (lane == 0) { s_m[wave][SAMP_NT] = m; s_c[wave][SAMP_NT] = all; }
  __syncthreads();
  if (tid <= SAMP_NT) {
    double m = 0.0; int c = 0;
    for (int v = 0; v < NW; ++v) { m += s_m[v][tid]; c += s_c[v][tid]; }
    a.pm[(size_t)blockIdx.x * (SAMP_NT + 1) + tid] = m;
    a.pc[(size_t)blockIdx.x * (SAMP_NT + 1) + tid] = c;
  }
}

// The draw.  What bounds it is one workgroup's latency: a search first finds the two thresholds its key lies between, collects
// the tokens between them in LDS (in a fixed order) and fixes the key's bits on those alone; while they are more than
// SAMP_CAP (a flat softmax, the tail below the last threshold) it looks through all tokens for a bit, until they are fewer.
// Measured (top-p 0.95), both kernels: 50272 tokens 358 us bit by bit over all tokens, 65 + 17 with the thresholds; logits of
// standard deviation 4: 76 + 19 -> 25 + 5 us, 22.5 + 5 with every thread's keys in its registers for both searches and requested behind the sums (in
// front of them: 24; as 64-bit addresses: 54, most of it spilled).  What went: workgroups' sums awaited one by one, a second look at every key where
// a thread has a token to collect (a memory latency for each of its keys, in turn), a barrier for every bit.
// In the far tail (p = 0.999, logits of standard deviation 4), 50272 / 32000 / 16000 tokens: every bit over all tokens 306 / 191 /
// 113 us, until few are left 151 / 106 / 76.
__global__ __launch_bounds__(SAMP_THREADS) void sample_kernel(SampleArgs a) {
  constexpr int NW = SAMP_THREADS / WAVE;
  __shared__ double s_m[2][NW];
  __shared__ int s_c[2][NW];
  __shared__ float s_redf[NW];
  __shared__ int s_bc[NW][16];
  __shared__ int s_cnt[16];
  __shared__ uint32_t s_prefix; __shared__ int s_need, s_min;
  __shared__ double s_gm[SAMP_NT + 1]; __shared__ int s_gc[SAMP_NT + 1];
  __shared__ double s_w[SAMP_CAP];
  __shared__ uint32_t s_key[SAMP_CAP];
  __shared__ int s_id[SAMP_CAP];
  __shared__ int s_off[NW];
  __shared__ double s_above; __shared__ uint32_t s_kappa; __shared__ int s_nabove, s_ties;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n;
  float mx = -INFINITY;
  for (int b = tid; b < a.nblk; b += SAMP_THREADS) mx = fmaxf(mx, a.pk_val[(size_t)b * MAXM]);
  // both searches look through all keys: up to SAMP_KEEP a thread are requested once (zero: no token), behind what is needed before them
  const bool keep = a.npad <= SAMP_KEEP * SAMP_THREADS;
  const __amdgpu_buffer_rsrc_t keys = __builtin_amdgcn_make_buffer_rsrc(a.keys, 0, a.npad * 4, 0x00020000);
  uint32_t kr[SAMP_KEEP];
  {
    // the workgroups' sums (through LDS, by all threads: a thread per threshold waiting for one workgroup's sums after the other took longer)
    constexpr int ROWS = SAMP_CAP / (SAMP_NT + 1), PER = (ROWS * (SAMP_NT + 1) + SAMP_THREADS - 1) / SAMP_THREADS;
    const int nb = a.npad / SAMP_THREADS;
    double m = 0.0; int c = 0;
    for (int b0 = 0; b0 < nb; b0 += ROWS) {
      const int rows = nb - b0 < ROWS ? nb - b0 : ROWS, at = b0 * (SAMP_NT + 1), ne = rows * (SAMP_NT + 1);
      double pm[PER]; int pc[PER];
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int e = tid + q * SAMP_THREADS < ne ? tid + q * SAMP_THREADS : 0;
        pm[q] = a.pm[at + e]; pc[q] = a.pc[at + e];
      }
      if (b0 == 0) {
#pragma unroll
        for (int q0 = 0; q0 < SAMP_KEEP; q0 += SAMP_MEMU)
#pragma unroll
          for (int q = q0; q < q0 + SAMP_MEMU; ++q)
            kr[q] = keep && q0 * SAMP_THREADS < a.npad ? __builtin_amdgcn_raw_buffer_load_b32(keys, tid * 4, q * SAMP_THREADS * 4, 0) : 0u;
        mx = wave_max(mx);
        if (lane == 0) s_redf[wave] = mx;
      }
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int e = tid + q * SAMP_THREADS;
        if (e < ne) { s_w[e] = pm[q]; s_id[e] = pc[q]; }
      }
      __syncthreads();
      if (tid <= SAMP_NT) {
#pragma unroll 8
        for (int b = 0; b < rows; ++b) { m += s_w[b * (SAMP_NT + 1) + tid]; c += s_id[b * (SAMP_NT + 1) + tid]; }
      }
      __syncthreads();
    }
    if (tid <= SAMP_NT) { s_gm[tid] = m; s_gc[tid] = c; }
  }
  __syncthreads();
  mx = s_redf[0];
  for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_redf[w]);
  const double zmax = (double)mx;

  // ---- mass and number of the tokens whose key is at least kth, every thread gets both: of the nl collected ones, or of all
  int par = 0, nl = 0;
  bool collected = false;          // the last search's tokens are in LDS, nl of them
  auto sum_up = [&](double m, int c, double& mass, int& count) {
    m = wave_sum_f64(m);
    if (lane == 0) { s_m[par][wave] = m; s_c[par][wave] = c; }
    __syncthreads();
    mass = 0.0; count = 0;
    for (int w = 0; w < NW; ++w) { mass += s_m[par][w]; count += s_c[par][w]; }
    par ^= 1;        // the next evaluation writes the other half: no second barrier needed
  };
  auto G_list = [&](uint32_t kth, double& mass, int& count) {
    double m = 0.0; int c = 0;
    for (int e = tid; e < (nl + WAVE - 1) / WAVE * WAVE; e += SAMP_THREADS) {
      const bool ge = e < nl && s_key[e] >= kth;
      m += ge ? s_w[e] : 0.0;
      c += __popcll(__ballot(ge));
    }
    sum_up(m, c, mass, count);
  };
  auto G_all = [&](uint32_t kth, double& mass, int& count) {
    double m = 0.0; int c = 0;
    for (int i0 = tid; i0 < a.npad; i0 += SAMP_THREADS * SAMP_MEMU) {
      uint32_t k[SAMP_MEMU]; double w[SAMP_MEMU];
#pragma unroll
      for (int q = 0; q < SAMP_MEMU; ++q) { k[q] = a.keys[i0 + q * SAMP_THREADS]; w[q] = a.w[i0 + q * SAMP_THREADS]; }
#pragma unroll
      for (int q = 0; q < SAMP_MEMU; ++q) {
        const bool ge = k[q] >= kth;
        m += ge ? w[q] : 0.0;
        c += __popcll(__ballot(ge));
      }
    }
    sum_up(m, c, mass, count);
  };
  // ---- the largest key kappa with G(kappa) >= T (kind 0), G(kappa) > T (kind 1) or count(kappa) >= K (kind 2).  Also the mass
  // and count strictly above kappa and the number of tokens at kappa.
  const double S = s_gm[SAMP_NT];
  auto search = [&](int kind, double T, int K, uint32_t& kappa, double& above, int& nabove, int& ties) {
    auto meets = [&](double g, int c) { return kind == 0 ? g >= T : (kind == 1 ? g > T : c >= K); };
    const unsigned long long at_least = __ballot(meets(s_gm[lane], s_gc[lane]));
    const int j = at_least ? __builtin_ctzll(at_least) : SAMP_NT;   // the first threshold that does (the same for every thread)
    uint32_t lo = j < SAMP_NT ? samp_threshold(mx, j) : 1u;
    const uint32_t top = j > 0 ? samp_threshold(mx, j - 1) - 1u : samp_key(mx);
    int c_at = s_gc[j], c_hi = j > 0 ? s_gc[j - 1] : 0;          // tokens at or above the prefix, above the range in question
    double g_hi = j > 0 ? s_gm[j - 1] : 0.0;                     // mass above that range
    if (c_at - c_hi > SAMP_CAP && j == SAMP_NT) {                // nothing bounds these from below yet
      uint32_t least = 0xffffffffu;
      for (int i = tid; i < n; i += SAMP_THREADS) least = min(least, a.keys[i]);
#pragma unroll
      for (int o = WAVE / 2; o >= 1; o >>= 1) least = min(least, (uint32_t)__shfl_xor((int)least, o));
      if (tid == 0) s_prefix = 0xffffffffu;
      __syncthreads();
      if (lane == 0) atomicMin(&s_prefix, least);
      __syncthreads();
      lo = s_prefix;
    }
    // bit by bit from the highest one in which lo and top differ; once a single token is left its key is kappa
    int bit = 31;
    while (bit >= 0 && !((lo ^ top) >> bit)) --bit;
    uint32_t pre = bit >= 31 ? 0u : lo >> (bit + 1) << (bit + 1);
    auto fix_bit = [&](auto&& G) {
      const uint32_t t = pre | (1u << bit--);
      if (t <= lo) { pre = t; return; }
      if (t > top) return;
      double g; int c;
      G(t, g, c);
      // (no token between the prefix and t: the bound holds at the prefix, and so here, whatever the sums' last bits say)
      if (meets(g, c) || c == c_at) { pre = t; c_at = c; }
      else { c_hi = c; g_hi = g; }
    };
    // over all tokens until few enough are left, then on those, collected in LDS
    while (bit >= 0 && c_at - c_hi > SAMP_CAP) fix_bit(G_all);
    const bool list = c_at - c_hi <= SAMP_CAP;
    collected = list;
    const double A = g_hi;
    const int cA = c_hi;
    if (list) {
      // the tokens in question, first <= key <= last, thread by thread
      const uint32_t first = pre > lo ? pre : lo, rest = pre | (bit < 0 ? 0u : (2u << bit) - 1u), last = rest < top ? rest : top;
      int mine = 0;
      static_assert(SAMP_KEEP <= 64, "a bit of the mask each");
      unsigned long long which = 0;                              // (keep: the ones to collect)
      if (keep) {
        // (few of a wave's keys are in question: four of them cost one comparison)
        const uint32_t d = last - first;
#pragma unroll
        for (int q = 0; q < SAMP_KEEP; q += 4) {
          const uint32_t r0 = kr[q] - first, r1 = kr[q + 1] - first, r2 = kr[q + 2] - first, r3 = kr[q + 3] - first;
          if (__ballot(min(min(r0, r1), min(r2, r3)) <= d))
            which |= (unsigned long long)((r0 <= d ? 1u : 0u) | (r1 <= d ? 2u : 0u) | (r2 <= d ? 4u : 0u) | (r3 <= d ? 8u : 0u)) << q;
        }
        mine = __popcll(which);
      } else
#pragma unroll 2
      for (int i0 = tid; i0 < a.npad; i0 += SAMP_THREADS * SAMP_MEMU) {
        uint32_t k[SAMP_MEMU];
#pragma unroll
        for (int q = 0; q < SAMP_MEMU; ++q) k[q] = a.keys[i0 + q * SAMP_THREADS];
#pragma unroll
        for (int q = 0; q < SAMP_MEMU; ++q) {
          const bool in = k[q] >= first && k[q] <= last;
          mine += in ? 1 : 0;
        }
      }
      int incl = mine;
#pragma unroll
      for (int o = 1; o < WAVE; o <<= 1) { const int v = __shfl_up(incl, o, WAVE); if (lane >= o) incl += v; }
      __syncthreads();                                           // (the list of an earlier search is done with)
      if (lane == WAVE - 1) s_off[wave] = incl;
      __syncthreads();
      int at = incl - mine;
      for (int w = 0; w < wave; ++w) at += s_off[w];
      nl = 0;
      for (int w = 0; w < NW; ++w) nl += s_off[w];
      if (nl > SAMP_CAP) nl = SAMP_CAP;
      auto take = [&](int i, uint32_t k) { s_key[at] = k; s_id[at] = i; s_w[at] = a.w[i]; ++at; };
      if (keep) {
        for (; which && at < SAMP_CAP; which &= which - 1) {
          const int i = tid + __builtin_ctzll(which) * SAMP_THREADS;
          take(i, a.keys[i]);
        }
      } else if (mine) {
        for (int i = tid; i < a.npad; i += SAMP_THREADS) {
          const uint32_t k = a.keys[i];
          if (k >= first && k <= last && at < SAMP_CAP) take(i, k);
        }
      }
      __syncthreads();
    }
    // few tokens: the first wave goes on alone, without a barrier, its lanes adding their own tokens (every 64th) first
    if (list && nl <= SAMP_SOLO) {
      if (wave == 0) {
        auto G = [&](uint32_t kth, double& mass, int& count) {
          double m = 0.0;
          count = 0;
          for (int e = lane; e < (nl + WAVE - 1) / WAVE * WAVE; e += WAVE) {
            const bool ge = e < nl && s_key[e] >= kth;
            m += ge ? s_w[e] : 0.0;
            count += __popcll(__ballot(ge));
          }
          mass = wave_sum_f64(m) + A; count += cA;
        };
        while (bit >= 0 && c_at - c_hi != 1) fix_bit(G);
        const bool single = c_at - c_hi == 1;
        uint32_t least = 0xffffffffu;
        for (int e = lane; e < nl; e += WAVE) if (s_key[e] >= pre) least = min(least, s_key[e]);
#pragma unroll
        for (int o = WAVE / 2; o >= 1; o >>= 1) least = min(least, (uint32_t)__shfl_xor((int)least, o));
        double ab = g_hi; int nab = c_hi, ti = 1;
        if (!single) {
          ab = 0.0; nab = 0; double g; int c;
          if (least != 0xffffffffu) G(least + 1u, ab, nab);
          G(least, g, c);
          ti = c - nab > 0 ? c - nab : 1;
        }
        if (lane == 0) { s_kappa = least; s_above = ab; s_nabove = nab; s_ties = ti; }
      }
      __syncthreads();
      kappa = s_kappa; above = s_above; nabove = s_nabove; ties = s_ties;
      return;
    }
    auto G = [&](uint32_t kth, double& mass, int& count) {
      if (list) { G_list(kth, mass, count); mass += A; count += cA; }
      else G_all(kth, mass, count);
    };
    while (bit >= 0 && c_at - c_hi != 1) fix_bit(G);
    const bool single = c_at - c_hi == 1;
    // kappa: the smallest key at or above the prefix (the prefix itself, unless bits are left open)
    __syncthreads();
    if (tid == 0) s_prefix = 0xffffffffu;
    __syncthreads();
    if (list) { for (int e = tid; e < nl; e += SAMP_THREADS) if (s_key[e] >= pre) atomicMin(&s_prefix, s_key[e]); }
    else for (int i = tid; i < a.npad; i += SAMP_THREADS) if (a.keys[i] >= pre && a.keys[i]) atomicMin(&s_prefix, a.keys[i]);
    __syncthreads();
    kappa = s_prefix;
    __syncthreads();
    above = g_hi; nabove = c_hi; ties = 1;
    if (!single) {
      above = 0.0; nabove = 0; double g; int c;
      if (kappa != 0xffffffffu) G(kappa + 1u, above, nabove);
      G(kappa, g, c);
      ties = c - nabove > 0 ? c - nabove : 1;
    }
  };
  const int pos_new = a.ds->pos + 1;
  const uint32_t word = philox4x32_10_word0((uint32_t)pos_new, 0u, 0u, 0u, (uint32_t)(a.seed & 0xffffffffu), (uint32_t)(a.seed >> 32));
  const double u = (double)(word >> 8) * (1.0 / 16777216.0);
  uint32_t kappa; double above; int nabove, ties;
  // ---- kept mass W (every thread computes the same numbers)
  double W = S;
  if (a.mode == 1) {
    const int ks = a.ks < 1 ? 1 : a.ks;
    if (ks < n) {
      search(2, 0.0, ks, kappa, above, nabove, ties);
      const double wk = exp((double)samp_unkey(kappa) - zmax);
      W = above;
      for (int r = nabove; r < ks; ++r) W += wk;
    }
  } else if (a.p < 1.0) {       // (all are kept otherwise)
    const double T = a.p * S;
    search(0, T, 0, kappa, above, nabove, ties);
    const double wk = exp((double)samp_unkey(kappa) - zmax);
    W = above;
    int r = 0;
    do { W += wk; ++r; } while (W < T && r < ties);
  }
  // ---- the first token of the ranking whose cumulative mass exceeds u W: the r-th smallest id among those at kappa
  const double t = u * W;
  search(1, t, 0, kappa, above, nabove, ties);
  int r = 0;
  {
    const double wk = exp((double)samp_unkey(kappa) - zmax);
    double c = above;
    do { c += wk; ++r; } while (!(c > t) && r < ties);
  }
  if (tid == 0) { s_min = 0x7fffffff; s_prefix = 0u; s_need = r; }
  __syncthreads();
  if (r == 1) {
    if (collected) { for (int e = tid; e < nl; e += SAMP_THREADS) if (s_key[e] == kappa) atomicMin(&s_min, s_id[e]); }
    else for (int i = tid; i < n; i += SAMP_THREADS) if (a.keys[i] == kappa) atomicMin(&s_min, i);
    __syncthreads();
    if (tid == 0) a.ds->sampled = s_min;
    return;
  }
  // several tokens share the logit and the draw falls past the first of them: the id is fixed four bits at a
  // time from the top (counts of the tied ids per digit, ascending)
  for (int shift = 28; shift >= 0; shift -= 4) {
    __syncthreads();
    const uint32_t prefix = s_prefix;
    int cn[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) cn[b] = 0;
    for (int i = tid; i < n; i += SAMP_THREADS) {
      const bool in = samp_key(a.z[i]) == kappa && (shift == 28 || ((uint32_t)i >> (shift + 4)) == prefix);
      if (in) {
        const int nib = ((uint32_t)i >> shift) & 15;
#pragma unroll
        for (int b = 0; b < 16; ++b) cn[b] += nib == b ? 1 : 0;
      }
    }
#pragma unroll
    for (int b = 0; b < 16; ++b) {
      int c = cn[b];
      for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
      if (lane == 0) s_bc[wave][b] = c;
    }
    __syncthreads();
    if (tid < 16) { int c = 0; for (int w = 0; w < NW; ++w) c += s_bc[w][tid]; s_cnt[tid] = c; }
    __syncthreads();
    if (tid == 0) {
      int need = s_need, pick = 15;
      for (int b = 0; b < 16; ++b) { if (s_cnt[b] >= need) { pick = b; break; } need -= s_cnt[b]; }
      s_need = need; s_prefix = (prefix << 4) | (uint32_t)pick;
    }
  }
  __syncthreads();
  if (tid == 0) a.ds->sampled = (int32_t)s_prefix;
}
#endif

// Threads of a merge of the heads' lists.  A thread reads its share of the entries one after the other, which 512 threads shorten;
// every wave more is one more to compare in each of the k steps that follow, which 256 shorten.  Measured, 256 / 512 threads:
// merge of 63 lists of 3 and the head before it 14.2 / 15.7 us, 250 lists of 8 26.7 / 27.9, 338 lists the same, 500 lists of 3
// 20.7 / 20.2, of 8 35.5 / 33.6; selection (it embeds or copies rows, too) over 64 lists of 3 7.4 / 8.5 us, 250 lists of 3 8.95 /
// 9.2, of 8 15.2 / 14.6, 500 lists of 3 9.75 / 9.65.
inline int merge_threads(int lists) { return lists <= 320 ? 256 : 512; }
inline int select_threads(int entries) { return entries <= 1024 ? 256 : 512; }

// Merge of the head GEMM's block lists (nblk lists, the first kk entries of each valid, MAXM apart): the best nk
// by (value descending, id ascending) land in win[] / winv[] (shared memory, MAXM entries each; wv / wi: shared
// scratch of one entry per wave).  Called by all T threads of a workgroup; ends with a barrier.
template <int T>
__device__ __forceinline__ void merge_block_lists(const float* pkv, const int32_t* pki, int nblk, int kk, int nk,
                                                  float* wv, int* wi, int* win, float* winv) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int total = nblk * kk;
  // each thread scans its strided share and keeps its own sorted best MAXM
  float lv[MAXM]; int li[MAXM];
#pragma unroll
  for (int q = 0; q < MAXM; ++q) { lv[q] = -INFINITY; li[q] = 0x7fffffff; }
  for (int e = tid; e < total; e += T) {
    int b = e / kk, r = e - b * kk;
    float v = pkv[b * MAXM + r]; int i = pki[b * MAXM + r];
    if (better(v, i, lv[MAXM - 1], li[MAXM - 1])) {
      lv[MAXM - 1] = v; li[MAXM - 1] = i;
#pragma unroll
      for (int q = MAXM - 1; q > 0; --q)
        if (better(lv[q], li[q], lv[q - 1], li[q - 1])) {
          float tv = lv[q]; lv[q] = lv[q - 1]; lv[q - 1] = tv;
          int ti = li[q]; li[q] = li[q - 1]; li[q - 1] = ti;
        }
    }
  }
  int head = 0;
  for (int r = 0; r < nk; ++r) {
    float v = -INFINITY; int i = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < MAXM; ++q) if (q == head) { v = lv[q]; i = li[q]; }
    wave_best(v, i);
    __syncthreads();
    if (lane == 0) { wv[wave] = v; wi[wave] = i; }
    __syncthreads();
    int bw = 0;
#pragma unroll
    for (int w = 1; w < T / WAVE; ++w) if (better(wv[w], wi[w], wv[bw], wi[bw])) bw = w;
    const int wid = wi[bw];
    if (tid == 0) { win[r] = wid; winv[r] = wv[bw]; }
    int cur = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < MAXM; ++q) if (q == head) cur = li[q];
    if (cur == wid) ++head;     // ids are unique: only the owner of the winner moves on
  }
  __syncthreads();
}

// Stand-alone early prediction: the merged top-k of one row's block lists written out (ids, and values when asked for).
struct TopkMergeArgs {
  const float* pk_val; const int32_t* pk_idx;   // [nblk][MAXM]
  int nblk, kk, k;
  int32_t* ids; float* vals;                    // [k]; vals may be null
};

// every workgroup merges the block candidates redundantly (they are few); winners land in win[]
template <typename WT, int T>
__global__ __launch_bounds__(T) void select_kernel(SelectArgs a) {
  __shared__ float wv[T / WAVE];
  __shared__ int wi[T / WAVE];
  __shared__ int win[MAXM];
  __shared__ float winv[MAXM];
  __shared__ int s_midx, s_tok;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // merge of one row's block lists: the best nk by (value descending, id ascending) land in win[]
  auto merge_row = [&](int prow, int nk) {
    merge_block_lists<T>(a.pk_val + (size_t)prow * a.pk_stride * MAXM, a.pk_idx + (size_t)prow * a.pk_stride * MAXM,
                      a.nblk, a.kk, nk, wv, wi, win, winv);
  };
  if (a.mode == 0 || !a.sampled) merge_row(0, a.mode == 0 ? a.k : (a.samp_topk > 0 ? a.samp_topk : 1));     // (a drawn token needs no arg max)
  if (a.mode == 0) {
    // candidates and their rows; block x handles row blockIdx.y
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid < a.k) { a.ds->cand[tid] = win[tid]; a.host_result[2 + tid] = win[tid]; }
    const int r = blockIdx.y;
    EmbedArgs e = a.emb;
    const int tok = id_in_vocab(win[r], a.vocab);
    int pos = a.ds->pos + e.pos_off;
    for (int i = blockIdx.x * T + tid; i < e.d_model; i += gridDim.x * T) {
      float v = WTr<WT>::load1(e.tok_emb, (size_t)tok * e.d_model + i);
      if (e.pos_emb) v += WTr<WT>::load1(e.pos_emb, (size_t)pos * e.d_model + i);
      e.h[(size_t)r * e.d_model + i] = v;
    }
    return;
  }
  // final: verification
  if (a.samp_topk > 0) {
    if (tid == 0) {
      const uint32_t word = philox4x32_10_word0((uint32_t)(a.ds->pos + 1), 0u, 0u, 0u, (uint32_t)(a.samp_seed & 0xffffffffu), (uint32_t)(a.samp_seed >> 32));
      const double u = (double)(word >> 8) * (1.0 / 16777216.0);
      double cum[MAXM], acc = 0.0;
      for (int r = 0; r < a.samp_topk; ++r) { acc += exp((double)winv[r] - (double)winv[0]); cum[r] = acc; }
      const double target = u * acc;
      int pick = a.samp_topk - 1;
      for (int r = a.samp_topk - 1; r >= 0; --r) if (cum[r] > target) pick = r;
      s_tok = win[pick];
    }
    __syncthreads();
  }
  const int pos = a.ds->pos;
  if (a.ds->aborted) {      // the one-launch chain of layers gave up: nothing of this round is taken over, the host runs it again
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
      a.host_result[0] = -1;
      const int32_t seq = a.ds->seq + 1;
      a.ds->seq = seq;
      __threadfence_system();
      *(volatile int32_t*)(a.host_result + 2 + MAXM) = seq;
    }
    return;
  }
  const int token = id_in_vocab(a.samp_topk > 0 ? s_tok : (a.sampled ? a.ds->sampled : win[0]), a.vocab);
  const int32_t* const cand = a.take_next ? a.ds->cand_next[pos & 1] : a.ds->cand;
  if (tid == 0) {
    int midx = -1;
    for (int q = 0; q < a.k; ++q) if (cand[q] == token) { midx = q; break; }
    s_midx = midx;
  }
  __syncthreads();
  const int midx = s_midx;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
    a.ds->result[0] = token; a.ds->result[1] = midx; a.ds->next_tok = token;
    a.host_result[0] = token; a.host_result[1] = midx;
    if (a.take_next) for (int q = 0; q < a.k; ++q) a.host_result[2 + q] = cand[q];
    // the round's record is complete: let the host see it, then the new count
    const int32_t seq = a.ds->seq + 1;
    a.ds->seq = seq;
    __threadfence_system();
    *(volatile int32_t*)(a.host_result + 2 + MAXM) = seq;
  }
  // The next round's position, once every workgroup is done with this one's
  const int nwg = gridDim.x * gridDim.y;
  auto leave = [&] {
    __syncthreads();
    if (tid == 0 && (nwg == 1 || atomicInc(&a.ds->sel_done, nwg - 1) == (unsigned)nwg - 1)) a.ds->pos = pos + 1;
  };
  const int pos_next = pos + 1;
  if (midx < 0 || a.nb == 0) {
    // the next round's row 0 is the token's embedding
    if (pos_next < a.max_ctx) {
      const EmbedArgs e = a.next;
      for (int i = ((int)blockIdx.y * (int)gridDim.x + (int)blockIdx.x) * T + tid; i < e.d_model; i += nwg * T) {
        float v = WTr<WT>::load1(e.tok_emb, (size_t)token * e.d_model + i);
        if (e.pos_emb) v += WTr<WT>::load1(e.pos_emb, (size_t)pos_next * e.d_model + i);
        e.h[i] = v;
      }
    }
    return leave();
  }
  // adoption: block (l, which), l < nb, copies one layer's K or V tail; block (0,0) also the hidden row.
  // With speculative early prediction the grid has further blocks (l >= nb) that prepare the next round.
  const int l = blockIdx.x;
  if (l >= a.nb) {
    if (!a.spec) return leave();
    const int b = l - a.nb, nblocks = gridDim.x - a.nb;
    if (blockIdx.y == 0) {
      // the matching row's logits are the next round's early logits
      const float* src = a.spec_logits + (size_t)midx * a.vocab;
      float* dst = a.early_spec + (size_t)(pos_next & 1) * a.vocab;
      for (int i = b * T + tid; i < a.vocab; i += nblocks * T) dst[i] = src[i];
      return leave();
    }
    // the next round's candidates: top-k of the matching row's logits; then, column by column (each thread
    // its own columns, so no thread waits for another): the matching row becomes row 0, and the candidates'
    // embeddings become rows 1..k, one position on
    merge_row(1 + midx, a.k);
    if (b == 0 && tid < a.k) a.ds->cand_next[pos_next & 1][tid] = win[tid];
    const EmbedArgs e = a.emb;
    const int pos2 = pos_next + 1;
    for (int i = b * T + tid; i < a.d_model; i += nblocks * T) {
      a.h[i] = a.h[(size_t)(1 + midx) * a.d_model + i];
      if (pos2 < a.max_ctx)
        for (int r = 0; r < a.k; ++r) {
          float v = WTr<WT>::load1(e.tok_emb, (size_t)id_in_vocab(win[r], a.vocab) * e.d_model + i);
          if (e.pos_emb) v += WTr<WT>::load1(e.pos_emb, (size_t)pos2 * e.d_model + i);
          e.h[(size_t)r * e.d_model + i] = v;
        }
    }
    return leave();
  }
  if (!a.spec && l == 0 && blockIdx.y == 0)
    for (int i = tid; i < a.d_model; i += T) a.h[i] = a.h[(size_t)(1 + midx) * a.d_model + i];
  // tails are [nb][k][H][hd] rows; the cache is blocked (k_index / v_index)
  const float* src = (blockIdx.y == 0 ? a.tailK : a.tailV) + ((size_t)l * a.k + midx) * a.d_model;
  float* dst = (blockIdx.y == 0 ? a.Kc : a.Vc) + (size_t)l * a.H * a.head_floats;
  for (int idx = tid; idx < a.H * a.hd; idx += T) {
    const int hh = idx / a.hd, i = idx - hh * a.hd;
    const size_t o = (size_t)hh * a.head_floats + (blockIdx.y == 0 ? k_index(pos_next, i, a.hd) : v_index(pos_next, i, a.hd));
    dst[o] = src[idx];
  }
  leave();
}

}  // namespace ppd

// ==================================================================== bf16 weights: MFMA path
// For bf16 models every linear weight is repacked once (at context creation) into blocks that are
// both one contiguous kilobyte in HBM and one A operand of v_mfma_f32_16x16x32_bf16: block (nt, kt)
// holds rows 16*nt .. 16*nt+15, columns 32*kt .. 32*kt+31; inside it lane l = i + 16*c owns the eight
// consecutive bf16 of row i, columns 8*c .. 8*c+7.  A wave-load is then a flat 1 KiB read, needs no
// unpacking, and a skinny GEMM with up to 16 rows costs the same as with one: the candidates' rows
// ride along in the B operand's other columns.
//
// The B operand carries the input rows split into two bf16 terms, x = hi + lo with hi = bf16(x) and
// lo = bf16(x - hi) (|x - hi - lo| <= 2^-17 |x|), so the products are exact in fp32 and the fp32
// activations keep 16 mantissa bits.
//
// The kernel is built around instruction count: at 8 TB/s a compute unit has about 80 cycles per
// kilobyte block, i.e. some twenty vector instructions per block and wave.  Everything that is the
// same for a whole wave lives in scalar registers (the wave index goes through readfirstlane), the
// weight stream uses buffer loads (scalar base + scalar offset + one lane offset), the input rows come
// into LDS with direct-to-LDS loads, and the main loop has no barrier: every wave streams its eighth
// of the reduction length of all the workgroup's tiles and leaves its partial sums in LDS; one
// barrier, then the epilogue adds the eight partials of every output in wave order.
namespace ppd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int MG_THREADS = 512;     // 8 waves: each takes one eighth of the reduction length of a 16-row tile
constexpr int MG_WAVES = MG_THREADS / WAVE;
constexpr int MG_BATCH = 4;         // 1 KiB blocks requested per register batch
// Register batches in flight per wave.  (Four are 1 % slower, and so is one: 7B shape, 8 layers, a PPD round behind a match 679 / 672 us, 13B 970 / 969
// and behind 4096 tokens 1152 / 1147, OPT-125m shape 295 / 292; three 682, 969, 1152, 293.)
constexpr int MG_RING = 2;
constexpr int MG_EP = 2;            // outputs per thread whose bias and residual are requested in the prologue
constexpr int MG_LDS_HLOG = 2048;   // byte offsets: [0, 2048) norm statistics, then 1 KiB of head logits,
constexpr int MG_LDS_G = 3072;      // then the norm's gain (and bias), the partial sums, the staged rows

struct RepackArgs {
  const uint16_t* src[3]; int nrows[3];   // up to three row segments, concatenated (Q | K | V); paired: src[0] gate, src[1] up
  int K, KT, NT, paired;
  uint16_t* dst;
};
#ifdef PPD_ENGINE_TU
__global__ void repack_kernel(RepackArgs a) {
  // one workgroup of 64 lanes per block
  const int blk = blockIdx.x, lane = threadIdx.x;
  const int nt = blk / a.KT, kt = blk - nt * a.KT;
  const int i = lane & 15, c = lane >> 4;
  const uint16_t* row = nullptr;
  if (a.paired) {
    int n = nt * 8 + (i & 7);
    if (n < a.nrows[0]) row = a.src[i < 8 ? 0 : 1] + (size_t)n * a.K;
  } else {
    int n = nt * 16 + i, seg = 0;
    while (seg < 3 && n >= a.nrows[seg]) { n -= a.nrows[seg]; ++seg; }
    if (seg < 3) row = a.src[seg] + (size_t)n * a.K;
  }
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    int k = kt * 32 + c * 8 + e;
    v[e] = (row && k < a.K) ? row[k] : (uint16_t)0;
  }
  uint4 o;
  o.x = v[0] | ((uint32_t)v[1] << 16); o.y = v[2] | ((uint32_t)v[3] << 16);
  o.z = v[4] | ((uint32_t)v[5] << 16); o.w = v[6] | ((uint32_t)v[7] << 16);
  *(uint4*)(a.dst + ((size_t)blk * 64 + lane) * 8) = o;
}
#endif

struct MGemmGroup {
  const float* X;     // [M][ldx] input rows (before the fused norm), rows 16-byte aligned
  const float* Rsd;   // residual rows [M][ldy] added in the epilogue, or null
  float* Y;           // [M][ldy]
  const void* P;      // repacked weights [NT][KT][64 lanes][8 bf16]
  const void* B[3];   // biases per row segment or null (paired: B[0] gate, B[1] up)
  const void* ng; const void* nb;  // gain / bias of the fused norm
  int M;              // rows, 1..16
  const float* part; int pos_off;  // nmerge > 0: the rows are these attention partials, merged (see MergeArgs)
};
struct MGemmArgs {
  MGemmGroup g[2];
  int K, KT, NT;    // reduction length (multiple of 8), its 32-column blocks, 16-row tiles
  int N[3];         // rows per segment (bias lookup)
  int ntot;         // logical output rows (paired: rows of one of the two matrices)
  int ldx, ldy;
  int norm;         // -1 none, 0 LayerNorm, 1 RMSNorm
  float eps;
  int act;          // 0 none, 1 GELU, 2 ReLU (paired launches apply SwiGLU)
  int topk; float* pk_val; int32_t* pk_idx;   // head launches: every workgroup leaves the top-k of each row's logits it made:
  int pk_stride;    // row m's list of workgroup b at ((m * pk_stride + b) * MAXM)
  int xrow;         // LDS bytes between two staged rows
  int tiles_wg;     // ceil(NT / gridDim.x); gridDim.x <= NT
  unsigned wbytes;  // NT * KT * 1024
  int passes;       // the reduction length is staged in LDS in this many passes (1: whole rows; > 1 only without a fused norm)
  int nmerge;       // gemm_mfma_narrow_kernel without a norm: chunks of positions that may be in use, up to MG_MERGE; 0: X has the rows
  int H, HD, nchunk_max; const DevState* ds;
  int halves;       // gemm_mfma_narrow_kernel, a tile per workgroup and no pairs: 1: two workgroups share a tile, eight of its rows each
};

// LDS bytes between staged rows: the row itself, moved off a multiple of 256 so that neighbouring rows
// start in different banks
__host__ __device__ inline int mg_xrow(int KT) { int r = KT * 128; return (r & 255) ? r : r + 128; }
// Staging in passes: every wave's share of the reduction length (nb8 blocks) is cut into `passes` runs of
// nbp blocks (a multiple of the batch size); pass p stages, for each of the 8 waves, run p of its share.
__host__ __device__ inline int mg_nbp(int KT, int passes) {
  const int nb8 = (KT + MG_WAVES - 1) / MG_WAVES;
  if (passes <= 1) return (nb8 + MG_BATCH - 1) / MG_BATCH * MG_BATCH;
  return ((nb8 + passes - 1) / passes + MG_BATCH - 1) / MG_BATCH * MG_BATCH;
}
__host__ __device__ inline int mg_xrow_pass(int KT, int passes) { return passes <= 1 ? mg_xrow(KT) : mg_nbp(KT, passes) * 1024 + 128; }
// LDS map behind MG_LDS_G; returns the total
__host__ __device__ inline int mg_lds_layout(int K, int M, int norm, int tiles_wg, int xrow, int& off_b, int& off_part, int& off_x) {
  const int gsz = (K * 2 + 1023) & ~1023;
  off_b = MG_LDS_G + (norm >= 0 ? gsz : 0);
  off_part = off_b + (norm == 0 ? gsz : 0);
  off_x = off_part + tiles_wg * MG_WAVES * M * 64;
  return off_x + M * xrow;
}

// MP: the instance that can stage the reduction length in several passes (a.passes > 1); the other one
// keeps the single-pass loop free of that bookkeeping.
template <bool PAIRED, bool MP = false>
__global__ __launch_bounds__(MG_THREADS) void gemm_mfma_kernel(MGemmArgs a) {
  extern __shared__ float4 lds4[];
  char* lds = (char*)lds4;
  const MGemmGroup& G = a.g[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = G.M, K = a.K, KT = a.KT;
  const int grid = gridDim.x, xrow = a.xrow;
  const int ntiles = (int)blockIdx.x + (a.tiles_wg - 1) * grid < a.NT ? a.tiles_wg : a.tiles_wg - 1;
  int off_b, off_part, off_x;
  mg_lds_layout(K, M, a.norm, a.tiles_wg, xrow, off_b, off_part, off_x);
  float* redA = (float*)lds;                  // [16][8] each
  float* redB = redA + 16 * MG_WAVES;
  float* hlog = (float*)(lds + off_x);        // head launches: [M][HEAD_MAX_ROWS] logits, over the staged rows once those are done with

  // ---- 1. input rows (and the norm's gain and bias) into LDS, fp32 as they are.  These requests come first: a wave's loads return in
  // order.  A wave brings exactly the share of every row that it multiplies (its eighth of the reduction length), and later converts that share
  // alone: without a norm no barrier stands between the two, so nothing else may be read from the rows before the main loop is done.
  // With passes (a barrier follows each), wave w takes the kilobyte pieces w, w + 8, ... of every row; a staged row is 8 runs (one per wave) of nbp blocks; float f of the row belongs to wave
  // f / (32 nbp)'s share, block (pass * nbp + (f / 32) % nbp) of it.  pass_col gives the input column, or -1.
  const int npass = MP ? a.passes : 1;
  const int nb8_ = (KT + MG_WAVES - 1) / MG_WAVES, nbp_ = mg_nbp(KT, npass);
  auto pass_col = [&](int pass, int f) -> int {
    const int seg = f / (32 * nbp_), rem = f - seg * 32 * nbp_;
    const int s = pass * nbp_ + (rem >> 5);
    const int k0 = seg * nb8_ < KT ? seg * nb8_ : KT;
    const int nb = (k0 + nb8_ < KT ? k0 + nb8_ : KT) - k0;
    const int col = (k0 + s) * 32 + (rem & 31);
    return (s < nb && col < K) ? col : -1;
  };
  auto dma_pass = [&](int pass) {
    for (int u = wave; u < nbp_; u += MG_WAVES) {
      const int col = pass_col(pass, u * 256 + lane * 4);      // (the same for every row)
      if (col >= 0)
        for (int m = 0; m < M; ++m) dma16(G.X + (size_t)m * a.ldx + col, lds + off_x + m * xrow + u * 1024);
    }
  };
  {
    if constexpr (MP) dma_pass(0);
    else {
      // (its own share of every row, and of the gains: without a norm a wave waits for no other before its first product)
      const int e0 = wave * nb8_ * 32, e1 = e0 + nb8_ * 32 < K ? e0 + nb8_ * 32 : K;
      for (int m = 0; m < M; ++m)
        for (int k0 = e0; k0 < e1; k0 += 256) {
          const int kk = k0 + lane * 4;
          if (kk < e1) dma16(G.X + (size_t)m * a.ldx + kk, lds + off_x + m * xrow + k0 * 4);
        }
      if (a.norm >= 0)
        for (int k0 = e0; k0 < e1; k0 += 512) {
          const int kk = k0 + lane * 8;
          if (kk < e1) {
            dma16((const uint16_t*)G.ng + kk, lds + MG_LDS_G + k0 * 2);
            if (a.norm == 0 && G.nb) dma16((const uint16_t*)G.nb + kk, lds + off_b + k0 * 2);
          }
        }
    }
  }

  // ---- 2. bias and residual of the outputs this thread will finish (output e = tid + 512 i:
  // row = e % R inside the tile, then the input row, then the tile ordinal)
  constexpr int R = PAIRED ? 8 : 16;
  const int nout = ntiles * M * R;
  auto out_coord = [&](int e, int& ord, int& col, int& row, int& n) {
    row = e & (R - 1);
    const int f = e / R;
    ord = f / M; col = f - ord * M;
    n = ((int)blockIdx.x + ord * grid) * R + row;
  };
  // (the bf16 bias values stay raw until the epilogue: converting them here would wait for the loads)
  const uint16_t* const B0 = (const uint16_t*)G.B[0];
  const uint16_t* const B1 = (const uint16_t*)G.B[1];
  const uint16_t* const B2 = (const uint16_t*)G.B[2];
  auto out_operands = [&](int col, int n, uint32_t& b0, uint32_t& b1, float& rsd) {
    b0 = 0u; b1 = 0u; rsd = 0.f;
    if (PAIRED) {
      if (B0) b0 = B0[n];
      if (B1) b1 = B1[n];
    } else if (B0) {      // a model has either all linear biases or none
      int seg = 0, loc = n;
      if (loc >= a.N[0]) { loc -= a.N[0]; seg = 1; if (loc >= a.N[1]) { loc -= a.N[1]; seg = 2; } }
      const uint16_t* bp = seg == 0 ? B0 : (seg == 1 ? B1 : B2);
      b0 = bp[loc];
    }
    if (G.Rsd) rsd = G.Rsd[(size_t)col * a.ldy + n];
  };
  uint32_t p_b0[MG_EP], p_b1[MG_EP]; float p_rsd[MG_EP];
#pragma unroll
  for (int i = 0; i < MG_EP; ++i) {
    p_b0[i] = 0u; p_b1[i] = 0u; p_rsd[i] = 0.f;
    const int e = tid + i * MG_THREADS;
    if (e < nout) {
      int ord, col, row, n; out_coord(e, ord, col, row, n);
      if (n < a.ntot) out_operands(col, n, p_b0[i], p_b1[i], p_rsd[i]);
    }
  }

  // ---- 3. the weight stream: wave w owns k-blocks [kb0, kb0 + nblk) of every tile blockIdx.x,
  // + gridDim.x, ...; MG_BATCH blocks per batch, MG_RING batches in flight.  Every batch is always
  // requested in full, as a buffer of its own that ends with the wave's share: nothing is read for slots past it (or past the last tile).
  const int nb8 = (KT + MG_WAVES - 1) / MG_WAVES;
  const int kb0 = wave * nb8 < KT ? wave * nb8 : KT;
  const int nblk = (kb0 + nb8 < KT ? kb0 + nb8 : KT) - kb0;
  // Passes (P > 1 when the staged rows would not fit LDS at once): pass p covers blocks [p * nbp, (p + 1) * nbp)
  // of every wave's share, for all tiles, before the next pass starts.  A wave's accumulator of a tile is
  // parked in its partial-sum slot between passes and taken up again as the MFMA's C input, so the chain of
  // additions is exactly the one of a single pass.
  const int P = npass;
  const int nbp = mg_nbp(KT, P);                             // blocks of a wave's share per pass
  const int NBT = MP ? nbp / MG_BATCH : (nb8 + MG_BATCH - 1) / MG_BATCH;   // batches per tile (and pass), the same for every wave
  const int sst = P == 1 ? nb8 : nbp;                        // blocks between two waves' staged runs
  const int Q = P * ntiles * NBT;
  const unsigned lane16 = lane * 16;
  int l_p = 0, l_tile = 0, l_b = 0;     // pass, tile ordinal and batch inside the tile of the next request
  auto issue = [&](u32x4 (&buf)[MG_BATCH]) {
    const bool live = MP ? l_p < P : l_tile < ntiles;
    const int s0 = (MP ? l_p * nbp : 0) + l_b * MG_BATCH, left = live ? nblk - s0 : 0, n = left < 0 ? 0 : (left < MG_BATCH ? left : MG_BATCH);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((char*)G.P + (unsigned)(((int)blockIdx.x + l_tile * grid) * KT + kb0 + s0) * 1024u, 0, n * 1024, 0x00020000);
#pragma unroll
    for (int j = 0; j < MG_BATCH; ++j) buf[j] = __builtin_amdgcn_raw_buffer_load_b128(r, lane16 + j * 1024u, 0, 2);   // 2: non-temporal
    if (++l_b == NBT) {
      l_b = 0; ++l_tile;
      if (MP && l_tile == ntiles) { l_tile = 0; ++l_p; }
    }
  };
  // One batch per wave is what a compute unit keeps in flight: it goes out now, the rest of the ring
  // after the rows are staged (a wave that asked for more would sit in the request queue instead of
  // working on the rows).
  u32x4 ring[MG_RING][MG_BATCH];
  issue(ring[0]);

  // ---- 4. norm statistics and the split into two bf16 terms, in place: the 32 bytes that held the
  // floats k .. k+7 (k a multiple of 8) then hold hi(k..k+7) | lo(k..k+7).  One fixed order per row:
  // thread t sums the 8-element chunks t, t + 512, ... in turn, butterfly inside each wave, the eight
  // wave sums in index order.  LayerNorm: mean first, then the squared deviations.
  // everything a wave has requested before its weights has arrived once only the MG_BATCH newest loads
  // are outstanding
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MG_BATCH) : "memory");
  auto combine8 = [&](const float* r) { return ((((((r[0] + r[1]) + r[2]) + r[3]) + r[4]) + r[5]) + r[6]) + r[7]; };
  float mu_l = 0.f, rs_l = 1.f;               // lane m: of row m
  if (MP || a.norm >= 0) asm volatile("s_barrier" ::: "memory");     // the workgroup's rows are complete in LDS
  if (!MP && a.norm >= 0) {
    if (a.norm == 0) {
      for (int m = 0; m < M; ++m) {
        float sm = 0.f;
        for (int c = tid; c * 8 < K; c += MG_THREADS) {
          const float4* px = (const float4*)(lds + off_x + m * xrow + c * 32);
          const float4 v = px[0], w = px[1];
          sm += v.x; sm += v.y; sm += v.z; sm += v.w; sm += w.x; sm += w.y; sm += w.z; sm += w.w;
        }
        sm = wave_sum(sm);
        if (lane == 0) redA[m * MG_WAVES + wave] = sm;
      }
      __syncthreads();
    }
    for (int m = 0; m < M; ++m) {
      const float mu = a.norm == 0 ? combine8(redA + m * MG_WAVES) / (float)K : 0.f;
      float s2 = 0.f;
      for (int c = tid; c * 8 < K; c += MG_THREADS) {
        const float4* px = (const float4*)(lds + off_x + m * xrow + c * 32);
        const float4 v = px[0], w = px[1];
        const float d[8] = {v.x - mu, v.y - mu, v.z - mu, v.w - mu, w.x - mu, w.y - mu, w.z - mu, w.w - mu};
#pragma unroll
        for (int e = 0; e < 8; ++e) s2 = fmaf(d[e], d[e], s2);
      }
      s2 = wave_sum(s2);
      if (lane == 0) redB[m * MG_WAVES + wave] = s2;
    }
    __syncthreads();                          // (and nobody reads another wave's share of the rows any more)
    const int m = lane < M ? lane : 0;
    mu_l = a.norm == 0 ? combine8(redA + m * MG_WAVES) / (float)K : 0.f;
    rs_l = 1.0f / sqrtf(combine8(redB + m * MG_WAVES) / (float)K + a.eps);
  }
  // hi = bf16(x) (the hardware's round-to-nearest-even pair conversion), lo = bf16(x - hi)
  auto split_to = [](char* px, const float (&xv)[8]) {
    uint32_t hp[4], lp[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      hp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){xv[2 * e], xv[2 * e + 1]}, bf16x2));
      const float r0 = xv[2 * e] - __uint_as_float(hp[e] << 16), r1 = xv[2 * e + 1] - __uint_as_float(hp[e] & 0xffff0000u);
      lp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){r0, r1}, bf16x2));
    }
    ((uint4*)px)[0] = make_uint4(hp[0], hp[1], hp[2], hp[3]);
    ((uint4*)px)[1] = make_uint4(lp[0], lp[1], lp[2], lp[3]);
  };
  // (with passes: the split for the runs of one pass; chunks outside every wave's share become zeros)
  auto convert_rows = [&](int pass) {
    // (no fused norm with passes; whether a chunk lies inside a wave's share is the same for every row)
    for (int c = tid; c < nbp_ * 32; c += MG_THREADS) {
      const bool inside = pass_col(pass, c * 8) >= 0;
      for (int m = 0; m < M; ++m) {
        char* px = lds + off_x + m * xrow + c * 32;
        float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (inside) {
          const float4 v = ((const float4*)px)[0], w = ((const float4*)px)[1];
          xv[0] = v.x; xv[1] = v.y; xv[2] = v.z; xv[3] = v.w; xv[4] = w.x; xv[5] = w.y; xv[6] = w.z; xv[7] = w.w;
        }
        split_to(px, xv);
      }
    }
  };
  if constexpr (MP) {
    convert_rows(0);
    __syncthreads();
  } else {
    // a wave's own share; its columns past the row's end become zeros
    for (int m = 0; m < M; ++m) {
      const float mu = lane_f32(mu_l, m), rs = lane_f32(rs_l, m);
      for (int c = kb0 * 4 + lane; c < (kb0 + nblk) * 4; c += WAVE) {
        char* px = lds + off_x + m * xrow + c * 32;
        float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (c * 8 < K) {
          const float4 v = ((const float4*)px)[0], w = ((const float4*)px)[1];
          xv[0] = v.x; xv[1] = v.y; xv[2] = v.z; xv[3] = v.w; xv[4] = w.x; xv[5] = w.y; xv[6] = w.z; xv[7] = w.w;
          if (a.norm >= 0) {
            const u32x4 gq = *(const u32x4*)(lds + MG_LDS_G + c * 16);
            float gf[8]; WTr<bf16_t>::unpack(gq, gf);
#pragma unroll
            for (int e = 0; e < 8; ++e) xv[e] = (xv[e] - mu) * rs * gf[e];
            if (a.norm == 0 && G.nb) {
              const u32x4 bq = *(const u32x4*)(lds + off_b + c * 16);
              float bf[8]; WTr<bf16_t>::unpack(bq, bf);
#pragma unroll
              for (int e = 0; e < 8; ++e) xv[e] += bf[e];
            }
          }
        }
        split_to(px, xv);
      }
    }
    asm volatile("" ::: "memory");            // (a wave's own LDS operations stay in order)
  }
#pragma unroll
  for (int r = 1; r < MG_RING; ++r) issue(ring[r]);

  // ---- 5. main loop.  B operand: lane l feeds column l % 16 (input row; lanes past M read row 0 and
  // their columns are never stored) and the eight k of chunk l / 16.
  const int bm = lane & 15, bc = lane >> 4;
  const char* xlane = lds + off_x + (bm < M ? bm : 0) * xrow + bc * 32 + ((!MP || P == 1) ? kb0 : wave * sst) * 128;
  float* plane = (float*)(lds + off_part) + (wave * M + bm) * 16 + bc * 4;   // + ord * 8 * M * 16
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  int c_p = 0, c_ord = 0, c_b = 0;
  auto consume = [&](u32x4 (&cur)[MG_BATCH]) {
    if constexpr (!MP) {
#pragma unroll
      for (int j = 0; j < MG_BATCH; ++j) {
        const int s = c_b * MG_BATCH + j;
        if (s < nblk) {                      // the same for the whole wave
          const u32x4* xp = (const u32x4*)(xlane + s * 128);
          const u32x4 bh = xp[0], bl = xp[1];
          const bf16x8 av = __builtin_bit_cast(bf16x8, cur[j]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh), acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bl), acc, 0, 0, 0);
        }
      }
      if (++c_b == NBT) {
        // this wave's partial sums of the tile: lane l holds rows 4 (l / 16) .. + 3 of column l % 16
        if (bm < M) *(f32x4*)(plane + c_ord * (MG_WAVES * 16) * M) = acc;
        acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        c_b = 0; ++c_ord;
      }
    } else {
      if (c_b == 0 && c_p > 0) {
        if (c_ord == 0) {
          // next pass: every wave is done with the staged runs; bring in the next ones (the weight requests
          // already made for this pass keep flying meanwhile)
          __syncthreads();
          dma_pass(c_p);
          asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
          convert_rows(c_p);
          __syncthreads();
        }
        if (bm < M) acc = *(const f32x4*)(plane + c_ord * (MG_WAVES * 16) * M);    // the chain goes on where it stopped
      }
#pragma unroll
      for (int j = 0; j < MG_BATCH; ++j) {
        const int s = c_p * nbp + c_b * MG_BATCH + j;
        if (s < nblk) {
          const u32x4* xp = (const u32x4*)(xlane + (s - c_p * nbp) * 128);
          const u32x4 bh = xp[0], bl = xp[1];
          const bf16x8 av = __builtin_bit_cast(bf16x8, cur[j]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh), acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bl), acc, 0, 0, 0);
        }
      }
      if (++c_b == NBT) {
        if (bm < M) *(f32x4*)(plane + c_ord * (MG_WAVES * 16) * M) = acc;
        acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        c_b = 0;
        if (++c_ord == ntiles) { c_ord = 0; ++c_p; }
      }
    }
  };
  for (int q = 0; q < Q; q += MG_RING) {
#pragma unroll
    for (int r = 0; r < MG_RING; ++r) {
      if (q + r < Q) consume(ring[r]);
      issue(ring[r]);
    }
  }
  __syncthreads();

  // ---- 6. epilogue: the eight partials of an output in wave order, bias, activation, residual
  auto finish = [&](int e, uint32_t rb0, uint32_t rb1, float rsd) {
    int ord, col, row, n; out_coord(e, ord, col, row, n);
    if (n >= a.ntot) return;
    const float b0 = __uint_as_float(rb0 << 16), b1 = __uint_as_float(rb1 << 16);
    const float* pp = (const float*)(lds + off_part) + (ord * MG_WAVES * M + col) * 16 + row;
    const int ws = M * 16;
    float s = pp[0];
#pragma unroll
    for (int w = 1; w < MG_WAVES; ++w) s += pp[w * ws];
    float y;
    if (PAIRED) {
      float u = pp[8];
#pragma unroll
      for (int w = 1; w < MG_WAVES; ++w) u += pp[w * ws + 8];
      y = silu(s + b0) * (u + b1);
    } else {
      y = s + b0;
      if (a.act == 1) y = gelu_erf(y);
      else if (a.act == 2) y = fmaxf(y, 0.f);
    }
    y += rsd;
    G.Y[(size_t)col * a.ldy + n] = y;
    if (a.topk > 0) hlog[col * HEAD_MAX_ROWS + ord * 16 + row] = y;
  };
#pragma unroll
  for (int i = 0; i < MG_EP; ++i) {
    const int e = tid + i * MG_THREADS;
    if (e < nout) finish(e, p_b0[i], p_b1[i], p_rsd[i]);
  }
  for (int e = tid + MG_EP * MG_THREADS; e < nout; e += MG_THREADS) {
    int ord, col, row, n; out_coord(e, ord, col, row, n);
    uint32_t b0 = 0u, b1 = 0u; float rsd = 0.f;
    if (n < a.ntot) out_operands(col, n, b0, b1, rsd);
    finish(e, b0, b1, rsd);
  }

  // ---- LM head: this workgroup's top-k of every row by (logit descending, id ascending); wave w takes rows w, w + 8, ...
  if (a.topk > 0) {
    __syncthreads();
    for (int col = wave; col < M; col += MG_WAVES) {
      constexpr int EPL = HEAD_MAX_ROWS / WAVE;
      float ev[EPL]; int ei[EPL];
#pragma unroll
      for (int u = 0; u < EPL; ++u) {
        const int e = lane + u * WAVE;       // entry e = tile ordinal * 16 + row
        ev[u] = -INFINITY; ei[u] = 0x7fffffff;
        const int id = ((int)blockIdx.x + (e >> 4) * grid) * 16 + (e & 15);
        if ((e >> 4) < ntiles && id < a.ntot) { ev[u] = hlog[col * HEAD_MAX_ROWS + e]; ei[u] = id; }
      }
      for (int r = 0; r < a.topk; ++r) {
        float v = -INFINITY; int i = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < EPL; ++u) if (better(ev[u], ei[u], v, i)) { v = ev[u]; i = ei[u]; }
        wave_best(v, i);
#pragma unroll
        for (int u = 0; u < EPL; ++u) if (ei[u] == i) { ev[u] = -INFINITY; ei[u] = 0x7fffffff; }
        if (lane == 0) {
          const size_t o = ((size_t)col * a.pk_stride + blockIdx.x) * MAXM + r;
          a.pk_val[o] = v; a.pk_idx[o] = i;
        }
      }
    }
  }
}

// Products of narrow models: a launch is a chain of latencies, not a stream.  A workgroup makes T tiles (blockIdx.x, + gridDim.x,
// ...) and requests every operand of them at once: rows, gains, all of its weights (T NB blocks in each wave's registers), biases,
// residuals.  The rows are worked on in units of 64 pieces of eight elements, a wave's part of one row in the norm's order of
// additions; a wave has every eighth unit, so that no element is normalised or split twice in a workgroup, and the
// statistics of all rows are made at the same time.  The arithmetic, and every order of additions, is gemm_mfma_kernel's.
// Measured (two groups, us a layer of the parallel phase with its attention, gemm_mfma_kernel / this one): OPT-125m shape k = 3
// 40 / 28, k = 8 49 / 30; 512 wide 34 / 18 and 46 / 21; each wave normalising its own blocks of all rows in registers, without a
// barrier, was the slower way (k = 3 34): half of what a compute unit issued then were the same normalisations again.
// NORM: -1 none, 0 LayerNorm (with a bias), 1 RMSNorm; NB: blocks of a wave's share at most.
constexpr int MG_NARROW_ROWS = 8;            // of a group
constexpr int MG_NARROW_LDS = 512;           // [2][MG_NARROW_ROWS][8] sums of the norm, then the partial sums, then the rows
__host__ __device__ inline int mg_narrow_lds(int KT, int M, int T) { return MG_NARROW_LDS + T * MG_WAVES * M * 64 + M * mg_xrow(KT); }
// MERGE: the rows are attention partials of up to MG_MERGE chunks, which every workgroup merges for itself, a piece per thread, in
// attn_merge_kernel's slices and order, and a launch goes.  (Where a workgroup had to merge the whole row one thread per component,
// before a streaming kernel's prologue, it lost: 16 against 15 us of a 4096-wide model.)  Measured (a PPD round of 12 layers, k = 3,
// us, with the merge's launch / without): OPT-like 768 wide at 140 positions 360 / 335, at 480 367 / 342; LLaMA-like 1024 375 / 344
// at 140; a plain token of the 768 wide one 310 / 283 and 321 / 289.
constexpr int MG_MERGE = 8;
template <bool PAIRED, int NORM, int T, int NB, bool MERGE = false>
__global__ __launch_bounds__(MG_THREADS) void gemm_mfma_narrow_kernel(MGemmArgs a) {
  static_assert(!MERGE || (NORM < 0 && !PAIRED), "the output projection");
  extern __shared__ float4 lds4[];
  char* const lds = (char*)lds4;
  const MGemmGroup& G = a.g[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = G.M, K = a.K, KT = a.KT, grid = gridDim.x, xrow = a.xrow;
  float* const red = (float*)lds;
  float* const part = (float*)(lds + MG_NARROW_LDS);                   // [T][8 waves][M][16]
  char* const xs = lds + MG_NARROW_LDS + T * MG_WAVES * M * 64;
  // ---- requests.  Unit u: row u / nv, pieces 64 (u % nv) ..
  constexpr int UM = MG_NARROW_ROWS * ((NB + 1) / 2) / MG_WAVES;       // units of a wave at most
  const int nv = (K + 511) / 512, units = M * nv;
  float x[UM][8]; u32x4 gq[UM], bq[UM];
  auto unit = [&](int i, int& m, int& c) { const int u = wave + i * MG_WAVES; m = u / nv; c = (u - m * nv) * WAVE + lane; };
  // (partials of chunks past the position are read, as far as there may be any, and left out)
  float2 pt[MERGE ? MG_MERGE : 1][5];
  auto partials = [&](int i) {
    int m, c; unit(i, m, c);
    const int k = c * 8 < K ? c * 8 : 0, h = k / a.HD;
    const float* const p0 = G.part + (((size_t)m * a.H + h) * a.nchunk_max) * (a.HD + 2);
#pragma unroll
    for (int q = 0; q < MG_MERGE; ++q)
      if (q < a.nmerge) {
        const float* const pq = p0 + (size_t)q * (a.HD + 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) pt[q][e] = ((const float2*)(pq + (k - h * a.HD)))[e];
        pt[q][4] = *(const float2*)(pq + a.HD);
      }
  };
  if constexpr (MERGE) {
    if (wave < units) partials(0);
  } else
#pragma unroll
  for (int i = 0; i < UM; ++i)
    if (wave + i * MG_WAVES < units) {
      int m, c; unit(i, m, c);
      const int k = c * 8 < K ? c * 8 : 0;
      const float4* const px = (const float4*)(G.X + (size_t)m * a.ldx + k);
      const float4 v = px[0], w = px[1];
      x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w; x[i][4] = w.x; x[i][5] = w.y; x[i][6] = w.z; x[i][7] = w.w;
      if constexpr (NORM >= 0) gq[i] = *(const u32x4*)((const uint16_t*)G.ng + k);
      if constexpr (NORM == 0) bq[i] = *(const u32x4*)((const uint16_t*)G.nb + k);
    }
  const int nb8 = (KT + MG_WAVES - 1) / MG_WAVES;
  const int kb0 = wave * nb8 < KT ? wave * nb8 : KT;
  const int nblk = (kb0 + nb8 < KT ? kb0 + nb8 : KT) - kb0;
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)G.P, 0, (int)a.wbytes, 0x00020000);
  // Blocks past the share or the last tile lie past the buffer's end: nothing is read for them.  (Re-reading the start of the matrix instead, one
  // kilobyte that every wave of the launch asked for, took a tenth of a narrow model's token: 384 wide, 12 layers, 262 -> 234 us, 768
  // 289 -> 264, its PPD round 320 -> 298.)
  // Half a tile per workgroup: lanes l % 16 of the other eight rows have nothing to read, and their rows' outputs are the other workgroup's
  constexpr bool CUT = T == 1 && !PAIRED;
  const int cut = CUT ? a.halves : 0, sub = (int)blockIdx.x & cut;
  const bool mine = !cut || (lane >> 3 & 1) == sub;
  u32x4 w[T][NB];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int tile = CUT ? (int)blockIdx.x >> cut : (int)blockIdx.x + t * grid;
#pragma unroll
    for (int j = 0; j < NB; ++j)
      w[t][j] = __builtin_amdgcn_raw_buffer_load_b128(wres, mine && tile < a.NT && j < nblk ? (unsigned)(tile * KT + kb0 + j) * 1024u + lane * 16u : a.wbytes, 0, 2);   // 2: non-temporal
  }
  // bias and residual of the output this thread will finish: row of the tile, row of the input, tile
  const int R = PAIRED ? 8 : 16 >> cut, rsh = PAIRED ? 3 : 4 - cut;
  const int orow = (tid & (R - 1)) + (sub << rsh), ord = (tid >> rsh) / M, ocol = (tid >> rsh) - ord * M;
  const int n = CUT ? ((int)blockIdx.x >> cut) * 16 + orow : ((int)blockIdx.x + ord * grid) * R + orow;
  const bool out = ord < T && n < a.ntot;
  const uint16_t* const B0 = (const uint16_t*)G.B[0];
  const uint16_t* const B1 = (const uint16_t*)G.B[1];
  const uint16_t* const B2 = (const uint16_t*)G.B[2];
  uint32_t b0 = 0u, b1 = 0u; float rsd = 0.f;
  if (out) {
    if (PAIRED) {
      if (B0) b0 = B0[n];
      if (B1) b1 = B1[n];
    } else if (B0) {
      int seg = 0, loc = n;
      if (loc >= a.N[0]) { loc -= a.N[0]; seg = 1; if (loc >= a.N[1]) { loc -= a.N[1]; seg = 2; } }
      b0 = (seg == 0 ? B0 : (seg == 1 ? B1 : B2))[loc];
    }
    if (G.Rsd) rsd = G.Rsd[(size_t)ocol * a.ldy + n];
  }
  if constexpr (MERGE) {
    const int nc = (a.ds->pos + G.pos_off) / ATT_CHUNK + 1;
#pragma unroll
    for (int i = 0; i < UM; ++i)
      if (wave + i * MG_WAVES < units) {
        if (i > 0) partials(i);
        float gm = -INFINITY, ll = 0.f, oo[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto add = [&](float wq, const float2 (&t)[5], float (&o)[8], float& l) {
          l = fmaf(wq, t[4].y, l);
#pragma unroll
          for (int e = 0; e < 4; ++e) { o[2 * e] = fmaf(wq, t[e].x, o[2 * e]); o[2 * e + 1] = fmaf(wq, t[e].y, o[2 * e + 1]); }
        };
#pragma unroll
        for (int q = 0; q < MG_MERGE; ++q) if (q < nc) gm = fmaxf(gm, pt[q][4].x);
        if (a.HD == 64) {                      // a slice has one chunk
#pragma unroll
          for (int q = 0; q < MG_MERGE; ++q) if (q < nc) add(expf(pt[q][4].x - gm), pt[q], oo, ll);
        } else {                               // chunks q and q + 4 are a slice
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q < nc) {
              const bool two = q + 4 < nc;
              const float ms = two ? fmaxf(pt[q][4].x, pt[q + 4][4].x) : pt[q][4].x;
              float2 sl[5] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
              float os[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
              add(expf(pt[q][4].x - ms), pt[q], os, sl[4].y);
              if (two) add(expf(pt[q + 4][4].x - ms), pt[q + 4], os, sl[4].y);
#pragma unroll
              for (int e = 0; e < 4; ++e) sl[e] = make_float2(os[2 * e], os[2 * e + 1]);
              add(expf(ms - gm), sl, oo, ll);
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) x[i][e] = oo[e] / ll;
      }
  }
  // ---- statistics: a unit's 64 pieces by butterfly, a row's units in order (what the norm's idle waves would add is zero)
  auto combine = [&](const float* r) { float s = r[0]; for (int v = 1; v < nv; ++v) s += r[v]; return s + 0.f; };
  float mu[UM], rs[UM];
#pragma unroll
  for (int i = 0; i < UM; ++i) { mu[i] = 0.f; rs[i] = 1.f; }
  if constexpr (NORM == 0) {
#pragma unroll
    for (int i = 0; i < UM; ++i)
      if (wave + i * MG_WAVES < units) {
        int m, c; unit(i, m, c);
        float sm = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sm += x[i][e];
        sm = wave_sum(c * 8 < K ? sm : 0.f);
        if (lane == 0) red[m * 8 + (c >> 6)] = sm;
      }
    __syncthreads();
  }
  if constexpr (NORM >= 0) {
    float* const redB = red + MG_NARROW_ROWS * 8;
#pragma unroll
    for (int i = 0; i < UM; ++i)
      if (wave + i * MG_WAVES < units) {
        int m, c; unit(i, m, c);
        if constexpr (NORM == 0) mu[i] = combine(red + m * 8) / (float)K;
        float s2 = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float d = x[i][e] - mu[i]; s2 = fmaf(d, d, s2); }
        s2 = wave_sum(c * 8 < K ? s2 : 0.f);
        if (lane == 0) redB[m * 8 + (c >> 6)] = s2;
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < UM; ++i)
      if (wave + i * MG_WAVES < units) {
        int m, c; unit(i, m, c);
        rs[i] = 1.0f / sqrtf(combine(redB + m * 8) / (float)K + a.eps);
      }
  }
  // ---- normalised, in two bf16 terms: hi(k .. k + 7) | lo(k .. k + 7) of a piece in 32 bytes
#pragma unroll
  for (int i = 0; i < UM; ++i)
    if (wave + i * MG_WAVES < units) {
      int m, c; unit(i, m, c);
      float xv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = x[i][e];
      if constexpr (NORM >= 0) {
        float gf[8]; WTr<bf16_t>::unpack(gq[i], gf);
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] = (xv[e] - mu[i]) * rs[i] * gf[e];
      }
      if constexpr (NORM == 0) {
        float bf[8]; WTr<bf16_t>::unpack(bq[i], bf);
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] += bf[e];
      }
      uint32_t hp[4], lp[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){xv[2 * e], xv[2 * e + 1]}, bf16x2));
        const float r0 = xv[2 * e] - __uint_as_float(hp[e] << 16), r1 = xv[2 * e + 1] - __uint_as_float(hp[e] & 0xffff0000u);
        lp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){r0, r1}, bf16x2));
      }
      const bool in = c * 8 < K;
      if (c < KT * 4) {
        uint4* const px = (uint4*)(xs + m * xrow + c * 32);
        px[0] = in ? make_uint4(hp[0], hp[1], hp[2], hp[3]) : make_uint4(0u, 0u, 0u, 0u);
        px[1] = in ? make_uint4(lp[0], lp[1], lp[2], lp[3]) : make_uint4(0u, 0u, 0u, 0u);
      }
    }
  __syncthreads();
  // ---- multiply: lane l feeds column l % 16 (input row; lanes past M read row 0), the eight k of piece l / 16 of a block
  const int bm = lane & 15, bc = lane >> 4;
  const char* const xlane = xs + (bm < M ? bm : 0) * xrow + bc * 32 + kb0 * 128;
  f32x4 acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (j < nblk) {                            // the same for the whole wave
      const u32x4* const xp = (const u32x4*)(xlane + j * 128);
      const bf16x8 bh = __builtin_bit_cast(bf16x8, xp[0]), bl = __builtin_bit_cast(bf16x8, xp[1]);
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[t][j]), bh, acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[t][j]), bl, acc[t], 0, 0, 0);
    }
  // lane l holds rows 4 (l / 16) .. + 3 of the tile for input row l % 16
  if (bm < M)
#pragma unroll
    for (int t = 0; t < T; ++t) *(f32x4*)(part + ((t * MG_WAVES + wave) * M + bm) * 16 + bc * 4) = acc[t];
  __syncthreads();
  // ---- the eight partials of an output in wave order, bias, activation, residual
  if (!out) return;
  const float c0 = __uint_as_float(b0 << 16), c1 = __uint_as_float(b1 << 16);
  const float* const pp = part + (ord * MG_WAVES * M + ocol) * 16 + orow;
  float s = pp[0];
#pragma unroll
  for (int v = 1; v < MG_WAVES; ++v) s += pp[v * M * 16];
  float y;
  if (PAIRED) {
    float u = pp[8];
#pragma unroll
    for (int v = 1; v < MG_WAVES; ++v) u += pp[v * M * 16 + 8];
    y = silu(s + c0) * (u + c1);
  } else {
    y = s + c0;
    if (a.act == 1) y = gelu_erf(y);
    else if (a.act == 2) y = fmaxf(y, 0.f);
  }
  y += rsd;
  G.Y[(size_t)ocol * a.ldy + n] = y;
}

}  // namespace ppd
