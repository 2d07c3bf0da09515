// All layers of one row in one launch (bf16 models, gfx950): plain steps, and the main token's way to the exit layer.
//
// One workgroup per compute unit stays for the whole chain and goes through the layers' steps -- QKV projection,
// attention, output projection, FFN in, FFN out -- exchanging the row after each.  The arithmetic of every step, and
// every order of additions, is that of the kernels that run the steps one launch at a time (gemm_mfma_kernel,
// attn_kernel, attn_merge_kernel), so the bits are the same.
//
// What bounds a decode step is the stream of weights, and one launch per step loses the stream at every boundary: ramp,
// row -> norm -> conversion -> first MFMA, uneven finish (7B shape: 90 us a layer where the stream alone takes 60).  None
// of that needs the stream to stop: the weights (and the cached keys and values) of a step are known long before its
// input row is.  Here a workgroup is eight multiplying waves, each with a ring of FU_RING register batches (24 KiB), and
// four helper waves.  A multiplying wave that is done with a step fills its ring with the first batches of the next one
// before it waits for anything: 256 workgroups hold 48 MiB that way, about seven microseconds of the stream.
// Meanwhile the helpers add up the step's outputs, publish them, and bring the next step's row into LDS; they have no
// weight requests in flight, so nothing of this queues behind the ring (a wave's loads return in order).
// Measured (MI355X, context 512, one token): 7B shape 3.09 -> 2.60 ms.  (Widths from 320 to 1024, the OPT-125m shape among them,
// go launch by launch: launches_pay, ppd_engine.hip.)  Every 1000 positions
// take about 1 us a layer from that: the attention's items pay for their barriers, and the launches are the faster way
// from some 4000 - 12000 positions on (the rule and its figures: chain_pays, ppd_engine.hip).
//
// Exchange between workgroups.  Every step of every layer has an output buffer of its own, filled with FU_EMPTY before the
// round.  FU_EMPTY is a signalling NaN, which no arithmetic returns, so a value says by itself that it is there: the
// consumer reads until it finds no FU_EMPTY.  No flag, no acknowledgement, no fence; a step's critical path is one
// store on its way to memory and one load.  (With flags: 2.82 instead of 3.16 ms per token.)  Stores and loads are
// relaxed atomic accesses of agent scope (sc1: past the XCD's L2, which is not coherent with the other seven).
//
// All workgroups of the launch have to be on the machine at once.  The host launches one per compute unit, and only while no
// other context has work in flight; should another program hold compute units all the same, every wait ends after
// spin_ticks of the 100 MHz clock: the workgroup then sets DevState::aborted, waits for nothing any more, and runs to
// the end on whatever is there; the selection kernel sees the mark and leaves the round's state alone, and the host
// runs the round again one launch per step (and keeps to that for a while).
//
// Two row groups (the pipelined steps) stay with one launch per step: k rows that every compute unit reads from memory
// instead of from its XCD's L2 cost more than the boundaries do (7B shape, k = 5: 189 us a step against 162).
#pragma once
#include "ppd_kernels.h"

namespace ppd {

constexpr int FU_HELPERS = 4;                      // helper waves (twelve waves in all: three per SIMD, 168 registers each)
constexpr int FU_THREADS = MG_THREADS + FU_HELPERS * WAVE;
constexpr int FU_PACE = 8;                         // a wave requests a batch when at most this many of its blocks are in flight
constexpr int FU_PACE_AHEAD = 0;                   // the same for what is requested ahead of a step (the helpers' few accesses
                                                   // go through the same queue)
constexpr int FU_RING = 6;                         // register batches of MG_BATCH KiB per multiplying wave
// NARROW instances of the kernel: every workgroup's share of every product fits the ring, so a layer is latency and no stream.
// What is requested ahead goes out at once and only what is wanted, where the others wait for one batch before they request
// the next, wanted or not: six memory latencies in the way of each product.  Measured (a plain token, us per layer,
// without / with): OPT-like 256 wide 24.0 / 22.7, LLaMA-like 2048 39.0 / 38.1; where shares do not fit: 2560 46.8 / 48.7, 4096
// 79.3 / 84.4.
constexpr int FU_KV = FU_RING - 4;                 // the last four take an attention item's keys and values
constexpr int FU_SLEEP = 4;                        // 64 clocks each, between two looks at pieces of a row that are not there yet
constexpr int FU_MAX_WG = 256;
constexpr uint32_t FU_EMPTY = 0x7fa5a5a5u;
constexpr int FU_LDS_SUMS = 0, FU_LDS_DONE = 1024, FU_LDS_G = 2048;   // sums of the norm, tiles done per wave, the norm's gain

// one layer's pointers (a table in device memory)
struct FLayer {
  const void* P[4];                 // repacked weights: QKV, O, FFN in, FFN out
  const void* ng[2]; const void* nb[2];   // gain and bias of the two norms
  const void* B[4][3];              // biases of the four products, per row segment (paired: gate, up)
  float *Kc, *Vc;
};
struct FPhase {                     // one of the four products
  int K, KT, NT, ntot, nseg;        // nseg: rows per bias segment
  int norm;                         // -1 none
  int paired, act;
  unsigned wbytes;
  int inv;                          // 2^16 / (batches per tile), rounded up
};
struct FusedArgs {
  const FLayer* L;
  FPhase ph[4];
  int layer0, nsteps;               // layers layer0 .. layer0 + nsteps - 1
  int off_res, off_part, off_x;     // LDS: residuals of the workgroup's outputs, partial sums, staged row (or the attention's)
  float *h, *part;                  // the row (first layer's input, last layer's output); attention partials [H][nchunk_max][hd+2],
                                    // FU_EMPTY whenever they are not in use
  float* ex;                        // outputs of the steps: fu_ex_row floats per layer
  const float2* rope;
  DevState* ds;
  int H, d_model, d_ff, max_ctx, nchunk_max;
  unsigned kv_bytes;                // bytes of one layer's keys
  float scale, eps;
  int spin_ticks;
};

// floats of ex per layer: the outputs of QKV, attention, O, FFN in, FFN out
__host__ __device__ inline size_t fu_ex_row(int dm, int F) { return (size_t)6 * dm + F; }
__host__ __device__ inline int fu_gain_bytes(int dm) { return (dm * 2 + 1023) & ~1023; }
// floats of the attention's LDS
__host__ __device__ inline int fu_att_floats(int HD) { return 15 * HD + 2 * ATT_CHUNK + 8 + MG_THREADS + 16; }

#ifdef PPD_FUSED_TU

typedef const __attribute__((address_space(4))) struct FusedArgs* FArgs;   // read by scalar loads (a vector load would queue
typedef const __attribute__((address_space(4))) struct FLayer* FTab;       // behind the ring), dynamic indexes included
extern __shared__ float4 fu_lds4[];

// a value the compiler may not compute ahead for all layers at once: what is derived from it lives only where it is used
__device__ __forceinline__ int fu_here(int v) { asm volatile("" : "+v"(v)); return v; }
__device__ __forceinline__ void fu_bar() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void fu_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// dma16 where the compiler cannot see that all lanes have the same destination
__device__ __forceinline__ unsigned fu_lds_addr(const void* p) { return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p); }
__device__ __forceinline__ void fu_dma16(const void* src, void* lds_dst) {
  const unsigned la = fu_lds_addr(lds_dst);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(la) : "memory", "m0");
}
// ... at agent scope: not from this XCD's L2
__device__ __forceinline__ void dma16_agent(const void* src, void* lds_dst) {
  const unsigned la = fu_lds_addr(lds_dst);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off sc1" ::"v"(src), "s"(la) : "memory", "m0");
}
template <typename T> __device__ __forceinline__ T ld_agent(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ void st_agent(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// A wave's share of one product: batch j is batch j % NBT of the workgroup's tile j / NBT
struct FSeg {
  const char* P; unsigned wbytes;
  int Q, NBT, inv;          // batches, batches per tile, 2^16 / NBT rounded up (j / NBT for small j)
  unsigned o0, tstride;     // byte offset of batch 0, distance of two tiles of the workgroup
  int nrun;                 // blocks of a tile
};
// MG_BATCH blocks to request: byte offset o of a buffer, the first n of them are wanted
struct FReq { const char* P; unsigned bytes, o; int n; };

// What a workgroup works on (the same for all its waves, but for the wave's own numbers)
struct FWg {
  FArgs a; FTab tab;
  int tid, lane, wave;
  int idx, G, pos;                       // this workgroup's number, workgroups, the row's position
  int nchunk, ncp, it0, it1;             // attention: 64-position chunks, pairs of them, this workgroup's items (head, pair)
  __device__ __forceinline__ char* lds() const { return (char*)fu_lds4; }
  __device__ __forceinline__ int my_tiles(int i) const { const int NT = a->ph[i].NT; return idx < NT ? (NT - idx + G - 1) / G : 0; }
};
// LDS of the attention: rotation, raw row, rotated q, k, v, scores, statistics, the blocks' outputs; the merge's
template <int HD> struct FAttLds {
  float *rope, *raw, *qs, *ko, *vo, *sc, *st, *ored, *merge;
  __device__ __forceinline__ FAttLds(int off) {
    rope = (float*)((char*)fu_lds4 + off);
    raw = rope + HD; qs = raw + 3 * HD; ko = qs + HD; vo = ko + HD;
    sc = vo + HD;                        // [2][ATT_CHUNK]
    st = sc + 2 * ATT_CHUNK;             // [2][4]
    ored = st + 8;                       // [2][ATT_WAVES][HD]
    merge = ored + 2 * ATT_WAVES * HD;   // [MG_THREADS], then maxima and sums of the slices
  }
};
// The output buffers of a layer's steps
struct FEx {
  float *qkv, *att, *o, *fin, *fout;
  __device__ __forceinline__ FEx(const FWg& w, int step) {
    const int dm = w.a->d_model, F = w.a->d_ff;
    qkv = w.a->ex + (size_t)step * fu_ex_row(dm, F);
    att = qkv + (size_t)3 * dm; o = att + dm; fin = o + dm; fout = fin + F;
  }
};

// ---- waits for other workgroups end: after spin_ticks the launch is given up and nothing is waited for any more
struct FWait {
  long long t0; bool dead;
  __device__ __forceinline__ void begin() { t0 = wall_clock64(); }
  __device__ __forceinline__ bool give_up(const FWg& w) {
    if (!dead && wall_clock64() - t0 > w.a->spin_ticks) {
      dead = true;
      if (w.lane == 0) st_agent(&w.a->ds->aborted, 1);
    }
    return dead;
  }
};

// ---- the helper waves
struct FHelper {
  int wave;                              // among the helpers
  uint32_t tiles;                        // tiles of the products that are over
  FWait wait;
};
// Pieces of a kilobyte each into LDS, this wave's being 0 .. n - 1 (n <= 32); piece(q, src, dst): address of this lane's 16
// bytes and the piece's place, false for a lane that has none.  A piece is there when no lane finds FU_EMPTY in it.
template <typename F>
__device__ __forceinline__ void fu_stage(const FWg& w, FHelper& hp, int n, F piece) {
  uint32_t todo = n >= 32 ? 0xffffffffu : (1u << n) - 1;
  hp.wait.begin();
  while (todo) {
    for (uint32_t b = todo; b; b &= b - 1) {
      const float* src; char* dst;
      if (piece(__builtin_ctz(b), src, dst)) dma16_agent(src, dst);
    }
    fu_landed();
    const uint32_t before = todo;
    for (uint32_t b = todo; b; b &= b - 1) {
      const float* src; char* dst;
      bool there = true;
      if (piece(__builtin_ctz(b), src, dst)) {
        const u32x4 v = *(const u32x4*)(dst + w.lane * 16);
        there = v.x != FU_EMPTY && v.y != FU_EMPTY && v.z != FU_EMPTY && v.w != FU_EMPTY;
      }
      if (__all(there)) todo &= ~(b & -b);
    }
    if (todo && hp.wait.give_up(w)) break;
    if (todo == before) __builtin_amdgcn_s_sleep(FU_SLEEP);
  }
}

// gain and bias of the norm in front of product i (0 or 2) into LDS
__device__ __forceinline__ void fu_gain(const FWg& w, const FHelper& hp, int i, int layer) {
  const int K = w.a->ph[i].K, norm = w.a->ph[i].norm;
  const uint16_t* const ng = (const uint16_t*)w.tab[layer].ng[i >> 1];
  const uint16_t* const nb = (const uint16_t*)w.tab[layer].nb[i >> 1];
  char* const dst = w.lds() + FU_LDS_G;
  for (int u = hp.wave; u * 512 < K; u += FU_HELPERS) {
    const int kk = u * 512 + w.lane * 8;
    if (kk < K) {
      fu_dma16(ng + kk, dst + u * 1024);
      if (norm == 0) fu_dma16(nb + kk, dst + fu_gain_bytes(w.a->d_model) + u * 1024);
    }
  }
}
// x = hi + lo in two bf16 terms, in place of eight floats
__device__ __forceinline__ void fu_split(char* px, const float (&xv)[8]) {
  uint32_t hp[4], lp[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    hp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){xv[2 * e], xv[2 * e + 1]}, bf16x2));
    const float r0 = xv[2 * e] - __uint_as_float(hp[e] << 16), r1 = xv[2 * e + 1] - __uint_as_float(hp[e] & 0xffff0000u);
    lp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){r0, r1}, bf16x2));
  }
  ((uint4*)px)[0] = make_uint4(hp[0], hp[1], hp[2], hp[3]);
  ((uint4*)px)[1] = make_uint4(lp[0], lp[1], lp[2], lp[3]);
}
// The input row of product i into LDS.  Kilobyte pieces 2 v, 2 v + 1, 2 v + 16, ... are those whose elements multiplying wave v's
// threads own in the norm's order of additions; helper wave v has them and those of wave v + 4.  Behind an RMS norm the
// helpers leave the eight waves' sums of squares; without a norm they split the row into its two terms right away.
__device__ __forceinline__ void fu_row(const FWg& w, FHelper& hp, int i, int step) {
  const auto& p = w.a->ph[i];
  const int K = p.K, KT = p.KT, norm = p.norm, lane = w.lane;
  char* const xs = w.lds() + w.a->off_x;
  const FEx ex(w, step);
  const float* const X = i == 0 ? (step ? FEx(w, step - 1).fout : w.a->h) : (i == 1 ? ex.att : (i == 2 ? ex.o : ex.fin));
  const int U = (KT * 32 + 255) >> 8, mine = (U + 15) / 16 * 4;
  // this wave's piece q: of multiplying wave hp.wave (q % 4 < 2) or hp.wave + 4
  const int v0 = hp.wave;
  for (int q0 = 0; q0 < mine; q0 += 32)
    fu_stage(w, hp, mine - q0 < 32 ? mine - q0 : 32, [&](int q, const float*& src, char*& dst) {
      q += q0;
      const int u = (q >> 2) * 16 + 2 * (v0 + 2 * (q & 2)) + (q & 1), col = u * 256 + lane * 4;
      src = X + col;
      dst = xs + u * 1024;
      return col < K;
    });
  if (norm == 1) {
    float* const redB = (float*)(w.lds() + FU_LDS_SUMS) + MG_WAVES;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int v = v0 + 4 * x;
      float s2 = 0.f;
      for (int c = v * WAVE + lane; c * 8 < K; c += MG_THREADS) {
        const float4* px = (const float4*)(xs + c * 32);
        const float4 a = px[0], b = px[1];
        const float d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) s2 = fmaf(d[e], d[e], s2);
      }
      s2 = wave_sum(s2);
      if (lane == 0) redB[v] = s2;
    }
  } else if (norm < 0) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
      for (int c = (v0 + 4 * x) * WAVE + lane; c < KT * 4; c += MG_THREADS) {
        char* const px = xs + c * 32;
        float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (c * 8 < K) {
          const float4 a = ((const float4*)px)[0], b = ((const float4*)px)[1];
          xv[0] = a.x; xv[1] = a.y; xv[2] = a.z; xv[3] = a.w; xv[4] = b.x; xv[5] = b.y; xv[6] = b.z; xv[7] = b.w;
        }
        fu_split(px, xv);
      }
  }
}
// all multiplying waves have left their partial sums of so many tiles since the launch began
__device__ __forceinline__ void fu_wait_tiles(const FWg& w, uint32_t n) {
  const uint32_t* const done = (const uint32_t*)(w.lds() + FU_LDS_DONE);
  for (;;) {
    const uint32_t v = __hip_atomic_load(done + (w.lane & (MG_WAVES - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__all((int)(v - n) >= 0)) break;
    __builtin_amdgcn_s_sleep(1);
  }
  asm volatile("" ::: "memory");
}
// The outputs of a product, tile by tile as they become complete (each helper wave its own tiles): the eight partial sums
// in wave order, bias, activation, residual.  Returns when the multiplying waves are done with the product.
__device__ __forceinline__ void fu_outputs(const FWg& w, FHelper& hp, int i, int step, bool end) {
  const auto& p = w.a->ph[i];
  const auto& L = w.tab[w.a->layer0 + step];
  const int ntiles = w.my_tiles(i), paired = p.paired, act = p.act, ntot = p.ntot, nseg = p.nseg, R = paired ? 8 : 16;
  const FEx ex(w, step);
  float* const Y = i == 0 ? ex.qkv : (i == 1 ? ex.o : (i == 2 ? ex.fin : (end ? w.a->h : ex.fout)));
  const uint16_t* const B0 = (const uint16_t*)L.B[i][0];
  const uint16_t* const B1 = (const uint16_t*)L.B[i][1];
  const uint16_t* const B2 = (const uint16_t*)L.B[i][2];
  const int row = w.lane & (R - 1);
  for (int ord = hp.wave; ord < ntiles; ord += FU_HELPERS) {
    const int n = (w.idx + ord * w.G) * R + row;
    const bool mine = w.lane < R && n < ntot;
    uint32_t b0 = 0u, b1 = 0u;
    if (B0 && mine) {
      if (paired) {
        b0 = B0[n];
        if (B1) b1 = B1[n];
      } else {
        const int seg = n / nseg, loc = n - seg * nseg;
        b0 = (seg == 0 ? B0 : (seg == 1 ? B1 : B2))[loc];
      }
    }
    fu_wait_tiles(w, hp.tiles + ord + 1);
    if (mine) {
      const float c0 = __uint_as_float(b0 << 16), c1 = __uint_as_float(b1 << 16);
      const float* pp = (const float*)(w.lds() + w.a->off_part) + ord * MG_WAVES * 16 + row;
      float s = pp[0];
#pragma unroll
      for (int v = 1; v < MG_WAVES; ++v) s += pp[v * 16];
      float y;
      if (paired) {
        float u = pp[8];
#pragma unroll
        for (int v = 1; v < MG_WAVES; ++v) u += pp[v * 16 + 8];
        y = silu(s + c0) * (u + c1);
      } else {
        y = s + c0;
        if (act == 1) y = gelu_erf(y);
        else if (act == 2) y = fmaxf(y, 0.f);
      }
      // (both products with a residual have the same tiles: a workgroup's residuals are its own earlier outputs)
      if (i & 1) {
        float* const r = (float*)(w.lds() + w.a->off_res) + ord * 16 + row;
        y += *r;
        *r = y;
      }
      st_agent(Y + n, y);
    }
  }
  hp.tiles += ntiles;
  fu_wait_tiles(w, hp.tiles);
}

template <int HD>
__device__ __forceinline__ void fu_help_attention(const FWg& w, FHelper& hp, int step) {
  const int lane = w.lane, dm = w.a->d_model, ncp = w.ncp;
  const FAttLds<HD> s(w.a->off_x);
  const float2* const rope = w.a->rope;
  const float* const qkv = FEx(w, step).qkv;
  for (int it = w.it0; it < w.it1; ++it) {
    if (it == w.it0 || it % ncp == 0) {  // another head: its query, key and value
      const int hh = it / ncp;
      if (it == w.it0 && hp.wave == FU_HELPERS - 1 && rope && lane * 4 < HD) fu_dma16((const float*)(rope + (size_t)w.pos * (HD / 2)) + lane * 4, s.rope);
      const int q0 = hp.wave;
      fu_stage(w, hp, q0 < (3 * HD + 255) / 256 ? 1 : 0, [&](int, const float*& src, char*& dst) {
        const int f = q0 * 256 + lane * 4, sec = f / HD, i = f - sec * HD;
        src = qkv + (size_t)sec * dm + (size_t)hh * HD + i;
        dst = (char*)(s.raw + q0 * 256);
        return f < 3 * HD;
      });
      fu_landed();
      fu_bar();      // raw row
      fu_bar();      // rotated
    }
    fu_bar();        // scores
    fu_bar();        // weights
    fu_bar();        // outputs of the blocks
  }
  for (int it = w.it0; it < w.it1; ++it)
    if (it % ncp == 0) { fu_bar(); fu_bar(); }     // heads merged here
  fu_bar();          // the attention's LDS is free
}

// ---- the multiplying waves
// Every batch is requested in full: blocks that are not wanted are asked for past the end of the buffer, and not read.  (The start of the
// buffer in their place: a plain token of 8 layers, 256 wide 207 -> 196 us, 1536 298 -> 293, 2048 348 -> 346, 4096 the same.)
template <int PACE>
__device__ __forceinline__ void fu_request(u32x4 (&buf)[MG_BATCH], unsigned lane16, const char* P, unsigned bytes, unsigned o, int n) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)P, 0, (int)bytes, 0x00020000);
  if constexpr (PACE < 16) __builtin_amdgcn_s_waitcnt(0xF70 | PACE);        // vmcnt(PACE)
#pragma unroll
  for (int j = 0; j < MG_BATCH; ++j) buf[j] = __builtin_amdgcn_raw_buffer_load_b128(r, j < n ? lane16 + j * 1024u : bytes, j < n ? o : 0u, 2);   // 2: non-temporal
}
#define FU_REQUEST(slot, q) do { const FReq q_ = (q); fu_request<FU_PACE>(ring[slot], lane16, q_.P, q_.bytes, q_.o, q_.n); } while (0)
#define FU_AHEAD(slot, q) do { const FReq q_ = (q); if constexpr (!NARROW) fu_request<FU_PACE_AHEAD>(ring[slot], lane16, q_.P, q_.bytes, q_.o, q_.n); \
    else if (q_.n > 0) fu_request<63>(ring[slot], lane16, q_.P, q_.bytes, q_.o, q_.n); } while (0)
__device__ __forceinline__ FSeg fu_seg(const FWg& w, int i, int layer) {
  const auto& p = w.a->ph[i];
  const int KT = p.KT, nb8 = (KT + MG_WAVES - 1) / MG_WAVES;
  const int kb0 = w.wave * nb8 < KT ? w.wave * nb8 : KT;
  FSeg s;
  s.P = (const char*)w.tab[layer].P[i]; s.wbytes = p.wbytes;
  s.NBT = (nb8 + MG_BATCH - 1) / MG_BATCH;
  s.inv = p.inv;
  s.Q = w.my_tiles(i) * s.NBT;
  s.o0 = (unsigned)(w.idx * KT + kb0) * 1024u;
  s.tstride = (unsigned)(w.G * KT) * 1024u;
  s.nrun = (kb0 + nb8 < KT ? kb0 + nb8 : KT) - kb0;
  return s;
}
// batch j < FU_RING of a product: what slot j of the ring holds when the product begins
__device__ __forceinline__ FReq fu_ahead(const FSeg& s, int j) {
  const int t = (j * s.inv) >> 16, bt = j - t * s.NBT;
  return FReq{s.P, s.wbytes, s.o0 + (unsigned)t * s.tstride + (unsigned)bt * (MG_BATCH * 1024u), j < s.Q ? s.nrun - bt * MG_BATCH : 0};
}
// ring slots FU_KV ..: an attention item's keys, then its values.  Waves 0-3 have the first chunk of the pair, 4-7 the second
template <int HD>
__device__ __forceinline__ FReq fu_kv(const FWg& w, int layer, int it, int slot) {
  constexpr int NS = HD / 16, NKB = NS / MG_BATCH;
  const bool isv = slot >= NKB;
  const int hh = it / w.ncp, cp = it - hh * w.ncp;
  int c = 2 * cp + (w.wave >> 2);
  if (c >= w.nchunk) c = w.nchunk - 1;
  const unsigned blk = (unsigned)hh * (unsigned)kv_blocks(w.a->max_ctx) + (unsigned)(c * (ATT_CHUNK / KV_BLOCK) + (w.wave & 3));
  const char* const kc = (const char*)w.tab[layer].Kc; const char* const vc = (const char*)w.tab[layer].Vc;
  return FReq{isv ? vc : kc, w.a->kv_bytes, blk * (NS * 1024u) + (unsigned)(isv ? slot - NKB : slot) * (MG_BATCH * 1024u), MG_BATCH};
}
// What ring slot r is to hold when product i is over: the next product's batches; in front of the attention, its last slots
// the first item's keys and values
template <int HD>
__device__ __forceinline__ FReq fu_next(const FWg& w, int r, int i, const FSeg& nx, int layer) {
  constexpr int NKB = HD / 16 / MG_BATCH;
  static_assert(FU_KV + 2 * NKB <= FU_RING, "an item's keys and values fit the ring's last slots");
  if (r >= FU_KV && r < FU_KV + 2 * NKB && i == 0) return fu_kv<HD>(w, layer, w.it0 < w.it1 ? w.it0 : 0, r - FU_KV);
  return fu_ahead(nx, r);
}

// The row of a product with a norm, split into two bf16 terms in place (as gemm_mfma_kernel does it).  LayerNorm: the
// statistics too (an RMS norm's are there, see fu_row).
__device__ __forceinline__ float fu_combine8(const float* r) { return ((((((r[0] + r[1]) + r[2]) + r[3]) + r[4]) + r[5]) + r[6]) + r[7]; }
__device__ __forceinline__ void fu_convert(const FWg& w, int i) {
  const auto& p = w.a->ph[i];
  const int K = p.K, KT = p.KT, norm = p.norm;
  const int tid = fu_here(w.tid), lane = tid & 63, wave = w.wave;
  char* const xs = w.lds() + w.a->off_x;
  float* const redA = (float*)(w.lds() + FU_LDS_SUMS);
  float* const redB = redA + MG_WAVES;
  float mu = 0.f;
  if (norm == 0) {
    float sm = 0.f;
    for (int c = tid; c * 8 < K; c += MG_THREADS) {
      const float4* px = (const float4*)(xs + c * 32);
      const float4 v = px[0], u = px[1];
      sm += v.x; sm += v.y; sm += v.z; sm += v.w; sm += u.x; sm += u.y; sm += u.z; sm += u.w;
    }
    sm = wave_sum(sm);
    if (lane == 0) redA[wave] = sm;
    fu_bar();
    mu = fu_combine8(redA) / (float)K;
    float s2 = 0.f;
    for (int c = tid; c * 8 < K; c += MG_THREADS) {
      const float4* px = (const float4*)(xs + c * 32);
      const float4 v = px[0], u = px[1];
      const float d[8] = {v.x - mu, v.y - mu, v.z - mu, v.w - mu, u.x - mu, u.y - mu, u.z - mu, u.w - mu};
#pragma unroll
      for (int e = 0; e < 8; ++e) s2 = fmaf(d[e], d[e], s2);
    }
    s2 = wave_sum(s2);
    if (lane == 0) redB[wave] = s2;
    fu_bar();
  }
  const float rs = 1.0f / sqrtf(fu_combine8(redB) / (float)K + w.a->eps);
  const char* const gain = w.lds() + FU_LDS_G;
  for (int c = tid; c < KT * 4; c += MG_THREADS) {
    char* const px = xs + c * 32;
    float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c * 8 < K) {
      const float4 v = ((const float4*)px)[0], u = ((const float4*)px)[1];
      xv[0] = v.x; xv[1] = v.y; xv[2] = v.z; xv[3] = v.w; xv[4] = u.x; xv[5] = u.y; xv[6] = u.z; xv[7] = u.w;
      const u32x4 gq = *(const u32x4*)(gain + c * 16);
      float gf[8]; WTr<bf16_t>::unpack(gq, gf);
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = (xv[e] - mu) * rs * gf[e];
      if (norm == 0) {
        const u32x4 bq = *(const u32x4*)(gain + fu_gain_bytes(w.a->d_model) + c * 16);
        float bf[8]; WTr<bf16_t>::unpack(bq, bf);
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] += bf[e];
      }
    }
    fu_split(px, xv);
  }
}

// State of a product's arithmetic and of its requests
struct FCursor {
  f32x4 acc; int c_b; float* plane;      // accumulator of the tile, its next batch, this lane's partial sums
  int l_b; unsigned l_o;                 // the next batch to request
  uint32_t* done; uint32_t tiles;        // this wave's count of tiles
};
__device__ __forceinline__ void fu_consume(u32x4 (&cur)[MG_BATCH], FCursor& k, const FSeg& s, const char* xlane, bool row) {
#pragma unroll
  for (int j = 0; j < MG_BATCH; ++j) {
    const int t = k.c_b * MG_BATCH + j;
    if (t < s.nrun) {
      const u32x4* xp = (const u32x4*)(xlane + t * 128);
      const u32x4 bh = xp[0], bl = xp[1];
      const bf16x8 av = __builtin_bit_cast(bf16x8, cur[j]);
      k.acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh), k.acc, 0, 0, 0);
      k.acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bl), k.acc, 0, 0, 0);
    }
  }
  if (++k.c_b == s.NBT) {
    if (row) *(f32x4*)k.plane = k.acc;
    asm volatile("" ::: "memory");       // (a wave's LDS writes are done in their order)
    __hip_atomic_store(k.done, ++k.tiles, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    k.plane += MG_WAVES * 16;
    k.acc = (f32x4){0.f, 0.f, 0.f, 0.f};
    k.c_b = 0;
  }
}
__device__ __forceinline__ FReq fu_current(FCursor& k, const FSeg& s) {
  const FReq q{s.P, s.wbytes, k.l_o, s.nrun - k.l_b * MG_BATCH};
  k.l_o += MG_BATCH * 1024u;
  if (++k.l_b == s.NBT) { k.l_b = 0; k.l_o += s.tstride - (unsigned)s.NBT * (MG_BATCH * 1024u); }
  return q;
}

// One product: its first FU_RING batches are in the ring (slot j holds batch j), its end leaves the next one's there.
template <int HD, bool NARROW>
__device__ __forceinline__ void fu_product(const FWg& w, u32x4 (&ring)[FU_RING][MG_BATCH], uint32_t& tiles, int i, const FSeg& s, const FSeg& nx, int layer) {
  const int Q = s.Q;
  const int lane = fu_here(w.tid) & 63;
  const unsigned lane16 = lane * 16;
  const bool next_full = i == 0 || nx.Q >= FU_RING;      // there is something for every slot
  if (Q < FU_RING && next_full) {          // slots this product does not need
#pragma unroll
    for (int r = 0; r < FU_RING; ++r) if (r >= Q) FU_AHEAD(r, fu_next<HD>(w, r, i, nx, layer));
  }
  fu_bar();
  if (w.a->ph[i].norm >= 0) {
    fu_convert(w, i);
    fu_bar();
  }
  // B operand: every lane feeds the eight k of chunk l / 16 (the row is column 0; the other columns are never stored)
  const int bc = lane >> 4;
  const bool row = (lane & 15) == 0;
  const int nb8 = (w.a->ph[i].KT + MG_WAVES - 1) / MG_WAVES;
  const char* const xlane = w.lds() + w.a->off_x + bc * 32 + w.wave * nb8 * 128;
  FCursor k;
  k.acc = (f32x4){0.f, 0.f, 0.f, 0.f}; k.c_b = 0;
  k.plane = (float*)(w.lds() + w.a->off_part) + w.wave * 16 + bc * 4;
  k.done = (uint32_t*)(w.lds() + FU_LDS_DONE) + w.wave; k.tiles = tiles;
  { const int t = (FU_RING * s.inv) >> 16; k.l_b = FU_RING - t * s.NBT; k.l_o = s.o0 + (unsigned)t * s.tstride + (unsigned)k.l_b * (MG_BATCH * 1024u); }
  int q = 0;
  for (; q + 2 * FU_RING <= Q; q += FU_RING) {
#pragma unroll
    for (int r = 0; r < FU_RING; ++r) { fu_consume(ring[r], k, s, xlane, row); FU_REQUEST(r, fu_current(k, s)); }
  }
  int rem = Q - q;                         // below 2 FU_RING; the first FU_RING of them are in the ring
  if (rem >= FU_RING) {
    rem -= FU_RING;
#pragma unroll
    for (int r = 0; r < FU_RING; ++r) {
      fu_consume(ring[r], k, s, xlane, row);
      if (r < rem) FU_REQUEST(r, fu_current(k, s));
    }
  }
#pragma unroll
  for (int r = 0; r < FU_RING - 1; ++r)
    if (r < rem) fu_consume(ring[r], k, s, xlane, row);
  // All other workgroups wait for this product: the next one is requested only now (its requests would queue in front of
  // what this one still waits for), and there is time for it until they are done.
#pragma unroll
  for (int r = 0; r < FU_RING; ++r)
    if (r < Q || !next_full) FU_AHEAD(r, fu_next<HD>(w, r, i, nx, layer));
  tiles = k.tiles;
}

// Attention of this workgroup's items: attn_kernel's arithmetic, then attn_merge_kernel's for the heads whose first item
// is here (their other items' partials are waited for as rows are, and made empty again).
template <int HD>
__device__ __forceinline__ void fu_attention(const FWg& w, u32x4 (&ring)[FU_RING][MG_BATCH], FWait& wait, int step, int layer) {
  constexpr int NS = HD / 16, half = HD / 2, NKB = NS / MG_BATCH;
  const int tid = fu_here(w.tid), lane = tid & 63;
  const unsigned lane16 = lane * 16;
  const int pos = w.pos, ncp = w.ncp, nchunk = w.nchunk;
  const int sub = w.wave >> 2, w4 = w.wave & 3, tid4 = tid & 255, bm = lane & 15, bc = lane >> 4;
  const FAttLds<HD> L(w.a->off_x);
  float* const sc = L.sc + sub * ATT_CHUNK;
  float* const st = L.st + sub * 4;
  float* const ored = L.ored + sub * ATT_WAVES * HD;
  const size_t pstride = (size_t)w.a->nchunk_max * (HD + 2);     // floats of one head's partials
  float* const part = w.a->part;
  for (int it = w.it0; it < w.it1; ++it) {
    const int hh = it / ncp, c = 2 * (it - hh * ncp) + sub;
    const bool live = c < nchunk;
    const int j0 = c * ATT_CHUNK;
    const bool owns = pos >= j0 && pos < j0 + ATT_CHUNK;
    if (it == w.it0 || it % ncp == 0) {
      fu_bar();
      if (tid < HD) {
        const int i = tid;
        float q = L.raw[i], k = L.raw[HD + i];
        const float v = L.raw[2 * HD + i];
        if (w.a->rope) {
          const float2 cz = ((const float2*)L.rope)[i < half ? i : i - half];
          const int ip = i < half ? i + half : i - half;
          const float qo = L.raw[ip], kk = L.raw[HD + ip];
          if (i < half) { q = fmaf(q, cz.x, -(qo * cz.y)); k = fmaf(k, cz.x, -(kk * cz.y)); }
          else          { q = fmaf(q, cz.x, qo * cz.y);    k = fmaf(k, cz.x, kk * cz.y); }
        }
        L.qs[i] = q * w.a->scale; L.ko[i] = k; L.vo[i] = v;
      }
      fu_bar();
    }
    {
      f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const f32x4_t q4 = *(const f32x4_t*)(L.qs + 16 * s + 4 * bc);
        const f32x4_t k4 = __builtin_bit_cast(f32x4_t, ring[FU_KV + s / MG_BATCH][s % MG_BATCH]);
#pragma unroll
        for (int u = 0; u < 4; ++u) sacc = __builtin_amdgcn_mfma_f32_16x16x4f32(k4[u], q4[u], sacc, 0, 0, 0);
      }
      if (it + 1 < w.it1) {
#pragma unroll
        for (int s = 0; s < NKB; ++s) FU_REQUEST(FU_KV + s, fu_kv<HD>(w, layer, it + 1, s));
      }
      if (bm == 0) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int jl = 16 * w4 + 4 * bc + jj, j = j0 + jl;
          if (j != pos) sc[jl] = j < pos ? sacc[jj] : -INFINITY;
        }
      }
    }
    if (owns && w4 == 0) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < HD / WAVE; ++e) s = fmaf(L.qs[lane + e * WAVE], L.ko[lane + e * WAVE], s);
      s = wave_sum(s);
      if (lane == 0) sc[pos - j0] = s;
    }
    fu_bar();
    if (live && w4 == 0) {
      const float v = sc[lane];
      const float mx = wave_max(v);
      const float e = expf(v - mx);
      const float sum = wave_sum(e);
      const bool own = owns && lane == pos - j0;
      sc[lane] = own ? 0.f : e;
      if (own) st[2] = e;
      if (lane == 0) { st[0] = mx; st[1] = sum; }
    }
    fu_bar();
    {
      const f32x4_t p4 = *(const f32x4_t*)(sc + 16 * w4 + 4 * bc);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        f32x4_t oacc = {0.f, 0.f, 0.f, 0.f};
        const f32x4_t v4 = __builtin_bit_cast(f32x4_t, ring[FU_KV + NKB + s / MG_BATCH][s % MG_BATCH]);
#pragma unroll
        for (int u = 0; u < 4; ++u) oacc = __builtin_amdgcn_mfma_f32_16x16x4f32(v4[u], p4[u], oacc, 0, 0, 0);
        if (live && bm == 0) *(f32x4_t*)(ored + w4 * HD + 16 * s + 4 * bc) = oacc;
      }
      if (it + 1 < w.it1) {
#pragma unroll
        for (int s = NKB; s < 2 * NKB; ++s) FU_REQUEST(FU_KV + s, fu_kv<HD>(w, layer, it + 1, s));
      }
    }
    fu_bar();
    if (live && tid4 < HD) {
      const int i = tid4;
      float o = ored[i];
#pragma unroll
      for (int v = 1; v < ATT_WAVES; ++v) o += ored[v * HD + i];
      if (owns) o = fmaf(st[2], L.vo[i], o);
      float* const dst = part + (size_t)hh * pstride + (size_t)c * (HD + 2);
      st_agent(dst + i, o);
      if (i == 0) { st_agent(dst + HD, st[0]); st_agent(dst + HD + 1, st[1]); }
      if (owns) {
        const size_t kb = (size_t)hh * kv_blocks(w.a->max_ctx) * (KV_BLOCK * HD);
        w.tab[layer].Kc[kb + k_index(pos, i, HD)] = L.ko[i];
        w.tab[layer].Vc[kb + v_index(pos, i, HD)] = L.vo[i];
      }
    }
  }
  // slices of attn_merge_kernel (a slice is one or two whole waves), 16 chunks' loads in flight together
  float* const att = FEx(w, step).att;
  constexpr int S = MG_THREADS / HD, UB = 16;
  const int t2 = fu_here(w.tid);
  float* const sm_o = L.merge;
  float* const sl_m = sm_o + MG_THREADS;
  float* const sl_l = sl_m + S;
  const int i = t2 % HD, sl = w.wave * WAVE / HD;
  for (int it = w.it0; it < w.it1; ++it) {
    if (it % ncp != 0) continue;
    const int hh = it / ncp;
    float* const pb = part + (size_t)hh * pstride;
    float mx = -INFINITY, o = 0.f, l = 0.f;
    wait.begin();
    for (int c0 = sl; c0 < nchunk; c0 += UB * S) {
      float tm[UB], ts[UB], to[UB];
      for (;;) {
        bool there = true;
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int c = c0 + u * S;
          tm[u] = ts[u] = to[u] = 0.f;
          if (c < nchunk) {
            const float* pc = pb + (size_t)c * (HD + 2);
            tm[u] = ld_agent(pc + HD); ts[u] = ld_agent(pc + HD + 1); to[u] = ld_agent(pc + i);
          }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u)
          there = there && __float_as_uint(tm[u]) != FU_EMPTY && __float_as_uint(ts[u]) != FU_EMPTY && __float_as_uint(to[u]) != FU_EMPTY;
        if (__all(there) || wait.give_up(w)) break;
      }
      float bmx = mx;
#pragma unroll
      for (int u = 0; u < UB; ++u) if (c0 + u * S < nchunk) bmx = fmaxf(bmx, tm[u]);
      const float rescale = expf(mx - bmx);
      o *= rescale; l *= rescale; mx = bmx;
#pragma unroll
      for (int u = 0; u < UB; ++u)
        if (c0 + u * S < nchunk) {
          const float e = expf(tm[u] - mx);
          o = fmaf(e, to[u], o);
          l = fmaf(e, ts[u], l);
        }
    }
    sm_o[t2] = o;
    if (i == 0) { sl_m[sl] = mx; sl_l[sl] = l; }
    fu_bar();
    if (t2 < HD) {
      float gm = -INFINITY;
      for (int q = 0; q < S; ++q) gm = fmaxf(gm, sl_m[q]);
      float oo = 0.f, ll = 0.f;
      for (int q = 0; q < S; ++q) {
        const float v = expf(sl_m[q] - gm);
        oo = fmaf(v, sm_o[q * HD + t2], oo);
        ll = fmaf(v, sl_l[q], ll);
      }
      st_agent(att + (size_t)hh * HD + t2, oo / ll);
    }
    // (written back before anything this workgroup publishes later, and so before the next layer's partials)
    for (int c = sl; c < nchunk; c += S) {
      float* const pc = pb + (size_t)c * (HD + 2);
      st_agent(pc + i, __uint_as_float(FU_EMPTY));
      if (i == 0) { st_agent(pc + HD, __uint_as_float(FU_EMPTY)); st_agent(pc + HD + 1, __uint_as_float(FU_EMPTY)); }
    }
    fu_landed();
    fu_bar();
  }
  fu_bar();
}

template <int HD, bool NARROW>
__global__ __launch_bounds__(FU_THREADS) void decode_layers_kernel(FusedArgs args) {
  FWg w;
  w.a = (FArgs)__builtin_amdgcn_kernarg_segment_ptr();
  w.tab = (FTab)(uintptr_t)w.a->L;
  w.tid = threadIdx.x; w.lane = w.tid & 63;
  w.wave = __builtin_amdgcn_readfirstlane(w.tid >> 6);
  w.idx = blockIdx.x; w.G = gridDim.x;
  w.pos = __builtin_amdgcn_readfirstlane(w.a->ds->pos);
  w.nchunk = w.pos / ATT_CHUNK + 1; w.ncp = (w.nchunk + 1) / 2;
  // a contiguous run of items per workgroup, among those that have a tile of the output projection or of FFN in (all
  // others read those outputs before the next layer's attention, and so know the partials merged there empty again)
  const int items = w.a->H * w.ncp, most = w.a->ph[2].NT > w.a->ph[1].NT ? w.a->ph[2].NT : w.a->ph[1].NT;
  const int Ga = most < w.G ? most : w.G, ia = w.idx < Ga ? w.idx : Ga, ib = w.idx + 1 < Ga ? w.idx + 1 : Ga;
  w.it0 = items * ia / Ga; w.it1 = items * ib / Ga;
  const int nsteps = w.a->nsteps, layer0 = w.a->layer0;
  if (w.tid < MG_WAVES) ((uint32_t*)(w.lds() + FU_LDS_DONE))[w.tid] = 0;
  fu_bar();

  if (w.wave >= MG_WAVES) {
    __builtin_amdgcn_s_setprio(3);
    FHelper hp;
    hp.wave = w.wave - MG_WAVES; hp.tiles = 0; hp.wait.dead = false;
    for (int ord = hp.wave; ord < w.my_tiles(1); ord += FU_HELPERS) {     // the residuals of this workgroup's outputs
      const int n = (w.idx + ord * w.G) * 16 + w.lane;
      if (w.lane < 16 && n < w.a->d_model) ((float*)(w.lds() + w.a->off_res))[ord * 16 + w.lane] = w.a->h[n];
    }
    fu_gain(w, hp, 0, layer0);
    for (int n = 0; n < 4 * nsteps; ++n) {
      const int i = n & 3, step = n >> 2, norm = w.a->ph[i].norm;
      fu_row(w, hp, i, step);
      fu_landed();
      fu_bar();                            // the row is in LDS
      if (norm == 0) { fu_bar(); fu_bar(); }
      if (norm >= 0) fu_bar();             // ... as two terms
      // the next norm's gain and bias while this product runs
      if ((i & 1) && n + 1 < 4 * nsteps) fu_gain(w, hp, (i + 1) & 3, layer0 + step + (i >> 1));
      fu_outputs(w, hp, i, step, n + 1 == 4 * nsteps);
      if (i == 0) fu_help_attention<HD>(w, hp, step);
    }
    return;
  }
  const unsigned lane16 = w.lane * 16;
  u32x4 ring[FU_RING][MG_BATCH];
  uint32_t tiles = 0;
  FWait wait; wait.dead = false;
  {
    const FSeg s = fu_seg(w, 0, layer0);
#pragma unroll
    for (int r = 0; r < FU_RING; ++r) FU_AHEAD(r, fu_ahead(s, r));
  }
  for (int n = 0; n < 4 * nsteps; ++n) {
    const int i = n & 3, layer = layer0 + (n >> 2);
    const bool end = n + 1 == 4 * nsteps;
    const FSeg s = fu_seg(w, i, layer);
    FSeg nx = fu_seg(w, (i + 1) & 3, i == 3 && !end ? layer + 1 : layer);
    if (end) nx.Q = 0;
    fu_product<HD, NARROW>(w, ring, tiles, i, s, nx, layer);
    if (i == 0) {
      fu_attention<HD>(w, ring, wait, n >> 2, layer);
#pragma unroll
      for (int r = FU_KV; r < FU_RING; ++r) FU_AHEAD(r, fu_ahead(nx, r));
    }
  }
}
#endif

// launcher (ppd_fused.hip); grid: one workgroup per compute unit
hipError_t launch_fused(hipStream_t stream, const FusedArgs& a, int head_dim, bool narrow, int grid, int lds);
hipError_t fused_setup(int head_dim, bool narrow, int lds);

}  // namespace ppd
