// Compute-bound prompt pass for bf16 models (gfx950).
//
// The method starts from a start token x_0 (Algorithm 1 / 2); a prompt is run through all d layers first to fill
// the key/value cache.  The decode kernels stream every weight once per 16 rows, which is the right shape for a
// handful of rows and the wrong one for a prompt: here the prompt's rows are a real matrix operand.
//
//   pack_rows_kernel    rows (after an optional norm) -> two bf16 terms x = hi + lo in MFMA operand blocks
//   pgemm_kernel        Y = epilogue(X W^T): tiled v_mfma_f32_32x32x16_bf16, weights in the repacked 1 KiB blocks of the
//                       decode path (A operand), packed rows as B operand, both through LDS (every request is one
//                       contiguous kilobyte); products exact in fp32 as in decoding
//   pkv_pack_kernel     queries, keys, values of the prompt rows -> two-term operand blocks, and keys and values into
//                       the fp32 cache in the decode path's layout
//   rgemm_kernel, sgemm_kernel   the GEMMs of a prompt chunk of up to 32 rows, in the decode path's summation order
//   pattn_kernel        causal attention of all prompt rows on the same MFMA (three products per pair of two-term
//                       operands), key/value steps staged through LDS for the four waves of a workgroup, running softmax
//
// Rounding order differs from the decode kernels (other tiles, other summation trees), so a cache filled here is
// close to, not bit-identical with, one filled row by row; every decode step after it is the same arithmetic
// whichever way the cache was filled, so PPD == plain greedy bit for bit still holds.
#pragma once
#include "ppd_kernels.h"

namespace ppd {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---- rows -> packed two-term operand blocks
// Block (mt, kt) holds rows 16 mt .. +15, columns 32 kt .. +31 as 64 lanes x 8 bf16: lane i + 16 c = row i, columns
// 8 c .. 8 c + 7 (the B operand of v_mfma_f32_16x16x32_bf16).  Plane 0: hi = bf16(x); plane 1: lo = bf16(x - hi).
// Rows past M and columns past K are zeros.
struct PackArgs {
  const float* X; int ld;        // [M][ld]
  int M, K, KT, MT;              // KT = ceil(K / 32), MT = ceil(M / 16)
  const void* g; const void* b;  // bf16 gain / bias of the norm (norm >= 0)
  int norm;                      // -1 none, 0 LayerNorm, 1 RMSNorm
  float eps;
  uint16_t* out;                 // [2][MT][KT][64][8]
  // S != null: the rows are still to be added up: X (which takes them) + bias + the eight partial sums that sgemm_kernel left
  const float* S; const void* bias;   // [8][M][K]; bias or null
};

__device__ __forceinline__ void split2(const float (&xv)[8], uint4& hi, uint4& lo) {
  uint32_t hp[4], lp[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    hp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){xv[2 * e], xv[2 * e + 1]}, bf16x2));
    const float r0 = xv[2 * e] - __uint_as_float(hp[e] << 16), r1 = xv[2 * e + 1] - __uint_as_float(hp[e] & 0xffff0000u);
    lp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){r0, r1}, bf16x2));
  }
  hi = make_uint4(hp[0], hp[1], hp[2], hp[3]);
  lo = make_uint4(lp[0], lp[1], lp[2], lp[3]);
}

#ifdef PPD_PREFILL_TU
// One workgroup per row (rows up to 16 MT: the padding rows write zeros).  A 64-byte line of the output holds four rows, so
// the 16 rows of a block go to one XCD (workgroups are handed to the eight of them in turn) and its L2 puts the lines
// together; spread over all, every quarter of a line was written to memory by itself: 4095 rows of 5120, 86 -> 43 us.
// The norm is the decode path's: thread t
// sums the 8-element pieces t, t + 512, ...; butterfly inside each wave; the eight wave sums in index order.
__global__ __launch_bounds__(MG_THREADS) void pack_rows_kernel(PackArgs a) {
  __shared__ float redA[MG_WAVES], redB[MG_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, K = a.K;
  const int mt = ((int)blockIdx.x >> 7) * 8 + ((int)blockIdx.x & 7), i = ((int)blockIdx.x >> 3) & 15, m = mt * 16 + i;
  if (mt >= a.MT) return;
  const size_t plane = (size_t)a.MT * a.KT * 512;        // bf16 elements per plane
  const float* x = a.X + (size_t)m * a.ld;
  const bool live = m < a.M;
  if (a.S && live) {
    // (a thread finds what it writes here: its own pieces)
    float* const xw = (float*)x;
    const size_t share = (size_t)a.M * K;
    for (int c = tid; c * 8 < K; c += MG_THREADS) {
      float4 v[MG_WAVES][2], r[2];
      const float* s = a.S + (size_t)m * K + c * 8;
#pragma unroll
      for (int w = 0; w < MG_WAVES; ++w) { v[w][0] = *(const float4*)(s + w * share); v[w][1] = *(const float4*)(s + w * share + 4); }
      r[0] = ((const float4*)(xw + c * 8))[0]; r[1] = ((const float4*)(xw + c * 8))[1];
      u32x4 bq = {0u, 0u, 0u, 0u};
      if (a.bias) bq = *(const u32x4*)((const char*)a.bias + (size_t)c * 16);
      float bf[8]; WTr<bf16_t>::unpack(bq, bf);
      // the order of the decode step's epilogue: the shares in turn, the bias, the residual
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float4 y = v[0][h];
#pragma unroll
        for (int w = 1; w < MG_WAVES; ++w) { y.x += v[w][h].x; y.y += v[w][h].y; y.z += v[w][h].z; y.w += v[w][h].w; }
        y.x = (y.x + bf[4 * h]) + r[h].x; y.y = (y.y + bf[4 * h + 1]) + r[h].y; y.z = (y.z + bf[4 * h + 2]) + r[h].z; y.w = (y.w + bf[4 * h + 3]) + r[h].w;
        ((float4*)(xw + c * 8))[h] = y;
      }
    }
  }
  auto combine8 = [&](const float* r) { return ((((((r[0] + r[1]) + r[2]) + r[3]) + r[4]) + r[5]) + r[6]) + r[7]; };
  float mu = 0.f, rs = 1.f;
  if (a.norm >= 0 && live) {
    if (a.norm == 0) {
      float sm = 0.f;
      for (int c = tid; c * 8 < K; c += MG_THREADS) {
        const float4* px = (const float4*)(x + c * 8);
        const float4 v = px[0], w = px[1];
        sm += v.x; sm += v.y; sm += v.z; sm += v.w; sm += w.x; sm += w.y; sm += w.z; sm += w.w;
      }
      sm = wave_sum(sm);
      if (lane == 0) redA[wave] = sm;
      __syncthreads();
      mu = combine8(redA) / (float)K;
    }
    float s2 = 0.f;
    for (int c = tid; c * 8 < K; c += MG_THREADS) {
      const float4* px = (const float4*)(x + c * 8);
      const float4 v = px[0], w = px[1];
      const float d[8] = {v.x - mu, v.y - mu, v.z - mu, v.w - mu, w.x - mu, w.y - mu, w.z - mu, w.w - mu};
#pragma unroll
      for (int e = 0; e < 8; ++e) s2 = fmaf(d[e], d[e], s2);
    }
    s2 = wave_sum(s2);
    if (lane == 0) redB[wave] = s2;
    __syncthreads();
    rs = 1.0f / sqrtf(combine8(redB) / (float)K + a.eps);
  }
  for (int c = tid; c < a.KT * 4; c += MG_THREADS) {     // 8-element pieces of the padded row
    float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (live && c * 8 < K) {
      const float4* px = (const float4*)(x + c * 8);
      const float4 v = px[0], w = px[1];
      xv[0] = v.x; xv[1] = v.y; xv[2] = v.z; xv[3] = v.w; xv[4] = w.x; xv[5] = w.y; xv[6] = w.z; xv[7] = w.w;
      if (a.norm >= 0) {
        const u32x4 gq = *(const u32x4*)((const char*)a.g + (size_t)c * 16);
        float gf[8]; WTr<bf16_t>::unpack(gq, gf);
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] = (xv[e] - mu) * rs * gf[e];
        if (a.norm == 0 && a.b) {
          const u32x4 bq = *(const u32x4*)((const char*)a.b + (size_t)c * 16);
          float bf[8]; WTr<bf16_t>::unpack(bq, bf);
#pragma unroll
          for (int e = 0; e < 8; ++e) xv[e] += bf[e];
        }
      }
    }
    uint4 hi, lo;
    split2(xv, hi, lo);
    const size_t o = (((size_t)mt * a.KT + (c >> 2)) * 64 + i + 16 * (c & 3)) * 8;
    *(uint4*)(a.out + o) = hi;
    *(uint4*)(a.out + plane + o) = lo;
  }
}
#endif

// ---- tiled GEMM
// How a product is cut: tile shape (index into pg_tiles) and number of parts of the reduction length
struct PGemmPlan { int tile, S; float us; };     // us: the time by plan_pgemm's account
constexpr int PG_TILES = 7;
struct PGemmArgs {
  const uint16_t* Xp;   // packed rows [2][MT][KT][64][8]
  const void* P;        // repacked weights [NT][KT][64][8]
  const void* B[3];     // biases per row segment or null (paired: B[0] gate, B[1] up)
  const float* Rsd;     // residual rows [M][ldy] or null
  float* Y;             // [M][ldy]
  int M, MT, KT, NT;
  int N[3], ntot;       // rows per segment (bias lookup); logical output rows
  int ldy;
  int act;              // 0 none, 1 GELU, 2 ReLU (paired launches apply SwiGLU)
  int NB, MB;           // tiles along the outputs and along the rows (launch_pgemm fills these and S)
  int S;                // parts of the reduction length, each a workgroup's
  float* ws; int* cnt;  // S > 1: partial sums [tile][part], parts that are done per tile (zero between launches)
  // the outputs in packed two-term form instead of Y (they are the next GEMM's rows: the feed-forward activations):
  // [2][MT][KTp][64][8]; only outputs below ntot are written, the padding columns of the buffer stay as they are (zero)
  uint16_t* Yp; int KTp;
};
constexpr size_t PG_WS_BYTES = (size_t)32 << 20;     // of partial sums at most
constexpr int PG_MAX_TILES = 1024;                   // tiles of a product whose reduction length is cut

// four consecutive outputs n0 .. n0 + 3 (n0 a multiple of 4) of row m into the packed form: half of an 8-column piece
__device__ __forceinline__ void put_packed4(uint16_t* out, size_t plane_elems, int KT, int m, int n0, const float (&y)[4]) {
  uint32_t hp[2], lp[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    hp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){y[2 * e], y[2 * e + 1]}, bf16x2));
    const float r0 = y[2 * e] - __uint_as_float(hp[e] << 16), r1 = y[2 * e + 1] - __uint_as_float(hp[e] & 0xffff0000u);
    lp[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){r0, r1}, bf16x2));
  }
  const int c8 = n0 >> 3;
  const size_t o = (((size_t)(m >> 4) * KT + (c8 >> 2)) * 64 + (m & 15) + 16 * (c8 & 3)) * 8 + ((n0 >> 2) & 1) * 4;
  *(uint2*)(out + o) = make_uint2(hp[0], hp[1]);
  *(uint2*)(out + plane_elems + o) = make_uint2(lp[0], lp[1]);
}


#ifdef PPD_PREFILL_TU
// 64 lanes x 16 bytes from sbase + voff (per lane) to LDS offset ldsoff + 16 * lane; see dma16
__device__ __forceinline__ void dma16s(unsigned voff, const void* sbase, unsigned ldsoff) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(ldsoff) : "memory", "m0");
}

// A workgroup makes a tile of WW TW x WX TX blocks of 32 x 32 outputs (weight rows x prompt rows), each of its WW x WX waves
// TW x TX of them.  Weights and both terms of the rows come through LDS, 32 columns a stage, in a ring of R stages filled by
// direct loads; a wave reads TW + 2 TX kilobytes for 2 TW TX MFMAs.  What bounds it: the MFMA pipes at the clock that the
// card's power allows under them, about 1.9 GHz on random data, so every byte moved less per MFMA shows twice.  The kernel
// before this one (weights from L2 into every wave's registers, 64 prompt rows a workgroup) moved three times the bytes
// through L2 per MFMA.  Measured (before -> now, PFLOP/s with both terms counted): 13B shape, 4095 rows, in the model: QKV 1.14
// -> 1.38, O 1.02 -> 1.25, FFN in 1.17 -> 1.42, FFN out 1.05 -> 1.38; 7B shape, 511 rows: QKV 0.87 -> 1.02, FFN in 1.08 -> 1.20,
// O and FFN out 0.76 and 0.93, as before; back to back, 128 rows of it 250 -> 156 us a layer, 40 rows 209 -> 115 us.
// Order of a stage: while the first 16 columns are multiplied the second ones' operands are read, and while those are
// multiplied the next stage's first ones; between the halves the one barrier of a stage, behind which the stage's slot takes
// requests again.  Requests and reads stand between the MFMAs, whose issue they do not hold up.
// The MFMA is v_mfma_f32_32x32x16_bf16: its operands come out of the 16-row blocks as they lie in memory: lane r + 32 h of a
// 32-row tile reads 16 bytes of the 16-row block r / 16 at lane position (r % 16) + 16 (2 w + h), w = 0, 1 being the two
// 16-column halves of the 32-column block, so one block pair feeds two MFMAs per operand pair, and weights and rows pair up
// column by column whatever order the hardware takes the 16 columns in.
// Tiles are dealt to the XCDs (workgroup b of a launch runs on XCD b % 8) in runs of equal length, in an order in which
// neighbours share panels: 4 tiles of outputs by all rows.  Dealing out whole columns of tiles left XCDs idle: 20 columns
// (13B shape, O and FFN out) on 8 XCDs take as long as 24.
// S > 1: few tiles, so the reduction length is cut into S parts to fill the machine.  A workgroup leaves its sums in memory,
// past its L2 (agent scope), and counts itself; the last of a tile to do so adds the parts in their order and goes on to the
// epilogue.  7B shape, 40 rows, FFN out: 90 us with S = 1, 29 with 6.
template <bool PAIRED, int WW, int WX, int TW, int TX, int R>
__global__ __launch_bounds__(WW * WX * WAVE, WW * WX <= 4 ? 1 : 2) void pgemm_kernel(PGemmArgs a) {
  constexpr int NW = WW * WX;
  constexpr int BW = 2 * WW * TW, BX = 2 * WX * TX;        // 16-row blocks of a tile: weights, rows
  constexpr int NBLK = BW + 2 * BX;                        // KiB per stage: weights, first terms, second terms
  constexpr int ND = (NBLK + NW - 1) / NW;                 // requests of a wave per stage (the last ones may repeat a block)
  static_assert((R - 1) * ND < 64, "the waits count requests in flight");
  extern __shared__ float4 pg_lds4[];
  char* const lds = (char*)pg_lds4;                        // [R][NBLK] KiB
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ww = wave % WW, wx = wave / WW;
  // this workgroup's part and tile
  constexpr int GQ = 4;
  const int T = a.NB * a.MB, U = T * a.S, xcd = blockIdx.x & 7, r = blockIdx.x >> 3, each = U >> 3, more = U & 7;
  if (r >= each + (xcd < more ? 1 : 0)) return;
  const int u = xcd * each + (xcd < more ? xcd : more) + r, sp = u / T, t = u - sp * T;
  const int g = t / (GQ * a.MB), gi = t - g * GQ * a.MB, gw = a.NB - g * GQ < GQ ? a.NB - g * GQ : GQ;
  const int mb = gi / gw, nb = g * GQ + gi - mb * gw;
  const int KT = a.KT, k0 = KT * sp / a.S, nst = KT * (sp + 1) / a.S - k0;
  const int ntb = nb * BW, mtb = mb * BX;                  // in 16-row blocks
  const size_t plane = (size_t)a.MT * KT * 1024;           // bytes per plane of the packed rows
  const unsigned voff = lane * 16;
  const char* src[ND];                                     // (blocks past the matrix or the prompt repeat its last one; never stored)
  auto blk_of = [&](int j) { return wave + j * NW < NBLK ? wave + j * NW : NBLK - 1; };
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    const int blk = blk_of(j);
    if (blk < BW) {
      const int nt = ntb + blk < a.NT ? ntb + blk : a.NT - 1;
      src[j] = (const char*)a.P + ((size_t)nt * KT + k0) * 1024;
    } else {
      const int x = blk - BW, pl = x / BX, m = mtb + x - pl * BX, mt = m < a.MT ? m : a.MT - 1;
      src[j] = (const char*)a.Xp + pl * plane + ((size_t)mt * KT + k0) * 1024;
    }
  }
  auto request = [&](int j, int s) {                       // (stages past the end repeat the last one; unused)
    dma16s(voff, src[j] + (size_t)(s < nst ? s : nst - 1) * 1024, lds0 + (unsigned)((s % R) * NBLK + blk_of(j)) * 1024u);
  };
  const int lr = lane & 31, lh = lane >> 5;
  const int lane_off = (lr >> 4) * 1024 + ((lr & 15) + 16 * lh) * 16;      // + 512 for the second 16 columns
  const char* const wl = lds + ww * TW * 2048 + lane_off;
  const char* const xl = lds + (BW + wx * TX * 2) * 1024 + lane_off;
  f32x16 acc[TW][TX];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TX; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  // operands of 16 columns: weights, first and second terms of the rows; one set is multiplied while the other is read
  u32x4 fw[2][TW], fh[2][TX], fl[2][TX];
  constexpr int NF = TW + 2 * TX, NM = TW * TX * 2;
  auto read = [&](int w, int f, int so) {
    if (f < TW) fw[w][f] = *(const u32x4*)(wl + so + f * 2048 + 512 * w);
    else if (f < TW + TX) fh[w][f - TW] = *(const u32x4*)(xl + so + (f - TW) * 2048 + 512 * w);
    else fl[w][f - TW - TX] = *(const u32x4*)(xl + so + (BX + 2 * (f - TW - TX)) * 1024 + 512 * w);
  };
  auto mac = [&](int w, int m) {
    const int i = m / (2 * TX), x = m % (2 * TX), j = x % TX;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fw[w][i]), __builtin_bit_cast(bf16x8, x < TX ? fh[w][j] : fl[w][j]), acc[i][j], 0, 0, 0);
  };
  // what the epilogue adds: registers 4 q .. 4 q + 3 of a 32 x 32 block are its rows 8 q + 4 (l / 32) .. + 3 (weight rows) for
  // column l % 32 (prompt row); ntot, ldy and the segments' rows are multiples of 4.  Small tiles, a latency's work, ask for it
  // before their operands; the others behind the loop, a column of blocks ahead (their registers are taken until then).  The residuals of
  // the next column are requested before this one's outputs are stored: they may be the same memory, and a load does not pass a store.
  // Behind the loop, one bias at a time, it took as long as the product of a narrow model: OPT-125m shape, 127 rows, us before / now: QKV
  // 11.1 / 8.3, O 10.5 / 8.2, FFN in 10.4 / 8.3, FFN out 13.0 / 11.2; 500 rows 15.8 / 12.5, 10.9 / 8.2, 15.6 / 13.1, 16.9 / 14.4.
  const int nt0 = ntb + ww * TW * 2, mt0 = mtb + wx * TX * 2;
  const uint16_t* const B0 = (const uint16_t*)a.B[0];
  const uint16_t* const B1 = (const uint16_t*)a.B[1];
  const uint16_t* const B2 = (const uint16_t*)a.B[2];
  constexpr bool EARLY = TW * TX <= 2;
  constexpr int NR = EARLY ? TW : 2;
  f32x4 rsd[PAIRED ? 1 : NR][TX][4];
  uint2 bias[PAIRED ? 1 : NR][4];              // (registers: of the next column only where they are enough)
  constexpr bool AHEAD = EARLY || TW * TX < 10;
  auto biases = [&](int i) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int n0 = (nt0 + 2 * i) * 16 + 8 * q4 + 4 * (lane >> 5);
      bias[i % NR][q4] = make_uint2(0u, 0u);
      if (B0 && n0 < a.ntot) {
        int loc = n0; const uint16_t* b = B0;
        if (loc >= a.N[0]) { loc -= a.N[0]; b = B1; if (loc >= a.N[1]) { loc -= a.N[1]; b = B2; } }
        bias[i % NR][q4] = *(const uint2*)(b + loc);
      }
    }
  };
  auto residuals = [&](int i) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
      for (int j = 0; j < TX; ++j) {
        const int m = (mt0 + 2 * j) * 16 + (lane & 31), n0 = (nt0 + 2 * i) * 16 + 8 * q4 + 4 * (lane >> 5);
        rsd[i % NR][j][q4] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (a.Rsd && m < a.M && n0 < a.ntot) rsd[i % NR][j][q4] = *(const f32x4*)(a.Rsd + (size_t)m * a.ldy + n0);
      }
  };
  if constexpr (!PAIRED && EARLY)
#pragma unroll
    for (int i = 0; i < TW; ++i) { biases(i); residuals(i); }
#pragma unroll
  for (int s = 0; s < R; ++s)
#pragma unroll
    for (int j = 0; j < ND; ++j) request(j, s);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((R - 1) * ND) : "memory");
#pragma unroll
  for (int f = 0; f < NF; ++f) read(0, f, 0);
  int so = 0;                                              // the stage's place in the ring
  for (int s = 0; s < nst; ++s) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mac(0, m);
#pragma unroll
      for (int f = 0; f < NF; ++f) if (f * NM / NF == m) read(1, f, so);
      __builtin_amdgcn_sched_barrier(0);
    }
    // stage s + 1 is in LDS for everybody, and everybody has read stage s
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((R - 2) * ND) : "memory");
    so += NBLK * 1024;
    if (so == R * NBLK * 1024) so = 0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mac(1, m);
#pragma unroll
      for (int f = 0; f < NF; ++f) if (f * NM / NF == m) read(0, f, so);
#pragma unroll
      for (int j = 0; j < ND; ++j) if (j * NM / ND == m) request(j, s + R);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (no request outlives the workgroup)

  if (a.S > 1) {
    constexpr unsigned TILE = NW * TW * TX * 4096;         // bytes of a tile's sums: [wave][32 x 32 block][4][64 lanes][4]
    constexpr int AGENT = 16;                              // sc1: past this XCD's L2
    const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc((char*)a.ws + (size_t)t * a.S * TILE, 0, (int)(a.S * TILE), 0x00020000);
    const unsigned o0 = (unsigned)wave * (TW * TX * 4096u) + lane * 16u;
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int j = 0; j < TX; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const f32x4 y = {acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]};
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), ws, o0 + ((i * TX + j) * 4 + v) * 1024u, sp * TILE, AGENT);
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's sums are where every XCD finds them
    __syncthreads();                                       // everybody's are (and everybody is done with the ring)
    int* const done = (int*)lds;
    if (tid == 0) {
      const int n = __hip_atomic_fetch_add(a.cnt + t, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (n == a.S - 1) __hip_atomic_store(a.cnt + t, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *done = n;
    }
    __syncthreads();
    if (*done != a.S - 1) return;
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int j = 0; j < TX; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    for (int p = 0; p < a.S; ++p)
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int j = 0; j < TX; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const f32x4 y = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ws, o0 + ((i * TX + j) * 4 + v) * 1024u, p * TILE, AGENT));
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][4 * v + e] += y[e];
          }
  }

  // ---- epilogue
  if constexpr (!PAIRED && !EARLY) { residuals(0); if constexpr (AHEAD) biases(0); }
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    if constexpr (!PAIRED && !EARLY) {
      if (i + 1 < TW) residuals(i + 1);
      if constexpr (!AHEAD) biases(i);
      else if (i + 1 < TW) biases(i + 1);
    }
#pragma unroll
    for (int j = 0; j < TX; ++j) {
      const int m = (mt0 + 2 * j) * 16 + lr;
      if (m >= a.M) continue;
      auto put = [&](int n0, const float (&y)[4]) {
        if (a.Yp) put_packed4(a.Yp, (size_t)a.MT * a.KTp * 512, a.KTp, m, n0, y);
        else *(float4*)(a.Y + (size_t)m * a.ldy + n0) = make_float4(y[0], y[1], y[2], y[3]);
      };
      if constexpr (PAIRED) {
        // a 16-row block holds the gate rows (0..7) and the up rows (8..15) of 8 outputs: register groups 0, 1 are
        // gate and up of the first block's outputs 4 (l / 32) .. + 3, groups 2, 3 of the second block's
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          const int n0 = (nt0 + 2 * i + hb) * 8 + 4 * lh;
          if (n0 >= a.ntot) continue;
          float y[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float bg = B0 ? bf16_to_f32(B0[n0 + q]) : 0.f, bu = B1 ? bf16_to_f32(B1[n0 + q]) : 0.f;
            y[q] = silu(acc[i][j][8 * hb + q] + bg) * (acc[i][j][8 * hb + 4 + q] + bu);
          }
          put(n0, y);
        }
      } else {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int n0 = (nt0 + 2 * i) * 16 + 8 * q4 + 4 * lh;
          if (n0 >= a.ntot) continue;
          float y[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t bw = q < 2 ? bias[i % NR][q4].x : bias[i % NR][q4].y;
            const float bv = __uint_as_float(q & 1 ? bw & 0xffff0000u : bw << 16);
            float tv = acc[i][j][4 * q4 + q] + bv;
            if (a.act == 1) tv = gelu_erf(tv);
            else if (a.act == 2) tv = fmaxf(tv, 0.f);
            if (a.Rsd) tv += rsd[i % NR][j][q4][q];
            y[q] = tv;
          }
          put(n0, y);
        }
      }
    }
  }
}
#endif

// ---- a prompt chunk of up to 32 rows: one pass over the weights, bound by their stream
// The arithmetic is gemm_mfma_kernel's (wave w of 8 owns one eighth of the reduction length; first terms, then second
// terms of a block; the eight partial sums in wave order), so a row's bits are those of a one-row pass.  The rows come as
// packed two-term operands straight from L2 instead of being staged and converted in LDS by every workgroup: 16 rows
// of fp32 do not fit LDS whole, and the staging passes took most of the time (7B shape, 16 rows: 30 us of staging in a
// 45 us FFN-in launch).  Every block of rows feeds TT weight tiles, so that L2 hands out (1 + 2 MT / TT) kilobytes per
// kilobyte of weights.  Measured (7B shape, 26 rows, all layers): two 16-row chunks through gemm_mfma_kernel 9.0 ms,
// one chunk through this kernel 4.3 ms (attention and its row split included); per layer QKV 24 us, FFN-in 37.  What is left
// over the weights' stream is the L2 traffic: six tiles at once instead of twice three took FFN-in from 42 to 37 us.
// (O and FFN-out are sgemm_kernel's.)
struct RGemmArgs {
  const uint16_t* Xp;   // packed rows [2 planes][2][KT][64][8] (always two 16-row tiles; see PackArgs)
  const void* P;        // repacked weights [NT][KT][64][8]
  const void* B[3];     // biases per row segment or null (paired: B[0] gate, B[1] up)
  float* Y;             // [M][ldy], or
  uint16_t* Yp; int KTp;   // the outputs as packed rows [2][2][KTp][64][8]
  int M, KT, NT, N[3], ntot, ldy;
  int act;              // 0 none, 1 GELU, 2 ReLU (paired launches apply SwiGLU)
  int tiles_wg; unsigned wbytes;
};
constexpr int RG_TILES_MAX = 8;      // tiles of a workgroup whose partial sums fit LDS (16 KiB each for 32 rows)

#ifdef PPD_PREFILL_TU
template <bool PAIRED, int TT, int MT>
__global__ __launch_bounds__(MG_THREADS) void rgemm_kernel(RGemmArgs a) {
  constexpr int D = TT >= 6 ? 3 : (TT >= 3 ? 4 : 6);       // reduction steps in flight per wave
  extern __shared__ float4 rg_lds4[];
  float* const part = (float*)rg_lds4;                     // [tile][8 waves][16 MT rows][16 outputs]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grid = gridDim.x, KT = a.KT, M = a.M;
  const int ntiles = (int)blockIdx.x + (a.tiles_wg - 1) * grid < a.NT ? a.tiles_wg : a.tiles_wg - 1;
  const int nb8 = (KT + MG_WAVES - 1) / MG_WAVES;
  const int kb0 = wave * nb8 < KT ? wave * nb8 : KT;
  const int nblk = (kb0 + nb8 < KT ? kb0 + nb8 : KT) - kb0;
  const int ngrp = (ntiles + TT - 1) / TT, Q = ngrp * nblk;
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)a.P, 0, (int)a.wbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)a.Xp, 0, KT * 4096, 0x00020000);
  const unsigned lane16 = lane * 16, plane = KT * 2048u;
  u32x4 wa[D][TT], xh[D][MT], xl[D][MT];
  int l_g = 0, l_s = 0;
  // every step is requested in full: what lies past the wave's share is asked for past the end of the matrix, and not read
  auto request = [&](int d) {
    const bool live = l_g < ngrp;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int ord = l_g * TT + t;
      const unsigned o = live && ord < ntiles ? (unsigned)(((int)blockIdx.x + ord * grid) * KT + kb0 + l_s) * 1024u + lane16 : a.wbytes;
      wa[d][t] = __builtin_amdgcn_raw_buffer_load_b128(wres, o, 0, 2);      // 2: non-temporal
    }
    const unsigned xo = (unsigned)(kb0 + l_s) * 1024u + lane16;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      xh[d][m] = __builtin_amdgcn_raw_buffer_load_b128(xres, live ? xo + m * KT * 1024u : KT * 4096u, 0, 0);
      xl[d][m] = __builtin_amdgcn_raw_buffer_load_b128(xres, live ? xo + m * KT * 1024u + plane : KT * 4096u, 0, 0);
    }
    if (++l_s >= nblk) { l_s = 0; ++l_g; }
  };
  f32x4 acc[TT][MT];
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[t][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
  int c_g = 0, c_s = 0;
  auto put = [&]() {                                       // this wave's partial sums of a group of tiles
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int ord = c_g * TT + t;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (ord < ntiles) *(f32x4*)(part + (((size_t)ord * MG_WAVES + wave) * (16 * MT) + 16 * m + (lane & 15)) * 16 + 4 * (lane >> 4)) = acc[t][m];
        acc[t][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  auto consume = [&](int d) {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[d][t]), __builtin_bit_cast(bf16x8, xh[d][m]), acc[t][m], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[d][t]), __builtin_bit_cast(bf16x8, xl[d][m]), acc[t][m], 0, 0, 0);
    if (++c_s == nblk) { put(); c_s = 0; ++c_g; }
  };
  if (nblk > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) request(d);
    for (int q = 0; q < Q; q += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (q + d < Q) consume(d);
        request(d);
      }
    }
  } else {
    for (; c_g < ngrp; ++c_g) put();                       // a wave without a share adds zeros
  }
  __syncthreads();
  // the eight partials of an output in wave order, bias, activation
  constexpr int R = PAIRED ? 8 : 16;
  const uint16_t* const B0 = (const uint16_t*)a.B[0];
  const uint16_t* const B1 = (const uint16_t*)a.B[1];
  const uint16_t* const B2 = (const uint16_t*)a.B[2];
  for (int e = tid; e < ntiles * M * R; e += MG_THREADS) {
    const int row = e & (R - 1), f = e / R, ord = f / M, m = f - ord * M, n = ((int)blockIdx.x + ord * grid) * R + row;
    if (n >= a.ntot) continue;
    const float* pp = part + ((size_t)ord * MG_WAVES * (16 * MT) + m) * 16 + row;
    constexpr int ws = 16 * MT * 16;
    float s = pp[0];
#pragma unroll
    for (int w = 1; w < MG_WAVES; ++w) s += pp[w * ws];
    float y;
    if (PAIRED) {
      float u = pp[8];
#pragma unroll
      for (int w = 1; w < MG_WAVES; ++w) u += pp[w * ws + 8];
      y = silu(s + (B0 ? bf16_to_f32(B0[n]) : 0.f)) * (u + (B1 ? bf16_to_f32(B1[n]) : 0.f));
    } else {
      float b = 0.f;
      if (B0) {
        int seg = 0, loc = n;
        if (loc >= a.N[0]) { loc -= a.N[0]; seg = 1; if (loc >= a.N[1]) { loc -= a.N[1]; seg = 2; } }
        b = bf16_to_f32((seg == 0 ? B0 : (seg == 1 ? B1 : B2))[loc]);
      }
      y = s + b;
      if (a.act == 1) y = gelu_erf(y);
      else if (a.act == 2) y = fmaxf(y, 0.f);
    }
    y += 0.f;      // (where the decode step adds the residual: -0 becomes 0)
    if (a.Yp) put_packed1(a.Yp, (size_t)2 * a.KTp * 512, a.KTp, m, n, y);
    else a.Y[(size_t)m * a.ldy + n] = y;
  }
}
#endif

// ---- the products of such a chunk whose outputs are few: one share of the reduction length per workgroup
// Workgroup (share, group): its waves take a 16-row weight tile each of the group, over the share of the reduction length that a wave
// of rgemm_kernel has, so that the rows' blocks of the share come into LDS once for all of them; the eight shares' sums go to memory and
// pack_rows_kernel, which reads the rows next, adds them in their order.  Block b of a launch is share b % 8: an XCD's workgroups read the same rows.
// The rows come in phases of SG_PB blocks, two buffers.
// What bounds it: what a compute unit can request at a time; the rows of 32 are still a third of its bytes (rgemm_kernel, with one tile to
// a workgroup, read four bytes of rows for one of weights).  7B shape, 27 rows: O 15.5 -> 9.2 us, FFN-out 33.7 -> 22, the sums in pack_rows_kernel
// 5.0 -> 6.2 (two of them).  A prompt of 27 tokens and its first token, 8 layers, rgemm_kernel / this, us: 7B shape 1179 / 1073 (9 tokens 1003 / 972), 13B 1656 /
// 1497 (1410 / 1347), 8192 wide, 2 layers, 874 / 840, 3072 wide 878 / 796, 2048 689 / 610, 1024 495 / 438, OPT-125m shape (12 layers) 675 / 570.  Eight blocks ahead and phases
// of 16 the same within 1 % but for the 13B shape, 1542: its 320 workgroups fit two to a compute unit with the smaller phases.
struct SGemmArgs {
  const uint16_t* Xp;   // packed rows [2 planes][2][KT][64][8]
  const void* P;        // repacked weights [NT][KT][64][8]
  float* S;             // [8][M][ntot]
  int M, KT, NT, ntot;
};
constexpr int SG_RING = 4;           // weight blocks in flight per wave
constexpr int SG_PB = 8;             // blocks of a phase: 32 KiB for 32 rows
static_assert(SG_PB >= SG_RING, "a phase's requests are done when the ring behind them has come round");

#ifdef PPD_PREFILL_TU
template <int MT>
__global__ __launch_bounds__(MG_THREADS) void sgemm_kernel(SGemmArgs a) {
  extern __shared__ float4 sg_lds4[];
  char* const lds = (char*)sg_lds4;                        // [2][SG_PB][2 planes][MT] KiB
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), W = (int)blockDim.x >> 6;
  const int share = blockIdx.x & 7, nt = ((int)blockIdx.x >> 3) * W + wave, KT = a.KT;
  const int nb8 = (KT + MG_WAVES - 1) / MG_WAVES;
  const int kb0 = share * nb8 < KT ? share * nb8 : KT;
  const int nblk = (kb0 + nb8 < KT ? kb0 + nb8 : KT) - kb0;
  const int np = (nblk + SG_PB - 1) / SG_PB;
  auto stage = [&](int p) {
    const int s0 = p * SG_PB, n = (nblk - s0 < SG_PB ? nblk - s0 : SG_PB) * 2 * MT;
    char* const to = lds + (size_t)(p & 1) * SG_PB * 2 * MT * 1024;
    for (int u = wave; u < n; u += W) {
      const int s = u / (2 * MT), v = u - s * 2 * MT, pl = v / MT, m = v - pl * MT;
      dma16((const char*)a.Xp + ((size_t)(pl * 2 + m) * KT + kb0 + s0 + s) * 1024 + lane * 16, to + u * 1024);
    }
  };
  if (np > 0) stage(0);
  // the wave's run of the tile as a buffer of its own: what is asked for past its end is not read (and neither is a tile past the last)
  const __amdgpu_buffer_rsrc_t run = __builtin_amdgcn_make_buffer_rsrc((char*)a.P + ((size_t)(nt < a.NT ? nt : 0) * KT + (nblk ? kb0 : 0)) * 1024, 0,
                                                                        nt < a.NT ? nblk * 1024 : 0, 0x00020000);
  u32x4 ring[SG_RING];
  unsigned o = lane * 16;
  auto request = [&](int i) { ring[i] = __builtin_amdgcn_raw_buffer_load_b128(run, o, 0, 2); o += 1024; };      // 2: non-temporal
#pragma unroll
  for (int i = 0; i < SG_RING; ++i) request(i);
  f32x4 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) acc[m] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < np; ++p) {
    // this phase's rows have arrived: they were requested before the newest SG_RING weight blocks; everybody has read the other buffer
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(SG_RING) : "memory");
    if (p + 1 < np) stage(p + 1);
    const int n = nblk - p * SG_PB < SG_PB ? nblk - p * SG_PB : SG_PB;
    const char* const x = lds + (size_t)(p & 1) * SG_PB * 2 * MT * 1024 + lane * 16;
    auto block = [&](int s, int i) {
      const bf16x8 w = __builtin_bit_cast(bf16x8, ring[i]);
      u32x4 xh[MT], xl[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        xh[m] = *(const u32x4*)(x + (s * 2 * MT + m) * 1024);
        xl[m] = *(const u32x4*)(x + (s * 2 * MT + MT + m) * 1024);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, __builtin_bit_cast(bf16x8, xh[m]), acc[m], 0, 0, 0);
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, __builtin_bit_cast(bf16x8, xl[m]), acc[m], 0, 0, 0);
      request(i);
    };
    int s = 0;
    for (; s + SG_RING <= n; s += SG_RING) {
#pragma unroll
      for (int i = 0; i < SG_RING; ++i) block(s + i, i);
    }
#pragma unroll
    for (int i = 0; i < SG_RING; ++i) if (s + i < n) block(s + i, i);     // (in the last phase only)
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (no request outlives the workgroup)
  const int n0 = nt * 16 + 4 * (lane >> 4);
  if (nt >= a.NT || n0 >= a.ntot) return;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = 16 * m + (lane & 15);
    if (row < a.M) *(float4*)(a.S + ((size_t)share * a.M + row) * a.ntot + n0) = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
  }
}
#endif

// ---- causal attention of the prompt rows
// Row m of the prompt sits at position m (the prompt pass starts from an empty cache) and attends to rows 0 .. m.
// Queries (rotated, scaled), keys (rotated exactly as the cache holds them) and values are first put into two-term
// bf16 operand blocks, so that scores and outputs run on v_mfma_f32_16x16x32_bf16 with the three products
// hi.hi + hi.lo + lo.hi each (the lo.lo term is below 2^-16 of the result) instead of the fp32 MFMA, which
// is a sixteenth as fast:
//   Qp, Kp  [2][H][2 JP][HD / 32][64][8]   block (tile of 16 rows, 32 components): lane i + 16 c = row i, components 8 c .. + 7
//   Vp      [2][H][JP][HD / 16][64][8]     block (32 rows, 16 components): lane i + 16 c = component i, and its 8 values
//                                          are rows 4 c .. 4 c + 3 and 16 + 4 c .. 16 + 4 c + 3 of the 32
// (JP = ceil(M / 32); rows past M are zeros.)  The odd row order of Vp is the one in which a lane holds its scores
// after the two score MFMAs of a 32-row step: lane n + 16 c has, for query n, rows 4 c .. + 3 of either 16-row tile,
// so the probabilities are the B operand of the output MFMA as they stand, without any exchange between lanes.
struct PKvPackArgs {
  const float* qkv;     // [M][3 * d_model]: q | k | v as the projection left them
  const float2* rope;   // [max_ctx][hd / 2] or null
  uint16_t* Qp; uint16_t* Kp; uint16_t* Vp;
  float* Kc; float* Vc; // this layer's fp32 cache (the decode path's blocks): positions 0 .. M - 1 are filled as well
  int M, H, d_model, JP, max_ctx;
  float scale;          // factor on the queries: log2(e) / sqrt(hd), the softmax being evaluated as 2^(s - max)
};
struct PAttnArgs {
  const uint16_t* Qp; const uint16_t* Kp; const uint16_t* Vp;
  uint16_t* outp;       // the outputs in packed two-term form [2][MT][d_model / 32][64][8] (rows of the output projection)
  int M, H, d_model, JP;
  int gx;               // workgroups of a head (launch_pattn fills this)
  // last: row M - 1 is the first round's and attends in fp32 to the cache, as it would in a round
  int last, max_ctx;
  int sp; float* lpart; unsigned* lcnt;    // its workgroups per head (launch_pattn), their partial results [H][PA_SPLIT][HD + 2], those done (zero between launches)
  const float* qkv; const float2* rope; const float* Kc; const float* Vc;
  float scale;
};
constexpr int PA_SPLIT = 16;
// bytes of lpart, with lcnt behind it
inline size_t pattn_last_bytes(int H, int HD) { return (size_t)H * (PA_SPLIT * (HD + 2) + 1) * sizeof(float); }
// bytes of each of Qp, Kp, Vp
inline size_t pattn_stage_bytes(int M, int H, int HD) { return (size_t)2 * H * ((M + 31) / 32) * (HD / 16) * 1024; }

#ifdef PPD_PREFILL_TU
// One workgroup per (32 rows, head).
template <int HD>
__global__ __launch_bounds__(256) void pkv_pack_kernel(PKvPackArgs a) {
  constexpr int half = HD / 2, CB = HD / 32, CT = HD / 16, P8 = HD / 8;
  const int jp = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const size_t plane = (size_t)a.H * a.JP * CT * 512;      // bf16 elements per plane (the same for all three)
  // queries and keys: one 8-component piece of one row per item
  for (int it = tid; it < 32 * P8; it += 256) {
    const int rl = it / P8, c8 = it - rl * P8;             // row of the 32, piece
    const int m = 32 * jp + rl, i0 = 8 * c8;
    float q[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, k[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (m < a.M) {
      const float* r = a.qkv + (size_t)m * 3 * a.d_model + (size_t)h * HD;
      const float4 qa = *(const float4*)(r + i0), qb = *(const float4*)(r + i0 + 4);
      const float4 ka = *(const float4*)(r + a.d_model + i0), kb = *(const float4*)(r + a.d_model + i0 + 4);
      const float qv[8] = {qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, qb.z, qb.w};
      const float kv[8] = {ka.x, ka.y, ka.z, ka.w, kb.x, kb.y, kb.z, kb.w};
      if (a.rope) {
        const int ip = i0 < half ? i0 + half : i0 - half;
        const float4 qc = *(const float4*)(r + ip), qd = *(const float4*)(r + ip + 4);
        const float4 kc = *(const float4*)(r + a.d_model + ip), kd = *(const float4*)(r + a.d_model + ip + 4);
        const float qo[8] = {qc.x, qc.y, qc.z, qc.w, qd.x, qd.y, qd.z, qd.w};
        const float ko[8] = {kc.x, kc.y, kc.z, kc.w, kd.x, kd.y, kd.z, kd.w};
        const float2* cz = a.rope + (size_t)m * half + (i0 < half ? i0 : i0 - half);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float2 w = cz[u];
          if (i0 < half) { q[u] = fmaf(qv[u], w.x, -(qo[u] * w.y)); k[u] = fmaf(kv[u], w.x, -(ko[u] * w.y)); }
          else           { q[u] = fmaf(qv[u], w.x, qo[u] * w.y);    k[u] = fmaf(kv[u], w.x, ko[u] * w.y); }
        }
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) { q[u] = qv[u]; k[u] = kv[u]; }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] *= a.scale;         // (scale carries log2(e): the attention kernel works with powers of two)
      // the cache takes the key as the decode path stores it: four components of one position are adjacent
      float* const kc = a.Kc + (size_t)h * kv_blocks(a.max_ctx) * (KV_BLOCK * HD);
      *(float4*)(kc + k_index(m, i0, HD)) = make_float4(k[0], k[1], k[2], k[3]);
      *(float4*)(kc + k_index(m, i0 + 4, HD)) = make_float4(k[4], k[5], k[6], k[7]);
    }
    const size_t o = ((((size_t)h * 2 * a.JP + 2 * jp + (rl >> 4)) * CB + (c8 >> 2)) * 64 + (rl & 15) + 16 * (c8 & 3)) * 8;
    uint4 hi, lo;
    split2(q, hi, lo);
    *(uint4*)(a.Qp + o) = hi; *(uint4*)(a.Qp + plane + o) = lo;
    split2(k, hi, lo);
    *(uint4*)(a.Kp + o) = hi; *(uint4*)(a.Kp + plane + o) = lo;
  }
  // values: one lane of one component tile per item
  for (int it = tid; it < CT * 64; it += 256) {
    const int ct = it >> 6, ln = it & 63, i = ln & 15, c = ln >> 4;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int m = 32 * jp + (e < 4 ? 4 * c + e : 16 + 4 * c + (e - 4));
      v[e] = m < a.M ? a.qkv[(size_t)m * 3 * a.d_model + 2 * (size_t)a.d_model + (size_t)h * HD + 16 * ct + i] : 0.f;
    }
    const size_t o = ((((size_t)h * a.JP + jp) * CT + ct) * 64 + ln) * 8;
    uint4 hi, lo;
    split2(v, hi, lo);
    *(uint4*)(a.Vp + o) = hi; *(uint4*)(a.Vp + plane + o) = lo;
    // the cache holds four consecutive positions of one component side by side: the lane's two quadruples
    float* const vc = a.Vc + (size_t)h * kv_blocks(a.max_ctx) * (KV_BLOCK * HD);
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int m0 = 32 * jp + 16 * x + 4 * c;
      float* const dst = vc + v_index(m0, 16 * ct + i, HD);
      if (m0 + 3 < a.M) *(float4*)dst = make_float4(v[4 * x], v[4 * x + 1], v[4 * x + 2], v[4 * x + 3]);
      else for (int u = 0; u < 4; ++u) if (m0 + u < a.M) dst[u] = v[4 * x + u];
    }
  }
}

// The last row of a prompt against the keys and values in the fp32 cache, up to PA_SPLIT workgroups per head, beside those of pattn_kernel's
// other rows (whose two-term operands made up a third of the error of a row's logits: 7B shape, 512 tokens, distance of the first
// token's logits from 64 bits 7.0e-5 with the last row among them, 5.4e-5 with it by itself in a round).  What bounds it: a wave's
// blocks of 16 positions one after the other, 16 KiB of keys and values each, some 3 us of latency: two of them to a wave, up to 512 positions,
// and the workgroup of a head that is done last merges (the others' results are past their L2).  With one workgroup per head the launch
// took as long as that: 333 rows 20 -> 34 us.  A lane i + 16 c has four components of position i's key per 16
// components, and of four positions' values component 16 s + i (see k_index, v_index).
template <int HD>
__device__ __forceinline__ void pattn_last_row(const PAttnArgs& a, int h, int part, float* lds) {
  constexpr int CT = HD / 16, half = HD / 2, NW = 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, c = lane >> 4, m = a.M - 1;
  float* const qs = lds;                                   // [HD], then the waves' outputs [NW][HD], maxima and sums [NW]
  if (tid < HD) {
    const float* r = a.qkv + (size_t)m * 3 * a.d_model + (size_t)h * HD;
    float q = r[tid];
    if (a.rope) {
      const float2 w = a.rope[(size_t)m * half + (tid < half ? tid : tid - half)];
      const float o = r[tid < half ? tid + half : tid - half];
      q = tid < half ? fmaf(q, w.x, -(o * w.y)) : fmaf(q, w.x, o * w.y);
    }
    qs[tid] = q * a.scale;
  }
  __syncthreads();
  float4 q[CT];
#pragma unroll
  for (int s = 0; s < CT; ++s) q[s] = *(const float4*)(qs + 16 * s + 4 * c);
  const size_t base = (size_t)h * kv_blocks(a.max_ctx) * (KV_BLOCK * HD) + lane * 4;
  const int nblk = m / KV_BLOCK + 1;
  float4 kn[CT], vn[CT];
  auto request = [&](int b) {                              // (past the last block: that one again, unused)
    const size_t o = base + (size_t)(b < nblk ? b : nblk - 1) * (KV_BLOCK * HD);
#pragma unroll
    for (int s = 0; s < CT; ++s) { kn[s] = *(const float4*)(a.Kc + o + s * 256); vn[s] = *(const float4*)(a.Vc + o + s * 256); }
  };
  float mx = -INFINITY, l = 0.f, acc[CT];
#pragma unroll
  for (int s = 0; s < CT; ++s) acc[s] = 0.f;
  const int stride = a.sp * NW;
  request(part * NW + wave);
  for (int b = part * NW + wave; b < nblk; b += stride) {
    float4 k[CT], v[CT];
#pragma unroll
    for (int s = 0; s < CT; ++s) { k[s] = kn[s]; v[s] = vn[s]; }
    request(b + stride);
    float z = 0.f;
#pragma unroll
    for (int s = 0; s < CT; ++s) { z = fmaf(q[s].x, k[s].x, z); z = fmaf(q[s].y, k[s].y, z); z = fmaf(q[s].z, k[s].z, z); z = fmaf(q[s].w, k[s].w, z); }
    z += __shfl_xor(z, 16, WAVE);
    z += __shfl_xor(z, 32, WAVE);
    if (b * KV_BLOCK + i > m) z = -INFINITY;
    float bm = z;
#pragma unroll
    for (int o = 1; o < 16; o *= 2) bm = fmaxf(bm, __shfl_xor(bm, o, WAVE));
    const float mnew = fmaxf(mx, bm), resc = __builtin_amdgcn_exp2f(mx - mnew);    // (finite: a block's first position is a row's)
    mx = mnew;
    const float p = __builtin_amdgcn_exp2f(z - mnew);
    l = fmaf(l, resc, p);
    const float p0 = __shfl(p, 4 * c, WAVE), p1 = __shfl(p, 4 * c + 1, WAVE), p2 = __shfl(p, 4 * c + 2, WAVE), p3 = __shfl(p, 4 * c + 3, WAVE);
#pragma unroll
    for (int s = 0; s < CT; ++s) {
      float t = acc[s] * resc;
      t = fmaf(p0, v[s].x, t); t = fmaf(p1, v[s].y, t); t = fmaf(p2, v[s].z, t); t = fmaf(p3, v[s].w, t);
      acc[s] = t;
    }
  }
#pragma unroll
  for (int o = 1; o < 16; o *= 2) l += __shfl_xor(l, o, WAVE);
  float* const wo = lds + HD;
  float* const wm = wo + NW * HD;
#pragma unroll
  for (int s = 0; s < CT; ++s) {
    acc[s] += __shfl_xor(acc[s], 16, WAVE);
    acc[s] += __shfl_xor(acc[s], 32, WAVE);
    if (c == 0) wo[wave * HD + 16 * s + i] = acc[s];
  }
  if (lane == 0) { wm[wave] = mx; wm[NW + wave] = l; }
  __syncthreads();
  float top = wm[0], num = 0.f, den = 0.f;                 // (finite: a workgroup's first wave has a block)
#pragma unroll
  for (int w = 1; w < NW; ++w) top = fmaxf(top, wm[w]);
  const int i0 = tid < HD ? tid : 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {                           // (a wave without a block adds zeros)
    const float f = __builtin_amdgcn_exp2f(wm[w] - top);
    num = fmaf(f, wo[w * HD + i0], num);
    den = fmaf(f, wm[NW + w], den);
  }
  if (a.sp > 1) {
    float* const mine = a.lpart + (size_t)(h * PA_SPLIT + part) * (HD + 2);
    auto put = [](float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto get = [](float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (tid < HD) put(mine + tid, num);
    if (tid == 0) { put(mine + HD, top); put(mine + HD + 1, den); }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (where every XCD finds them)
    __syncthreads();
    int* const done = (int*)(wm + 2 * NW);
    if (tid == 0) *done = atomicInc(a.lcnt + h, a.sp - 1) == (unsigned)a.sp - 1;
    __syncthreads();
    if (!*done) return;
    top = -INFINITY;
    for (int p = 0; p < a.sp; ++p) top = fmaxf(top, get(a.lpart + (size_t)(h * PA_SPLIT + p) * (HD + 2) + HD));
    num = den = 0.f;
    for (int p = 0; p < a.sp; ++p) {
      float* const q = a.lpart + (size_t)(h * PA_SPLIT + p) * (HD + 2);
      const float f = __builtin_amdgcn_exp2f(get(q + HD) - top);
      num = fmaf(f, get(q + i0), num);
      den = fmaf(f, get(q + HD + 1), den);
    }
  }
  if (tid >= HD) return;
  const int MT = (a.M + 15) / 16, KT = a.d_model / 32;
  put_packed1(a.outp, (size_t)MT * KT * 512, KT, m, h * HD + tid, num / den);
}

// A workgroup is 4 waves of one head; a wave owns QT consecutive 16-row query tiles (the columns of its MFMAs),
// the workgroup 64 QT consecutive rows.  The workgroup walks the 32-row steps of keys and values up to its last
// row: a step's blocks (keys hi, lo; values hi, lo: 4 HD / 16 KiB) come into LDS by direct loads, a step ahead of
// their use, two buffers; every wave reads them from there (a fourth of the traffic of four waves loading for
// themselves) and keeps a running maximum and sum per row.
template <int HD, int QT>
__global__ __launch_bounds__(256, (QT <= 2 ? 2 : 1)) void pattn_kernel(PAttnArgs a) {
  constexpr int CB = HD / 32, CT = HD / 16;
  constexpr int STEP_BLKS = 4 * CB + 2 * CT;               // 1 KiB blocks per step: K hi (2 CB), K lo (2 CB), V hi (CT), V lo (CT)
  extern __shared__ float4 pattn_lds4[];
  char* const lds = (char*)pattn_lds4;                     // [2][STEP_BLKS] KiB
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the longest rows first; heads that divide among the XCDs (workgroup b runs on XCD b % 8) stay on one each, where a dozen
  // workgroups of a head walk the same steps and find them in its L2.  With a head's rows spread over all XCDs the steps came from
  // memory eight times, 3 TB/s of them: 13B shape, 4095 rows, 892 -> 526 us.  (Other numbers of heads, 12, 20 or 36, keep
  // that order.)
  // (The workgroups of the last row, where there are any, come behind them all: in front of them they held up the longest ones, 7B shape, 2000
  // rows, 149 -> 163 us.)
  const int b = blockIdx.x;
  if (b >= a.gx * a.H) { const int r = b - a.gx * a.H; pattn_last_row<HD>(a, r % a.H, r / a.H, (float*)lds); return; }
  int h = b / a.gx, wg = a.gx - 1 - (b - h * a.gx);
  if ((a.H & 7) == 0) {
    const int r = b >> 3, per = a.H >> 3;
    h = (b & 7) + 8 * (r % per); wg = a.gx - 1 - r / per;
  }
  const int MT2 = 2 * a.JP;
  const int qt0 = (wg * 4 + wave) * QT;                    // this wave's first tile (may lie past the prompt: then it only helps to load)
  const int bn = lane & 15, bc = lane >> 4;
  const size_t plane = (size_t)a.H * a.JP * CT * 1024;     // bytes per plane
  u32x4 qh[QT][CB], ql[QT][CB];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int tile = qt0 + t < MT2 ? qt0 + t : MT2 - 1;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const char* src = (const char*)a.Qp + (((size_t)h * MT2 + tile) * CB + cb) * 1024 + lane * 16;
      qh[t][cb] = *(const u32x4*)src;
      ql[t][cb] = *(const u32x4*)(src + plane);
    }
  }
  f32x4 oacc[QT][CT];
  float mx[QT], l[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    mx[t] = -INFINITY; l[t] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) oacc[t][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  int wg_last = (wg * 4 + 3) * QT + QT - 1;
  if (wg_last > MT2 - 1) wg_last = MT2 - 1;
  const int nsteps = wg_last / 2 + 1;                      // steps the workgroup walks (<= JP)
  auto stage = [&](int jp, int buf) {
    for (int b = wave; b < STEP_BLKS; b += 4) {
      const char* src;
      if (b < 4 * CB) {
        const int pl = b / (2 * CB), idx = b - pl * 2 * CB;
        src = (const char*)a.Kp + pl * plane + (((size_t)h * MT2 + 2 * jp) * CB + idx) * 1024;
      } else {
        const int bb = b - 4 * CB, pl = bb / CT, idx = bb - pl * CT;
        src = (const char*)a.Vp + pl * plane + (((size_t)h * a.JP + jp) * CT + idx) * 1024;
      }
      dma16(src + lane * 16, lds + ((size_t)buf * STEP_BLKS + b) * 1024);
    }
  };
  stage(0, 0);
  // the queries are waited for here, once: the compiler's own count of outstanding loads knows nothing of the
  // direct-to-LDS requests, and a wait for a query register inside the loop would drain the step in flight
#pragma unroll
  for (int t = 0; t < QT; ++t)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) asm volatile("" : "+v"(qh[t][cb]), "+v"(ql[t][cb]));
  for (int jp = 0; jp < nsteps; ++jp) {
    // this step's blocks have arrived (this wave's requests, then everybody's); everybody is done with the other buffer
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (jp + 1 < nsteps) stage(jp + 1, (jp + 1) & 1);
    const char* const kb = lds + (size_t)(jp & 1) * STEP_BLKS * 1024 + lane * 16;
    const char* const vb = kb + 4 * CB * 1024;
    // the wave takes part while the step begins at or before the last row of its last tile; a tile that lies
    // wholly before the step is computed all the same and masked (its weights come out as exact zeros)
    if (2 * jp > qt0 + QT - 1) continue;
    f32x4 s[QT][2];
#pragma unroll
    for (int t = 0; t < QT; ++t) { s[t][0] = (f32x4){0.f, 0.f, 0.f, 0.f}; s[t][1] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
    // (consecutive MFMAs go to different accumulators: none waits for the one before it)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      bf16x8 kh[2], kl[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        kh[x] = __builtin_bit_cast(bf16x8, *(const u32x4*)(kb + (x * CB + cb) * 1024));
        kl[x] = __builtin_bit_cast(bf16x8, *(const u32x4*)(kb + ((2 + x) * CB + cb) * 1024));
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < QT; ++t) s[t][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[x], __builtin_bit_cast(bf16x8, qh[t][cb]), s[t][x], 0, 0, 0);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < QT; ++t) s[t][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl[x], __builtin_bit_cast(bf16x8, qh[t][cb]), s[t][x], 0, 0, 0);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < QT; ++t) s[t][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[x], __builtin_bit_cast(bf16x8, ql[t][cb]), s[t][x], 0, 0, 0);
    }
    // s[t][x][r]: row 32 jp + 16 x + 4 bc + r against query row 16 (qt0 + t) + bn
    const bool diag = 32 * jp + 31 > 16 * qt0;             // the step reaches past the first row of the wave's first tile
    u32x4 ph[QT], plo[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const int qrow = 16 * (qt0 + t) + bn;
      float sv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] = s[t][e >> 2][e & 3];
      if (diag) {                                          // mask what lies after each row
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (32 * jp + 16 * (e >> 2) + 4 * bc + (e & 3) > qrow) sv[e] = -INFINITY;
      }
      float bm = sv[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) bm = fmaxf(bm, sv[e]);
      // the running maximum of a query is the same in its four lanes; it moves only when some lane of the wave has
      // met a larger score (rare after the first steps), and only then are the lanes compared and the sums rescaled
      if (__any(bm > mx[t])) {
        bm = fmaxf(bm, __shfl_xor(bm, 16, WAVE));
        bm = fmaxf(bm, __shfl_xor(bm, 32, WAVE));
        const float mnew = fmaxf(mx[t], bm);               // finite from the first step on: row 0 is visible to every query
        const float resc = __builtin_amdgcn_exp2f(mx[t] - mnew);
        mx[t] = mnew;
        l[t] *= resc;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r) oacc[t][ct][r] *= resc;
      }
      float pv[8], ps = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) { pv[e] = __builtin_amdgcn_exp2f(sv[e] - mx[t]); ps += pv[e]; }
      l[t] += ps;                                          // this lane's 8 rows of the step; the four lanes of a query are added at the end
      uint4 hi, lo;
      split2(pv, hi, lo);
      ph[t] = (u32x4){hi.x, hi.y, hi.z, hi.w}; plo[t] = (u32x4){lo.x, lo.y, lo.z, lo.w};
    }
    // outputs: rows = components 16 ct + 4 bc + r, reduction over the step's 32 rows in the order Vp holds them
#pragma unroll
    for (int c2 = 0; c2 < CT; c2 += 2) {
      bf16x8 vh[2], vl[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        vh[x] = __builtin_bit_cast(bf16x8, *(const u32x4*)(vb + (c2 + x) * 1024));
        vl[x] = __builtin_bit_cast(bf16x8, *(const u32x4*)(vb + (CT + c2 + x) * 1024));
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < QT; ++t) oacc[t][c2 + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vh[x], __builtin_bit_cast(bf16x8, ph[t]), oacc[t][c2 + x], 0, 0, 0);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < QT; ++t) oacc[t][c2 + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vl[x], __builtin_bit_cast(bf16x8, ph[t]), oacc[t][c2 + x], 0, 0, 0);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int t = 0; t < QT; ++t) oacc[t][c2 + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vh[x], __builtin_bit_cast(bf16x8, plo[t]), oacc[t][c2 + x], 0, 0, 0);
    }
  }
  const int MT = (a.M + 15) / 16, KT = a.d_model / 32;
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int mrow = 16 * (qt0 + t) + bn;
    float lt = l[t];                                       // lanes bc = 0, 1, 2, 3 of the query, in that order
    {
      const float l1 = __shfl(lt, bn + 16, WAVE), l2 = __shfl(lt, bn + 32, WAVE), l3 = __shfl(lt, bn + 48, WAVE);
      lt = ((__shfl(lt, bn, WAVE) + l1) + l2) + l3;
    }
    if (mrow >= a.M - (a.last ? 1 : 0)) continue;
    const float inv = 1.0f / lt;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float y[4] = {oacc[t][ct][0] * inv, oacc[t][ct][1] * inv, oacc[t][ct][2] * inv, oacc[t][ct][3] * inv};
      put_packed4(a.outp, (size_t)MT * KT * 512, KT, mrow, h * HD + 16 * ct + 4 * bc, y);
    }
  }
}
#endif

// launchers (ppd_prefill.hip)
hipError_t launch_pack_rows(hipStream_t stream, const PackArgs& a);
PGemmPlan plan_pgemm(int M, int KT, int NT, bool cut);
hipError_t launch_pgemm(hipStream_t stream, PGemmArgs a, bool paired, PGemmPlan plan);
hipError_t pgemm_setup(PGemmPlan plan, bool paired);
hipError_t launch_rgemm(hipStream_t stream, RGemmArgs a, bool paired);
hipError_t rgemm_setup();
hipError_t launch_sgemm(hipStream_t stream, const SGemmArgs& a);
hipError_t sgemm_setup();
hipError_t launch_pkv_pack(hipStream_t stream, const PKvPackArgs& a, int head_dim);
hipError_t launch_pattn(hipStream_t stream, const PAttnArgs& a, int head_dim);
// bytes of the packed form of M rows of K columns
inline size_t packed_bytes(int M, int K) { return (size_t)2 * ((M + 15) / 16) * ((K + 31) / 32) * 1024; }

}  // namespace ppd
