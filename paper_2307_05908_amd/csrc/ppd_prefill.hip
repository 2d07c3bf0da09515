// Kernel instances and launchers of the compute-bound prompt pass (ppd_prefill.h).
#define PPD_PREFILL_TU 1
#include "ppd_prefill.h"

#include <math.h>
#include <string.h>


namespace ppd {

hipError_t launch_pack_rows(hipStream_t stream, const PackArgs& a) {
  if (a.M < 1 || a.K < 8 || (a.K & 7) || (a.ld & 3) || a.MT < (a.M + 15) / 16 || a.KT != (a.K + 31) / 32) return hipErrorInvalidValue;
  if (a.S && ((a.K & 7) || a.ld != a.K)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pack_rows_kernel, dim3((a.MT + 7) / 8 * 128), dim3(MG_THREADS), 0, stream, a);
  return hipGetLastError();
}

// The tiles a product is cut into, and what their workgroups take (MI355X, us): a stage of 32 columns, and everything else of a
// workgroup; per: workgroups on a compute unit at a time, which take as long as one after the other but hide that rest.
struct PGemmTile { int ww, wx, tw, tx, r; float stage, rest; int per; };
constexpr PGemmTile pg_tiles[PG_TILES] = {
  {2, 2, 1, 1, 5, 0.144f, 3.0f, 2},      //  64 x  64 (weight rows x prompt rows)
  {2, 2, 2, 1, 4, 0.224f, 3.0f, 2},      // 128 x  64
  {2, 2, 2, 2, 3, 0.390f, 3.3f, 2},      // 128 x 128
  {2, 2, 3, 2, 5, 0.524f, 6.7f, 1},      // 192 x 128
  {2, 2, 3, 4, 3, 0.978f, 8.4f, 1},      // 192 x 256
  {2, 4, 4, 2, 3, 1.276f, 4.9f, 1},      // 256 x 256
  {2, 4, 5, 2, 3, 1.549f, 6.3f, 1},      // 320 x 256
};

// The shortest time by this account: workgroups of a compute unit times stages, or the weights at 4 TB/s, whichever is longer
// (a fourth-power mean of the two); cutting the reduction length adds the way through memory.  Fitted to 280 products (20 matrices
// of 768 x 768 to 27648 x 5120, 33 to 4095 rows) with every tile and cut, products on their own: the choice is 1.0 % from
// the best one in the geometric mean, 12 % at worst, and 1.49 times the speed of the kernel before (at worst 1.5 % slower: 320 rows,
// 22016 x 4096).  Between a layer's other launches a product takes 1.15 to 1.4 times what the account says (7B shape, 511 rows, QKV, O, FFN
// in, FFN out: 74, 32, 134, 80 us by it, 97, 44, 154, 97 in the model), whatever the tile: of the tiles and cuts measured there, with
// 127 and with 511 rows, none was faster than the choice.
// (cut: whether the reduction length may be cut)
PGemmPlan plan_pgemm(int M, int KT, int NT, bool cut) {
  const int MT = (M + 15) / 16;
  PGemmPlan best = {0, 1, 0.f};
  float tbest = 0.f;
  for (int c = 0; c < PG_TILES; ++c) {
    const PGemmTile& p = pg_tiles[c];
    const int64_t T = (int64_t)((NT + 2 * p.ww * p.tw - 1) / (2 * p.ww * p.tw)) * ((MT + 2 * p.wx * p.tx - 1) / (2 * p.wx * p.tx));
    const size_t bytes = (size_t)p.ww * p.wx * p.tw * p.tx * 4096;
    for (const int S : {1, 2, 3, 4, 6, 8}) {
      if (S > 1 && (!cut || KT < 6 * S || T > PG_MAX_TILES || T * S * bytes > PG_WS_BYTES)) break;
      const int64_t m = (T * S + 255) / 256;
      const float comp = (float)m * (float)((KT + S - 1) / S) * p.stage + (float)((m + p.per - 1) / p.per) * p.rest;
      const float mem = (float)NT * (float)KT * (1024.f / 4.05e6f);
      float t = sqrtf(sqrtf(comp * comp * comp * comp + mem * mem * mem * mem));
      if (S > 1) t += 1.95f + 0.305e-6f * (float)bytes * (float)(T * S) + 1.455e-5f * (float)bytes * (float)S;
      if ((c == 0 && S == 1) || t < tbest) { tbest = t; best = {c, S, t}; }
    }
  }
  return best;
}

template <bool PAIRED, int C>
static hipError_t launch_pgemm_t(hipStream_t stream, const PGemmArgs& a) {
  constexpr PGemmTile p = pg_tiles[C];
  constexpr int lds = p.r * (2 * p.ww * p.tw + 4 * p.wx * p.tx) * 1024;
  const auto k = pgemm_kernel<PAIRED, p.ww, p.wx, p.tw, p.tx, p.r>;
  if (a.M == 0) return hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  hipLaunchKernelGGL(k, dim3((a.NB * a.MB * a.S + 7) / 8 * 8), dim3(p.ww * p.wx * WAVE), lds, stream, a);
  return hipGetLastError();
}

template <int C>
static hipError_t launch_pgemm_c(hipStream_t stream, const PGemmArgs& a, bool paired, int tile) {
  if constexpr (C < PG_TILES) {
    if (C == tile) return paired ? launch_pgemm_t<true, C>(stream, a) : launch_pgemm_t<false, C>(stream, a);
    return launch_pgemm_c<C + 1>(stream, a, paired, tile);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pgemm(hipStream_t stream, PGemmArgs a, bool paired, PGemmPlan plan) {
  if (a.M < 1 || a.MT != (a.M + 15) / 16 || a.KT < 1 || a.NT < 1 || (a.ntot & 3) || (a.ldy & 3) ||
      plan.tile < 0 || plan.tile >= PG_TILES) return hipErrorInvalidValue;
  const PGemmTile& p = pg_tiles[plan.tile];
  a.NB = (a.NT + 2 * p.ww * p.tw - 1) / (2 * p.ww * p.tw);
  a.MB = (a.MT + 2 * p.wx * p.tx - 1) / (2 * p.wx * p.tx);
  a.S = plan.S;
  const int64_t T = (int64_t)a.NB * a.MB;
  if (a.S < 1 || a.S > a.KT || T * a.S > (1 << 24) || (int64_t)a.KT * (a.S + 1) >= (1 << 30)) return hipErrorInvalidValue;
  if (a.S > 1 && (!a.ws || !a.cnt || T > PG_MAX_TILES || (size_t)T * a.S * p.ww * p.wx * p.tw * p.tx * 4096 > PG_WS_BYTES)) return hipErrorInvalidValue;
  return launch_pgemm_c<0>(stream, a, paired, plan.tile);
}

hipError_t pgemm_setup(PGemmPlan plan, bool paired) {
  PGemmArgs a; memset(&a, 0, sizeof a);            // (no rows: the kernel's LDS only)
  return launch_pgemm_c<0>(nullptr, a, paired, plan.tile);
}

template <bool PAIRED, int TT>
static hipError_t launch_rgemm_t(hipStream_t stream, const RGemmArgs& a, int grid) {
  const size_t lds = (size_t)a.tiles_wg * MG_WAVES * 16 * 16 * sizeof(float) * (a.M > 16 ? 2 : 1);
  if (a.M > 16) hipLaunchKernelGGL((rgemm_kernel<PAIRED, TT, 2>), dim3(grid), dim3(MG_THREADS), lds, stream, a);
  else hipLaunchKernelGGL((rgemm_kernel<PAIRED, TT, 1>), dim3(grid), dim3(MG_THREADS), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_rgemm(hipStream_t stream, RGemmArgs a, bool paired) {
  if (a.M < 1 || a.M > 32 || a.KT < 1 || a.NT < 1 || (size_t)a.NT * a.KT * 1024 > 0x7fffffffu) return hipErrorInvalidValue;
  a.wbytes = (unsigned)((size_t)a.NT * a.KT * 1024);
  // one workgroup per compute unit, the smallest grid with the same number of tiles in each; more than RG_TILES_MAX tiles do
  // not fit LDS (then more workgroups)
  a.tiles_wg = (a.NT + 255) / 256;
  if (a.tiles_wg > RG_TILES_MAX) a.tiles_wg = RG_TILES_MAX;
  const int grid = (a.NT + a.tiles_wg - 1) / a.tiles_wg;
  // tiles that share their loads of the rows: all of a workgroup's, or half of them past 6 (registers)
  const int tt = a.tiles_wg <= 4 ? a.tiles_wg : (a.tiles_wg <= 6 ? 6 : 4);
  switch (tt) {
    case 1: return paired ? launch_rgemm_t<true, 1>(stream, a, grid) : launch_rgemm_t<false, 1>(stream, a, grid);
    case 2: return paired ? launch_rgemm_t<true, 2>(stream, a, grid) : launch_rgemm_t<false, 2>(stream, a, grid);
    case 3: return paired ? launch_rgemm_t<true, 3>(stream, a, grid) : launch_rgemm_t<false, 3>(stream, a, grid);
    case 4: return paired ? launch_rgemm_t<true, 4>(stream, a, grid) : launch_rgemm_t<false, 4>(stream, a, grid);
    default: return paired ? launch_rgemm_t<true, 6>(stream, a, grid) : launch_rgemm_t<false, 6>(stream, a, grid);
  }
}

template <bool PAIRED, int TT>
static hipError_t rgemm_setup_t() {
  const int lds = RG_TILES_MAX * MG_WAVES * 32 * 16 * (int)sizeof(float);
  hipError_t e = hipFuncSetAttribute((const void*)rgemm_kernel<PAIRED, TT, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void*)rgemm_kernel<PAIRED, TT, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  return e;
}

hipError_t rgemm_setup() {
  hipError_t e = hipSuccess;
  for (auto f : {rgemm_setup_t<true, 4>, rgemm_setup_t<true, 6>, rgemm_setup_t<false, 4>, rgemm_setup_t<false, 6>})
    if (e == hipSuccess) e = f();
  return e;
}

hipError_t launch_sgemm(hipStream_t stream, const SGemmArgs& a) {
  if (a.M < 1 || a.M > 32 || a.KT < 1 || a.NT < 1 || a.ntot > a.NT * 16 || (a.ntot & 3)) return hipErrorInvalidValue;
  // a wave per tile, and so many waves to a workgroup that there are some 256 workgroups
  const int W = a.NT >= 192 ? 8 : (a.NT >= 96 ? 4 : 2);
  const int grid = (a.NT + W - 1) / W * 8;
  const int nb8 = (a.KT + MG_WAVES - 1) / MG_WAVES, MT = a.M > 16 ? 2 : 1;
  const size_t lds = (size_t)(nb8 > SG_PB ? 2 * SG_PB : nb8) * 2 * MT * 1024;
  if (MT == 2) hipLaunchKernelGGL(sgemm_kernel<2>, dim3(grid), dim3(W * WAVE), lds, stream, a);
  else hipLaunchKernelGGL(sgemm_kernel<1>, dim3(grid), dim3(W * WAVE), lds, stream, a);
  return hipGetLastError();
}

hipError_t sgemm_setup() {
  hipError_t e = hipFuncSetAttribute((const void*)sgemm_kernel<1>, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * SG_PB * 2 * 1024);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void*)sgemm_kernel<2>, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * SG_PB * 4 * 1024);
  return e;
}

hipError_t launch_pkv_pack(hipStream_t stream, const PKvPackArgs& a, int head_dim) {
  if (a.M < 1 || a.JP != (a.M + 31) / 32 || (head_dim != 64 && head_dim != 128) || (a.d_model & 3)) return hipErrorInvalidValue;
  const dim3 grid(a.JP, a.H);
  if (head_dim == 128) hipLaunchKernelGGL(pkv_pack_kernel<128>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(pkv_pack_kernel<64>, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

template <int HD, int QT>
static hipError_t launch_pattn_t(hipStream_t stream, PAttnArgs a) {
  const int MT = (a.M + 15) / 16;
  a.gx = (MT + 4 * QT - 1) / (4 * QT);
  const int nblk = (a.M + 15) / 16;                  // blocks of positions of the last row: two to a wave of its workgroups
  a.sp = nblk <= 8 ? 1 : (nblk + 7) / 8;
  if (a.sp > PA_SPLIT) a.sp = PA_SPLIT;
  const dim3 grid((a.gx + (a.last ? a.sp : 0)) * a.H);
  const size_t lds = (size_t)2 * (4 * (HD / 32) + 2 * (HD / 16)) * 1024;
  hipLaunchKernelGGL((pattn_kernel<HD, QT>), grid, dim3(256), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_pattn(hipStream_t stream, const PAttnArgs& a, int head_dim) {
  if (a.M < 1 || a.JP != (a.M + 31) / 32 || (head_dim != 64 && head_dim != 128) || a.d_model % 32) return hipErrorInvalidValue;
  if (a.last && (!a.qkv || !a.Kc || !a.Vc || !a.lpart || !a.lcnt || a.M > a.max_ctx)) return hipErrorInvalidValue;
  // rows per workgroup (64 QT): two query tiles per wave once the prompt gives enough workgroups (four would leave
  // one wave per SIMD: measured slower)
  const bool two = a.M >= 1024;
  if (head_dim == 128) return two ? launch_pattn_t<128, 2>(stream, a) : launch_pattn_t<128, 1>(stream, a);
  return two ? launch_pattn_t<64, 2>(stream, a) : launch_pattn_t<64, 1>(stream, a);
}

}  // namespace ppd
