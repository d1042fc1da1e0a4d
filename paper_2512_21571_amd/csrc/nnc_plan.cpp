// Analytic tile chooser: see nnc_plan.h for the model (paper Section 3.2.2).
#include "nnc_plan.h"

#include <algorithm>
#include <cmath>

namespace nnc {

Machine machine_mi355x(int cus) {
  Machine m{};
  m.cus = cus > 0 ? cus : 256;
  m.lds_bytes = 160 * 1024;
  m.vgprs_per_wave = 256;
  // measured on these kernels, not datasheet values: inside a pass the GEMMs stream at 5.8 TB/s
  // once every CU has work
  m.hbm_bytes_per_us = 5.8e6;
  m.launch_us = 5.0;
  // whole prompt passes with and without k slices on the large tiles (0.6B .. 8B layer shapes, 768 ..
  // 4096 tokens): slices pay (4 - 9 %) while the partials are a few tens of MB and cost 2 - 3 % once
  // they are not; the second rate is the one at which the model stops choosing the losing launches.
  // A limit of 60 MB for every block picks launches that lose, O and down with their norms, us per layer: 8B 768 tokens
  // 147 -> 163, 1.7B 1536 55 -> 70 (prompts of 4 layers: 8B 640 tokens 1640 -> 1720, 900 1950 -> 2084, 1.7B 3088 1831 -> 1874).
  // Two-piece blocks of up to 512 tokens have it: there only O and down of 4096-wide models at 489 - 512 tokens lie
  // between, with four slices (8B 512: down 116 -> 99, O 46 -> 48, the prompt 1693 -> 1580)
  m.fold_cached_bytes = 48e6;
  m.fold_cached_short_bytes = 60e6;
  m.fold_bytes_per_us = 2.0e6;
  // the weight-streaming GEMM alone, launches back to back, 200 (rows, k, batch, row tiles,
  // k slices) combinations of the five model shapes: least-squares / best-pick fit
  m.stream_bytes_per_us = 6.4e6;
  m.cu_bytes_per_us = 58e3;
  m.skinny_launch_us = 2.5;
  m.skinny_round_us = 0.6;
  // prompt GEMM with direct copies, us per k step of the 256 / 192 / 128 x 128 tiles: two workgroups per CU, and a lone one as a
  // share of that, a tenth more in one-piece residual projections, whose epilogue reads and writes twice the outputs per tile with
  // no other workgroup to hide it; of the 256 x 256 and 192 x 256 tiles, one workgroup per CU, and of a last round of 128 x 256 halves of the former.
  // Fitted to every tile and slice count at 14 sizes of 200 - 4096 tokens of the 0.6B .. 8B shapes (224 GEMMs, the norms' share of the
  // slices included): the picks are 2.4 % above the best tiles in the sum, 32 in 1000 in the mean
  m.pg_pair[0] = 0.844; m.pg_solo[0] = 0.585;
  m.pg_pair[1] = 0.631; m.pg_solo[1] = 0.727;
  m.pg_pair[2] = 0.482; m.pg_solo[2] = 0.552;
  m.pg_solo_resid1 = 1.086;
  m.pg_big = 0.77;
  m.pg_half = 0.547;
  m.pg_big12 = 0.63;
  // the register-ring kernel of the 64-row tiles: 0.26 us per k step with 4 matrix-core
  // instructions per wave (64 x 64), 0.37 with 8 (64 x 128)
  m.rg_c1 = 0.0275;
  m.rg_c0 = 0.150;
  m.rg_solo = 0.73;
  m.rg_solo_resid1 = 0.78;
  return m;
}

namespace {
int ceil_div(int a, int b) { return (a + b - 1) / b; }

struct PgTile {
  int code, nt, tt;
  bool lds_direct;  // LDS stages (three, 128 x 128: four) filled by direct copies; else register ring, two stages
  int wgs_per_cu;   // resident workgroups per CU the kernel is built for
};
// every block tile the prompt GEMM kernels are instantiated for, plus one that is not (256 x 256
// with two workgroups per CU: it shows the capacity constraints at work and is never chosen)
const PgTile kPgTiles[] = {{1, 16, 8, true, 2}, {4, 12, 8, true, 2}, {2, 8, 8, true, 2}, {0, 4, 8, false, 2},
                           {3, 4, 4, false, 2}, {5, 16, 16, true, 1}, {6, 12, 16, true, 1}, {-1, 16, 16, true, 2}};
}  // namespace

PrefillGemmPlan plan_prefill_gemm(const Machine& mc, int n_tiles, int KT, int col_tiles, int n_tokens, int pieces,
                                  int epi, int max_k_slices) {
  PrefillGemmPlan best{};
  best.tile = -1;
  best.t_us = 1e30;
  const double W = (double)n_tiles * KT * 1024.0, X = (double)col_tiles * KT * 1024.0;
  const double N = (double)n_tiles * 16.0;
  const double out_bytes = epi == PLAN_EPI_STORE ? n_tokens * N * 4.0
                           : epi == PLAN_EPI_RESID ? n_tokens * N * 8.0  // read-modify-write of the residual stream
                                                   : n_tokens * (N / 2.0) * 2.0 * pieces;
  for (const PgTile& t : kPgTiles) {
    const int wgs_per_cu = t.wgs_per_cu;
    ++best.candidates;
    // capacity: staged operands of the resident workgroups in LDS; accumulators and two sets of
    // fragments (one for the ring kernels) in the wave's registers
    const int stages = t.lds_direct ? t.nt == 8 ? 4 : 3 : 2;
    const int lds = stages * (t.nt + t.tt) * 1024 * wgs_per_cu;
    const int wi = t.nt / 2, wj = t.tt / 2;
    const int regs = wi * wj * 4 + (t.lds_direct ? 2 : 1) * (wi + wj) * 4 + (t.lds_direct ? 0 : 8 * (t.nt / 4 + t.tt / 4) * 4);
    // (a wave alone on its SIMD has the accumulation registers on top of the ordinary ones)
    if (lds > mc.lds_bytes || regs > mc.vgprs_per_wave * (wgs_per_cu == 1 ? 2 : 1) || t.code < 0) {
      ++best.rejected_by_capacity;
      continue;
    }
    const int ks_max = epi != PLAN_EPI_RESID ? 1 : std::max(1, max_k_slices);
    // a slice shorter than the register ring (or, for the tiles with three LDS stages in flight,
    // than a few times their pipeline) gains nothing
    const int kts_min = !t.lds_direct ? 8 : wgs_per_cu == 1 ? 32 : 16;
    for (int ks = 1; ks <= ks_max; ++ks) {
      const int kts = ceil_div(KT, ks);
      if (ks > 1 && kts < kts_min) break;
      const int slices = ceil_div(KT, kts);
      if (slices != ks) continue;            // same launch as a smaller ks
      const int wgs = ceil_div(n_tiles, t.nt) * ceil_div(col_tiles, t.tt) * slices;
      const int slots = wgs_per_cu * mc.cus;
      const int full = wgs / slots, rem = wgs - full * slots;
      const bool resid1 = epi == PLAN_EPI_RESID && pieces == 1;
      double t_comp;
      if (wgs_per_cu == 1) {
        const double t_last = t.nt == 16 && 2 * rem <= mc.cus ? mc.pg_half : t.nt == 16 ? mc.pg_big : mc.pg_big12;
        t_comp = kts * (full * (t.nt == 16 ? mc.pg_big : mc.pg_big12) + (rem ? t_last : 0.0));
      } else {
        const int q = t.nt == 16 ? 0 : t.nt == 12 ? 1 : 2;
        const double t2 = t.lds_direct ? mc.pg_pair[q] : mc.rg_c0 + mc.rg_c1 * wi * wj;
        const double t1 = t2 * (t.lds_direct ? mc.pg_solo[q] * (resid1 ? mc.pg_solo_resid1 : 1.0) : resid1 ? mc.rg_solo_resid1 : mc.rg_solo);
        t_comp = kts * (full * t2 + (rem == 0 ? 0.0 : rem <= mc.cus ? t1 : t2));
      }
      const double fold = (slices - 1) * n_tokens * N * 4.0 * 2.0;  // partials written, then read by the norm kernel
      const double t_mem = (W + X) / mc.hbm_bytes_per_us;
      const double cached = pieces == 2 && n_tokens <= 512 ? mc.fold_cached_short_bytes : mc.fold_cached_bytes;
      const double t_fold = fold / (fold <= cached ? mc.hbm_bytes_per_us : mc.fold_bytes_per_us);
      const double total = std::max(t_comp, t_mem) + out_bytes / mc.hbm_bytes_per_us + t_fold + mc.launch_us;
      if (total < best.t_us * 0.999) {
        best.tile = t.code; best.nt = t.nt; best.tt = t.tt;
        best.k_slices = slices; best.kts_per_split = slices > 1 ? kts : 0;
        best.workgroups = wgs;
        best.t_comp_us = t_comp; best.t_mem_us = t_mem; best.t_us = total;
      }
    }
  }
  return best;
}

SkinnyGemmPlan plan_skinny_gemm(const Machine& mc, int n_tiles, int KT, int ncols, int nseq, int rt_choices,
                                int max_k_slices) {
  SkinnyGemmPlan best{};
  best.rt = 0;
  best.t_us = 1e30;
  const double W = (double)n_tiles * KT * 1024.0;
  // operand bytes per k tile: one 16-byte group per (k / 8 or k / 4, column), i.e. 64 bytes per
  // column, and the kernel loads whole blocks of 16 columns
  const double x_per_kt = 64.0 * ((ncols + 15) / 16 * 16);
  for (int rt = 1; rt <= 8; ++rt) {
    if (!((rt_choices >> rt) & 1) || (n_tiles % rt && !(rt_choices & 1))) continue;
    for (int ks = 1; ks <= std::max(1, max_k_slices); ++ks) {
      const int kts = ceil_div(KT, ks);
      if (ks > 1 && kts < 8) break;  // at least two k tiles per wave
      const int slices = ceil_div(KT, kts);
      if (slices != ks) continue;
      const int wgs = ceil_div(n_tiles, rt) * slices;
      // T_mem, level 1: what the busiest CU pulls through its vector memory path.  A workgroup
      // reads its rt x kts weight tiles once, and the operand of its k slice once for all its
      // row tiles; the operand comes from L2, but it crosses the same per-CU path as the
      // weights, and with 48 operand columns a workgroup of one row tile moves three operand
      // bytes per weight byte.  Measured: a CU sustains 58 GB/s on this access pattern whether
      // one workgroup or three share it.
      const int per_cu = ceil_div(wgs, mc.cus);
      const double wg_bytes = (double)rt * kts * 1024.0 + kts * x_per_kt;
      const double t_cu = per_cu * wg_bytes / mc.cu_bytes_per_us;
      // T_mem, level 2: the weights from HBM; fewer workgroups than CUs cannot draw the full rate
      const double cover = std::min(1.0, (double)wgs / mc.cus);
      const double t_hbm = W / (mc.stream_bytes_per_us * std::sqrt(cover));
      // epilogue: the four waves' partial tiles meet in LDS two row tiles at a time (one at a
      // time for an odd count), one round after the other, for every workgroup a CU runs
      const int rounds = rt % 2 == 0 ? rt / 2 : rt;
      const double t_epi = mc.skinny_round_us * rounds * per_cu;
      // partial sums: written per slice and read once more by the consumer, a norm kernel of one
      // workgroup per sequence that runs at an eighth of the streaming rate at best
      const double fold = slices > 1 ? slices * (double)n_tiles * 16.0 * nseq * 4.0 * 2.0 / (mc.hbm_bytes_per_us / 8.0) : 0.0;
      const double total = std::max(t_cu, t_hbm) + t_epi + fold + mc.skinny_launch_us;
      if (total < best.t_us * 0.999) {
        best.rt = rt; best.k_slices = slices; best.kts_per_split = kts; best.workgroups = wgs;
        best.t_mem_us = t_hbm; best.t_operand_us = t_cu; best.t_us = total;
      }
    }
  }
  return best;
}

SmallGemmPlan plan_small_gemm(const Machine& mc, int epi, int n_tiles, int KT, int col_tiles, int xt) {
  static const int tiles[3][5][2] = {{{8, 2}, {8, 4}}, {{1, 2}, {2, 2}, {4, 2}, {2, 4}, {4, 4}}, {{2, 2}, {4, 2}, {4, 4}, {6, 4}, {8, 4}}};
  SmallGemmPlan best{};
  best.t_us = 1e30;
  for (const auto& t : tiles[epi]) {
    const int nt = t[0], ct = t[1];
    if (!nt) continue;
    const int wgs = ceil_div(n_tiles, nt) * ceil_div(col_tiles, ct), rounds = ceil_div(wgs, mc.cus);
    const double bytes = (double)KT * (nt + ct * xt) * 1024.0;
    // what the busiest CU pulls out of L2 (a loads-only kernel reaches 100 - 120 GB/s per CU, these 55 - 90),
    // the matrix-core time, the weights from HBM; an epilogue per workgroup; launch
    const double t_cu = rounds * bytes / 100e3;
    const double t_mfma = (double)rounds * KT * xt * nt * ct / 4 * 16 / 2200.0;
    // (Every round starts cold streams anew.  A slope, not a step at the second round: it has to tell one round from
    // two and two from ten.  Every tile forced in turn at 55 prompt shapes (0.6B .. 8B, bf16, binary16, bytes, 9 - 512 tokens):
    // the picks' GEMM time is 2.9 % above the best tiles' without the term, 2.1 % with it (any slope of 0.05 - 0.3), 2.8 - 3.3 %
    // with a step of 0.1 - 0.6.  gate|up of 4B, us and rounds by tile (rows / 16 x columns / 16): 24 tokens 2 x 2 38.6 in 5, 4 x 2
    // 40.8 in 3, 4 x 4 35.3 in 2, 6 x 4 28.2 in 1; 64 tokens 60.4 in 10, 55.9 in 5, 46.0 in 3, 42.8 in 2.)
    const double t_hbm = (double)n_tiles * KT * 1024.0 / mc.hbm_bytes_per_us * (1.0 + 0.1 * (rounds - 1));
    const double total = std::max(std::max(t_cu, t_mfma), t_hbm) + 0.15 * nt * ct / 2 * rounds + 3.0;
    if (total < best.t_us) {
      best.nt = nt; best.ct = ct; best.workgroups = wgs; best.t_us = total;
    }
  }
  return best;
}

}  // namespace nnc
