// Prompt GEMMs of short blocks (two 16-bit pieces per activation), where every kernel of a layer is
// bound by latency and by what one CU pulls out of L2, not by the matrix cores.
//
// Five kernels per layer instead of eight:
//   q|k|v GEMM + per-head QK norm + rotary embedding + cache append   (k_gemm_small<SEPI_QKV>)
//   attention                                    (k_attn_small; k_attn_prefill for larger launches)
//   output projection + residual + operand of the next GEMM            (k_gemm_small<SEPI_RESID>)
//   gate|up GEMM + SwiGLU                                              (k_gemm_small<SEPI_SWIGLU>)
//   down projection + residual + operand of the next GEMM              (k_gemm_small<SEPI_RESID>)
// The RMSNorm between a residual projection and the GEMM it feeds needs no kernel: the projection's
// epilogue writes gain * x as the next operand and, per row block and token, the sum of x^2; the
// next GEMM multiplies its outputs by 1 / rms, which is exact because the matmul is linear.
// (binary16 models: an un-normalised row may leave the format's range, so there the norm kernel stays.)
#include "nnc_ahead.h"
#include "nnc_half.h"
#include "nnc_internal.h"
#include "nnc_lanes.h"

namespace nnc {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A workgroup owns NT row tiles x CT operand column tiles (CT / 2 token tiles); its four waves take
// the k tiles round-robin and meet in LDS once, after the loop.  No LDS staging and no barrier in
// the loop: both operands lie in fragment order in memory, a wave's load is 1 KiB contiguous, and
// with two register sets of U k tiles a workgroup keeps 4 U (NT + CT) KiB in flight, which is what
// bounds a launch this short.
// AHEAD: it touches the next GEMM's weights too (not for bytes, nor where a launch has only one or two token tiles).
template <int EPI, int NT, int CT, int U, class HF, bool AHEAD>
__global__ __launch_bounds__(256) void k_gemm_small(SmallGemmArgs a) {
  constexpr bool W8 = HF::kW8;      // byte weights: two operand k tiles per weight tile
  constexpr int XT = W8 ? 2 : 1;
  constexpr int QT = CT / 2;        // token tiles
  constexpr int NTOK = QT * 16, PARTS = 256 / NTOK;
  __shared__ float red[4][NT * QT][256];
  __shared__ float sq[PARTS][NTOK];
  __shared__ float sqr[4][NTOK];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int c16 = lane & 15, g = lane >> 4;
  // Consecutive workgroups go to the 8 XCDs in turn: all column blocks of a row block run on one
  // XCD, one after the other, so its L2 serves the weights to all but the first.
  const int gy = (a.t_tiles + CT - 1) / CT, gx = (a.n_tiles + NT - 1) / NT;
  const int slot_ = blockIdx.x >> 3;
  const int bx = (slot_ / gy) * 8 + (blockIdx.x & 7), by = slot_ % gy;
  if (bx >= gx) return;
  const int nt0 = bx * NT, ct0 = by * CT, KT = a.KT;

  // 1 / rms of this block's tokens: each thread adds a share of the producers' sums of squares
  // (fixed order); the loads are in flight while the k loop runs
  float ssum = 0.f;
  if (a.ssq) {
    const float* p = a.ssq + (size_t)ct0 * 8 + tid % NTOK;
    for (int b = tid / NTOK; b < a.ssq_blocks; b += PARTS) ssum += p[(size_t)b * a.ssq_stride];
  }

  // what the epilogue adds or multiplies by: loaded before the loop, so that the end of the kernel
  // (a chain of short dependent steps) waits for no memory
  const int nts = min(NT, a.n_tiles - nt0), cts = min(CT, a.t_tiles - ct0);
  const int tt0 = by * QT;      // first token tile
  const int QTV = cts / 2;      // token tiles that exist
  constexpr int NRES = EPI == SEPI_RESID ? (NT * QT + 3) / 4 : 1, NROT = EPI == SEPI_QKV ? QT : 1;
  f32x4 res[NRES], gn[NRES];        // RESID: residual rows and gains of this wave's tiles
  f32x4 ga, gb, cs[NROT][2];        // QKV: gains of this lane's dimensions, rotary factors of its tokens
  if constexpr (EPI == SEPI_RESID) {
#pragma unroll
    for (int n = 0; n < NRES; ++n) {
      const int o = min(wave + 4 * n, NT * QT - 1), i = min(o / QT, nts - 1), q = min(o % QT, QTV - 1);
      const int t = min((tt0 + q) * 16 + c16, a.n_tokens - 1), k0 = (nt0 + i) * 16 + g * 4;
      res[n] = *reinterpret_cast<const f32x4*>(a.x + (size_t)t * a.H + k0);
      gn[n] = a.gain ? *reinterpret_cast<const f32x4*>(a.gain + k0) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  if constexpr (EPI == SEPI_QKV) {
    const float* gp = (bx < a.nq ? a.gq : a.gk) + wave * 16 + g * 4;
    ga = *reinterpret_cast<const f32x4*>(gp);
    gb = *reinterpret_cast<const f32x4*>(gp + 64);
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const uint32_t pos = a.pos0 + (uint32_t)min((tt0 + q) * 16 + c16, a.n_tokens - 1);
      const f32x4* rp = reinterpret_cast<const f32x4*>(a.rope + (size_t)pos * 64 + wave * 16 + g * 4);
      cs[q][0] = rp[0];
      cs[q][1] = rp[1];
    }
  }

  f32x4 acc[NT][CT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const u32x4* __restrict__ Wv = static_cast<const u32x4*>(a.Wp);
  const u32x4* __restrict__ Xv = static_cast<const u32x4*>(a.Xf);
  // buffer descriptors over this block's tiles: per-lane offset fixed, scalar offset per tile (tiles
  // past the edge repeat the last one; their results are never stored)
  const __amdgpu_buffer_rsrc_t wres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(Wv + (size_t)nt0 * KT * 64), 0, nts * KT * 1024, 0x00020000);
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(Xv + (size_t)ct0 * KT * XT * 64), 0, cts * KT * XT * 1024, 0x00020000);
  const uint32_t voff = (uint32_t)lane * 16u;
  const int n_mine = wave < KT ? (KT - wave + 3) >> 2 : 0;  // this wave's k tiles: wave, wave + 4, ...
  const int last_kt = wave + 4 * (n_mine - 1);
  u32x4 avA[U][NT], bvA[U][XT * CT], avB[U][NT], bvB[U][XT * CT];
  auto load_tile = [&](int kt, u32x4(&av)[NT], u32x4(&bv)[XT * CT]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
      av[i] = __builtin_amdgcn_raw_buffer_load_b128(wres, voff, (min(i, nts - 1) * KT + kt) * 1024, 0);
#pragma unroll
    for (int x = 0; x < XT; ++x)
#pragma unroll
      for (int j = 0; j < CT; ++j)
        bv[x * CT + j] =
            __builtin_amdgcn_raw_buffer_load_b128(xres, voff, (min(j, cts - 1) * KT * XT + kt * XT + x) * 1024, 0);
  };
  auto load_group = [&](int t0, u32x4(&av)[U][NT], u32x4(&bv)[U][XT * CT]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) load_tile(min(wave + 4 * (t0 + u), last_kt), av[u], bv[u]);
  };
  auto mma_tile = [&](const u32x4(&av)[NT], const u32x4(&bv)[XT * CT]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if constexpr (W8) {
        const u32x4 a0 = HF::widen8(av[i][0], av[i][1]), a1 = HF::widen8(av[i][2], av[i][3]);
#pragma unroll
        for (int j = 0; j < CT; ++j) {
          acc[i][j] = HF::mfma(a0, bv[j], acc[i][j]);
          acc[i][j] = HF::mfma(a1, bv[CT + j], acc[i][j]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = HF::mfma(av[i], bv[j], acc[i][j]);
      }
    }
  };
  auto mma_group = [&](const u32x4(&av)[U][NT], const u32x4(&bv)[U][XT * CT]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) mma_tile(av[u], bv[u]);
  };
  const int n_groups = n_mine / U;
  if (n_groups > 0) load_group(0, avA, bvA);
  Ahead<SMALL_AHEAD> ahead;
  if constexpr (AHEAD) ahead.prepare(a.ahead, blockIdx.x, a.wgs);
  if (n_groups > 0) {
    // (scheduling barriers: the next set's loads are issued before the products on the current one)
    for (int gi = 0;;) {
      load_group((gi + 1) * U, avB, bvB);
      __builtin_amdgcn_sched_barrier(0);
      mma_group(avA, bvA);
      __builtin_amdgcn_sched_barrier(0);
      if (++gi >= n_groups) break;
      load_group((gi + 1) * U, avA, bvA);
      __builtin_amdgcn_sched_barrier(0);
      mma_group(avB, bvB);
      __builtin_amdgcn_sched_barrier(0);
      if (++gi >= n_groups) break;
    }
  }
  for (int t = n_groups * U; t < n_mine; ++t) {
    load_tile(wave + 4 * t, avA[0], bvA[0]);
    mma_tile(avA[0], bvA[0]);
  }

  if constexpr (AHEAD) ahead.issue(a.ahead);  // in flight during the epilogue

  // the two pieces of a token are added in the wave, the four waves' sums in LDS (fixed order)
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      f32x4 v = acc[i][2 * q];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += acc[i][2 * q + 1][e];
      *reinterpret_cast<f32x4*>(&red[wave][i * QT + q][lane * 4]) = v;
    }
  if (a.ssq) sq[tid / NTOK][tid % NTOK] = ssum;
  __syncthreads();
  auto total = [&](int i, int q) __attribute__((always_inline)) {
    f32x4 v = *reinterpret_cast<const f32x4*>(&red[0][i * QT + q][lane * 4]);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f32x4 o = *reinterpret_cast<const f32x4*>(&red[w][i * QT + q][lane * 4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += o[e];
    }
    if constexpr (W8) {
      const float4 sc = *reinterpret_cast<const float4*>(a.wscale + (size_t)min(nt0 + i, a.n_tiles - 1) * 16 + g * 4);
      v[0] *= sc.x; v[1] *= sc.y; v[2] *= sc.z; v[3] *= sc.w;
    }
    return v;
  };
  // 1 / rms of this lane's token in token tile q
  auto rms = [&](int q) __attribute__((always_inline)) {
    if (!a.ssq) return 1.0f;
    float s = 0.f;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) s += sq[p][q * 16 + c16];
    return 1.0f / sqrtf(s / (float)a.H + a.eps);
  };

  if constexpr (EPI == SEPI_QKV) {
    static_assert(EPI != SEPI_QKV || NT == 8, "one head per row block");
    // wave w holds rows w * 16 .. + 15 and their rotary partners 64 rows further
    const int hh = bx, nq = a.nq, nkv = a.nkv;
    const bool is_v = hh >= nq + nkv;
    f32x4 lo[QT], hi[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const float r = rms(q);
      lo[q] = total(wave, q);
      hi[q] = total(wave + 4, q);
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[q][e] *= r;
        hi[q][e] *= r;
        ss += lo[q][e] * lo[q][e] + hi[q][e] * hi[q][e];
      }
      ss = col4_sum(ss);
      if (g == 0) sqr[wave][q * 16 + c16] = ss;
    }
    __syncthreads();
    const int i0 = wave * 16 + g * 4;  // first of the four head dimensions of `lo`
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int t = (tt0 + q) * 16 + c16;
      if (q >= QTV || t >= a.n_tokens) continue;
      const uint32_t pos = a.pos0 + (uint32_t)t;
      if (!is_v) {
        const float ss = (sqr[0][q * 16 + c16] + sqr[1][q * 16 + c16]) + (sqr[2][q * 16 + c16] + sqr[3][q * 16 + c16]);
        const float r = 1.0f / sqrtf(ss * (1.0f / 128.0f) + a.eps);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = lo[q][e] * r * ga[e], y = hi[q][e] * r * gb[e];
          const float c = cs[q][e / 2][e % 2 * 2], sn = cs[q][e / 2][e % 2 * 2 + 1];
          lo[q][e] = x * c - y * sn;
          hi[q][e] = y * c + x * sn;
        }
      }
      if (hh < nq) {
        float* dst = a.q + (size_t)t * a.ldq + (size_t)hh * 128 + i0;
        *reinterpret_cast<f32x4*>(dst) = lo[q];
        *reinterpret_cast<f32x4*>(dst + 64) = hi[q];
        continue;
      }
      uint32_t bl[4], bh[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bl[e] = HF::bits(lo[q][e]);
        bh[e] = HF::bits(hi[q][e]);
      }
      const int kvh = is_v ? hh - nq - nkv : hh - nq;
      uint16_t* row = static_cast<uint16_t*>(is_v ? a.vc : a.kc) + (((size_t)a.slot * nkv + kvh) * a.max_seq + pos) * 128 + i0;
      *reinterpret_cast<uint2*>(row) = make_uint2(bl[0] | (bl[1] << 16), bl[2] | (bl[3] << 16));
      *reinterpret_cast<uint2*>(row + 64) = make_uint2(bh[0] | (bh[1] << 16), bh[2] | (bh[3] << 16));
      if (is_v) {  // and the transposed copy [kv head][dim][position] the attention kernel reads
        uint16_t* vt = static_cast<uint16_t*>(a.vt) + ((size_t)kvh * 128 + i0) * a.vt_stride + pos;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vt[(size_t)e * a.vt_stride] = (uint16_t)bl[e];
          vt[(size_t)(64 + e) * a.vt_stride] = (uint16_t)bh[e];
        }
      }
    }
  } else if constexpr (EPI == SEPI_RESID) {
    // x += y; with a gain, gain * x as the next GEMM's operand and the row block's sums of squares
    float ssp[(NT * QT + 3) / 4];
#pragma unroll
    for (int n = 0; n < (NT * QT + 3) / 4; ++n) {
      const int o = wave + 4 * n;  // (row tile, token tile)
      ssp[n] = 0.f;
      if (NT * QT % 4 && o >= NT * QT) continue;
      const int i = o / QT, q = o % QT, nt = nt0 + i, t = (tt0 + q) * 16 + c16;
      if (i < nts && q < QTV && t < a.n_tokens) {
        f32x4 v = total(i, q);
        const int k0 = nt * 16 + g * 4;
        float* xp = a.x + (size_t)t * a.H + k0;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = res[n][e] + v[e];
        *reinterpret_cast<f32x4*>(xp) = v;
        if (a.gain) {
          const float h[4] = {v[0] * gn[n][0], v[1] * gn[n][1], v[2] * gn[n][2], v[3] * gn[n][3]};
          uint32_t pc[4][3];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            split_pieces<HF>(h[e], 2, pc[e]);
            ssp[n] += v[e] * v[e];
          }
          const int KTH = a.H / 32;
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const size_t el =
                (((size_t)((tt0 + q) * 2 + s) * KTH + (k0 >> 5)) * 64 + c16 + 16 * ((k0 & 31) >> 3)) * 8 + (k0 & 7);
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.Xn) + el) =
                make_uint2(pc[0][s] | (pc[1][s] << 16), pc[2][s] | (pc[3][s] << 16));
          }
        }
      }
    }
    if (a.gain) {
      __syncthreads();  // every wave has read its tiles: reuse red for the per-tile sums
      float* tile_sq = &red[0][0][0];
#pragma unroll
      for (int n = 0; n < (NT * QT + 3) / 4; ++n) {
        const int o = wave + 4 * n;
        if (NT * QT % 4 && o >= NT * QT) continue;
        const float s = col4_sum(ssp[n]);
        if (g == 0) tile_sq[o * 16 + c16] = s;
      }
      __syncthreads();
      if (tid < NTOK) {
        const int q = tid >> 4;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NT; ++i) s += tile_sq[(i * QT + q) * 16 + (tid & 15)];
        if (q < QTV) a.ssq_out[(size_t)bx * a.ssq_stride + (size_t)tt0 * 16 + tid] = s;
      }
    }
  } else {
    // row tiles come as (gate, up) pairs; feature tile = row tile / 2
    static_assert(EPI != SEPI_SWIGLU || NT % 2 == 0, "SwiGLU needs (gate, up) tile pairs");
    constexpr int PAIRS = NT / 2 * QT;
    const int FKT = a.n_tiles / 4;  // k tiles of the next GEMM
#pragma unroll
    for (int n = 0; n < (PAIRS + 3) / 4; ++n) {
      const int o = wave + 4 * n;
      if (PAIRS % 4 && o >= PAIRS) continue;
      const int i = o / QT * 2, q = o % QT, nt = nt0 + i, t = (tt0 + q) * 16 + c16;
      if (i >= nts || q >= QTV || t >= a.n_tokens) continue;
      const float r = rms(q);
      const f32x4 gate = total(i, q), up = total(i + 1, q);
      const int f0 = (nt >> 1) * 16 + g * 4;
      uint32_t pc[4][3];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float z = gate[e] * r;
        split_pieces<HF>(z / (1.0f + expf(-z)) * (up[e] * r), 2, pc[e]);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const size_t el = (((size_t)((tt0 + q) * 2 + s) * FKT + (f0 >> 5)) * 64 + c16 + 16 * ((f0 & 31) >> 3)) * 8 + (f0 & 7);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.packed_out) + el) =
            make_uint2(pc[0][s] | (pc[1][s] << 16), pc[2][s] | (pc[3][s] << 16));
      }
    }
  }
  if constexpr (AHEAD) ahead.done();
}

hipError_t launch_gemm_small(hipStream_t s, bool f16, int epi, const SmallGemmArgs& a, int nt, int ct) {
  if (a.n_tiles <= 0 || a.t_tiles <= 0 || a.t_tiles % 2 || a.KT <= 0 || a.n_tokens <= 0 || a.n_tokens > a.t_tiles * 8 ||
      (f16 && (a.wscale || a.gain || a.ssq)))
    return hipErrorInvalidValue;
  if (a.ssq && (a.ssq_blocks <= 0 || a.ssq_stride < a.t_tiles * 8)) return hipErrorInvalidValue;
  if (epi == SEPI_QKV && (nt != 8 || a.n_tiles != (a.nq + 2 * a.nkv) * 8 || a.pos0 + (uint32_t)a.n_tokens > a.max_seq))
    return hipErrorInvalidValue;
  if (epi == SEPI_SWIGLU && (a.n_tiles % 4 || nt % 2)) return hipErrorInvalidValue;
  if (epi == SEPI_RESID && (a.n_tiles * 16 != a.H || (a.gain && (!a.Xn || !a.ssq_out || a.ssq_stride < a.t_tiles * 8))))
    return hipErrorInvalidValue;
  const int gx = (a.n_tiles + nt - 1) / nt, gy = (a.t_tiles + ct - 1) / ct;
  const unsigned grid = (unsigned)((gx + 7) / 8 * 8 * gy);
  SmallGemmArgs b = a;
  b.wgs = (int)grid;
  const bool ahead = a.ahead.W != nullptr;
#define SG_HF(E, NT, CT, U)                                                             \
  do {                                                                                  \
    if (a.wscale) k_gemm_small<E, NT, CT, 2, Bf16W8, false><<<grid, 256, 0, s>>>(b);    \
    else if (f16 && ahead) k_gemm_small<E, NT, CT, U, Fp16, true><<<grid, 256, 0, s>>>(b); \
    else if (f16) k_gemm_small<E, NT, CT, U, Fp16, false><<<grid, 256, 0, s>>>(b);      \
    else if (ahead) k_gemm_small<E, NT, CT, U, Bf16, true><<<grid, 256, 0, s>>>(b);     \
    else k_gemm_small<E, NT, CT, U, Bf16, false><<<grid, 256, 0, s>>>(b);               \
    return hipGetLastError();                                                           \
  } while (0)
#define SG(E, NT, CT, U) \
  if (epi == E && nt == NT && ct == CT) SG_HF(E, NT, CT, U)
  SG(SEPI_QKV, 8, 2, 2);
  SG(SEPI_QKV, 8, 4, 2);
  SG(SEPI_RESID, 1, 2, 4);
  SG(SEPI_RESID, 2, 2, 4);
  SG(SEPI_RESID, 4, 2, 4);
  SG(SEPI_RESID, 2, 4, 4);
  SG(SEPI_RESID, 4, 4, 2);
  SG(SEPI_SWIGLU, 2, 2, 4);
  SG(SEPI_SWIGLU, 4, 2, 4);
  SG(SEPI_SWIGLU, 4, 4, 2);
  SG(SEPI_SWIGLU, 6, 4, 2);
  SG(SEPI_SWIGLU, 8, 4, 2);
#undef SG
#undef SG_HF
  return hipErrorInvalidValue;
}

// x[t] = E[tokens[t]] and, with a gain, gain * x as two pieces in fragment order and the row's sum of
// squares (one block per row: ssq[t]); the first layer's counterpart of the residual epilogue.
template <class HF>
__global__ __launch_bounds__(256) void k_embed_rows_pack(const void* __restrict__ Ep, int H, const int32_t* __restrict__ tokens,
                                                         const float* __restrict__ gain, float* __restrict__ x,
                                                         uint4* __restrict__ Xn, float* __restrict__ ssq) {
  __shared__ float sm[4];
  const int t = blockIdx.x, r = tokens[t], KT = H / 32;
  const uint4* row = static_cast<const uint4*>(Ep) + ((size_t)(r >> 4) * KT) * 64 + (r & 15);
  uint4* out = Xn + (size_t)(t >> 4) * 2 * KT * 64 + (t & 15);
  float ss = 0.f;
  for (int kg = threadIdx.x; kg < H / 8; kg += 256) {
    const size_t at = (size_t)(kg >> 2) * 64 + 16 * (kg & 3);
    const uint4 w = row[at];
    const float v[8] = {HF::lo(w.x), HF::hi(w.x), HF::lo(w.y), HF::hi(w.y), HF::lo(w.z), HF::hi(w.z), HF::lo(w.w), HF::hi(w.w)};
    float* dst = x + (size_t)t * H + kg * 8;
    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
    const float4 g0 = *reinterpret_cast<const float4*>(gain + kg * 8), g1 = *reinterpret_cast<const float4*>(gain + kg * 8 + 4);
    const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    uint32_t pc[8][3];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      ss += v[e] * v[e];
      split_pieces<HF>(v[e] * gg[e], 2, pc[e]);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
      out[(size_t)s * KT * 64 + at] = uint4{pc[0][s] | (pc[1][s] << 16), pc[2][s] | (pc[3][s] << 16), pc[4][s] | (pc[5][s] << 16),
                                            pc[6][s] | (pc[7][s] << 16)};
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) ssq[t] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

hipError_t launch_embed_rows_pack(hipStream_t s, const void* Ep, int H, const int32_t* tokens_dev, int n, const float* gain,
                                  float* x, void* Xn, float* ssq) {
  if (H % 32 || n <= 0) return hipErrorInvalidValue;
  k_embed_rows_pack<Bf16><<<n, 256, 0, s>>>(Ep, H, tokens_dev, gain, x, static_cast<uint4*>(Xn), ssq);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// causal attention of short blocks
// ---------------------------------------------------------------------------
// The arithmetic of k_attn_prefill (both products transposed, base-2 softmax with a running bound of the
// maximum, weights and queries in two pieces), for launches too small to fill the chip with 64-token
// workgroups: a workgroup takes 16 tokens x GH query heads of one kv head and its four waves take the
// 32-position chunks round-robin, merging their (maximum, sum, value sums) in LDS at the end.  Four times
// the workgroups, a quarter of the serial chunks (each about 1.2 us of dependent products and softmax), no
// barrier in the loop; the K and V^T fragments come straight from L2, the next chunk's K and this chunk's V^T in
// flight while the products run.
template <int GH, class HF>
__global__ __launch_bounds__(256) void k_attn_small(const float* __restrict__ qkv, int nq, int nkv,
                                                    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vt,
                                                    uint32_t S, uint32_t slot, uint32_t max_seq, uint32_t pos0, int n,
                                                    void* __restrict__ Of) {
  __shared__ f32x4 red[4][GH][8][64];
  __shared__ float smm[4][GH][16], sml[4][GH][16];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int c16 = lane & 15, g = lane >> 4;
  const int G = nq / nkv;
  const int kvh = blockIdx.y / (G / GH), head0 = kvh * G + (blockIdx.y % (G / GH)) * GH;
  const int tq = (n + 15) / 16 - 1 - (int)blockIdx.x;  // token tile, longest first (gridDim would be a load of its own)
  const int ld = (nq + 2 * nkv) * 128;
  const int t = min(tq * 16 + c16, n - 1);  // rows past the prompt repeat the last token (never stored)
  const uint32_t p = pos0 + (uint32_t)t, p_first = pos0 + (uint32_t)tq * 16, p_last = pos0 + (uint32_t)min(tq * 16 + 15, n - 1);

  const uint16_t* kbase = kc + ((size_t)slot * nkv + kvh) * max_seq * 128;
  const uint16_t* vbase = vt + (size_t)kvh * 128 * S;
  const uint32_t r4 = (uint32_t)((c16 >> 2) * 8 + (c16 & 3));  // K row of tile a for A-operand row c16; tile b: + 4
  u32x4 ka[4], kb[4], vf[8];
  auto load_k = [&](uint32_t kv0) __attribute__((always_inline)) {  // rows past the cache's end repeat its last (masked)
    const uint16_t* ra = kbase + (size_t)min(kv0 + r4, max_seq - 1) * 128 + g * 8;
    const uint16_t* rb = kbase + (size_t)min(kv0 + r4 + 4, max_seq - 1) * 128 + g * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      ka[ks] = *reinterpret_cast<const u32x4*>(ra + ks * 32);
      kb[ks] = *reinterpret_cast<const u32x4*>(rb + ks * 32);
    }
  };
  auto load_v = [&](uint32_t kv0) __attribute__((always_inline)) {  // kv0 + 31 < S
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      vf[dt] = *reinterpret_cast<const u32x4*>(vbase + (size_t)(dt * 16 + c16) * S + kv0 + g * 8);
  };
  uint32_t kv0 = (uint32_t)wave * 32;
  if (kv0 <= p_last) load_k(kv0);

  u32x4 qf[GH][4][2];
#pragma unroll
  for (int h = 0; h < GH; ++h)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const float* src = qkv + (size_t)t * ld + (size_t)(head0 + h) * 128 + ks * 32 + g * 8;
      const float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 4);
      float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
      for (int pc = 0; pc < 2; ++pc) {
        uint32_t b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          b[e] = HF::pack2(v[2 * e], v[2 * e + 1]);
          v[2 * e] -= HF::lo(b[e]);
          v[2 * e + 1] -= HF::hi(b[e]);
        }
        qf[h][ks][pc] = u32x4{b[0], b[1], b[2], b[3]};
      }
    }

  f32x4 acc[GH][8], lacc[GH];
  float mrun[GH];
#pragma unroll
  for (int h = 0; h < GH; ++h) {
    mrun[h] = -INFINITY;
    lacc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[h][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const u32x4 ones = u32x4{HF::kOnes2, HF::kOnes2, HF::kOnes2, HF::kOnes2};
  for (; kv0 <= p_last; kv0 += 128) {
    load_v(kv0);
    f32x4 sa[GH], sb[GH];
#pragma unroll
    for (int h = 0; h < GH; ++h) {
      sa[h] = sb[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int pc = 0; pc < 2; ++pc) {
          sa[h] = HF::mfma(ka[ks], qf[h][ks][pc], sa[h]);
          sb[h] = HF::mfma(kb[ks], qf[h][ks][pc], sb[h]);
        }
    }
    if (kv0 + 128 <= p_last) load_k(kv0 + 128);
    u32x4 pf[GH][2];
#pragma unroll
    for (int h = 0; h < GH; ++h) {
      float sc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) sc[i] = i < 4 ? sa[h][i] : sb[h][i - 4];
      if (kv0 + 31 > p_first) {  // the chunk reaches past the tile's first token: mask per lane
#pragma unroll
        for (int i = 0; i < 8; ++i) sc[i] = kv0 + g * 8 + i <= p ? sc[i] : -INFINITY;
      }
      constexpr float kScale = 0.12751743082459868f;  // log2(e) / sqrt(128)
      float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7]))) * kScale;
      if (__any(mx > mrun[h])) {
        const float mn = fmaxf(mrun[h], col4_max(mx));
        // a token that sees nothing of this wave's chunks yet keeps maximum -inf and sums of zero
        const float alpha = __builtin_amdgcn_exp2f(mrun[h] - (mn == -INFINITY ? 0.f : mn));
        mrun[h] = mn;
#pragma unroll
        for (int e = 0; e < 4; ++e) lacc[h][e] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[h][dt][e] *= alpha;
      }
      const float mn = mrun[h] == -INFINITY ? 0.f : mrun[h];
      uint32_t pw[2][4];
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        float w0 = __builtin_amdgcn_exp2f(fmaf(sc[i], kScale, -mn));
        float w1 = __builtin_amdgcn_exp2f(fmaf(sc[i + 1], kScale, -mn));
        pw[0][i / 2] = HF::pack2(w0, w1);
        w0 -= HF::lo(pw[0][i / 2]);
        w1 -= HF::hi(pw[0][i / 2]);
        pw[1][i / 2] = HF::pack2(w0, w1);
      }
#pragma unroll
      for (int pc = 0; pc < 2; ++pc) {
        pf[h][pc] = u32x4{pw[pc][0], pw[pc][1], pw[pc][2], pw[pc][3]};
        lacc[h] = HF::mfma(ones, pf[h][pc], lacc[h]);
      }
    }
    if (kv0 + 31 > p_last) {
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int e = 0; e < 4; ++e) vf[dt][e] &= column_mask((int)p_last - (int)(kv0 + g * 8), e);
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int h = 0; h < GH; ++h)
#pragma unroll
        for (int pc = 0; pc < 2; ++pc) acc[h][dt] = HF::mfma(vf[dt], pf[h][pc], acc[h][dt]);
  }

  // merge of the four waves (fixed order)
#pragma unroll
  for (int h = 0; h < GH; ++h) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) red[wave][h][dt][lane] = acc[h][dt];
    if (g == 0) {
      smm[wave][h][c16] = mrun[h];
      sml[wave][h][c16] = lacc[h][0];
    }
  }
  __syncthreads();
  if (tq * 16 + c16 >= n) return;
  const int KTQ = nq * 4;
#pragma unroll
  for (int h = 0; h < GH; ++h) {
    float M = smm[0][h][c16], f[4], l = 0.f;
#pragma unroll
    for (int w = 1; w < 4; ++w) M = fmaxf(M, smm[w][h][c16]);  // finite: wave 0 sees position 0
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      f[w] = __builtin_amdgcn_exp2f(smm[w][h][c16] - M);
      l += f[w] * sml[w][h][c16];
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int d2 = 0; d2 < 2; ++d2) {
      const int dt = wave * 2 + d2, k0 = (head0 + h) * 128 + dt * 16 + g * 4;
      float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const f32x4 o = red[w][h][dt][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += f[w] * o[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= inv;
#pragma unroll
      for (int pc = 0; pc < 2; ++pc) {
        const uint32_t b0 = HF::pack2(v[0], v[1]), b1 = HF::pack2(v[2], v[3]);
        v[0] -= HF::lo(b0);
        v[1] -= HF::hi(b0);
        v[2] -= HF::lo(b1);
        v[3] -= HF::hi(b1);
        const size_t el = (((size_t)(tq * 2 + pc) * KTQ + (k0 >> 5)) * 64 + c16 + 16 * ((k0 & 31) >> 3)) * 8 + (k0 & 7);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(Of) + el) = make_uint2(b0, b1);
      }
    }
  }
}

// Query heads per workgroup for a block, 0 where k_attn_prefill is the better kernel: as long as one
// workgroup per CU holds the launch, first with one head each, then with two.  Beyond, the fragment loads
// of the extra workgroups cost more than the shorter chains save.  us per launch, k_attn_prefill / one
// head / two heads: 16 heads, 128 tokens 7.9 / 5.3 / 7.0; 256 10.6 / 7.4 / 9.1; 333 12.1 / 13.6 / 10.2; 512 16.9 / 19 / 13;
// 32 heads, 128 tokens 7.2 / 5.4 / 7.2; 256 11.4 / 12.6 / 10.0; 333 13.4 / 18.7 / 17.7.  The line does not move with the
// position the block starts at (timed by events, which add 2 us): at 256, 1024 and 4000 earlier positions 16
// heads, 128 tokens 16.2 / 11.4 / 13.4, 34.0 / 21.7 / 23.5, 132 / 63 / 65; 400 tokens 22.3 / 24.3 / 18.2, 40.5 / 45.1 / 28.7,
// 137 / 128 / 72; 32 heads, 256 tokens 20.7 / 21.5 / 15.8, 44.2 / 43.1 / 27.8, 138 / 131 / 74.
int attn_small_heads(int nq, int nkv, int n, int n_cus) {
  const int tt = (n + 15) / 16;
  if (tt * nq <= n_cus) return 1;
  return nq / nkv % 2 == 0 && tt * (nq / 2) <= n_cus ? 2 : 0;
}

hipError_t launch_attn_small(hipStream_t s, bool f16, const float* qkv, int nq, int nkv, const void* kc, const void* vt,
                             uint32_t S, uint32_t slot, uint32_t max_seq, uint32_t pos0, int n, void* Of, int n_cus) {
  if (n <= 0 || nkv <= 0 || nq % nkv || S % 32 || pos0 + (uint32_t)n > max_seq || max_seq > S) return hipErrorInvalidValue;
  const int GH = attn_small_heads(nq, nkv, n, n_cus) == 2 ? 2 : 1;
  dim3 grid((n + 15) / 16, nq / GH);
  const uint16_t *k = static_cast<const uint16_t*>(kc), *v = static_cast<const uint16_t*>(vt);
#define AS(GHV, HF) k_attn_small<GHV, HF><<<grid, 256, 0, s>>>(qkv, nq, nkv, k, v, S, slot, max_seq, pos0, n, Of)
  if (GH == 2) {
    if (f16) AS(2, Fp16);
    else AS(2, Bf16);
  } else {
    if (f16) AS(1, Fp16);
    else AS(1, Bf16);
  }
#undef AS
  return hipGetLastError();
}

}  // namespace nnc
