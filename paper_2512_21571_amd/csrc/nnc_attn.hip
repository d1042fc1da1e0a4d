// Causal attention of prompt blocks on 32 x 32 matrix-core products.
//
// A wave owns 32 prompt tokens of one query head, a workgroup four waves = 128 consecutive tokens, and walks the
// positions in chunks of CH.  Both products run transposed, so that no operand is shuffled between them:
//   S^T = K Q^T    A = 32 cached K rows (8 k steps of 16 dims), B = the wave's 32 query rows.  D holds, per lane, one token
//                  (column lane % 32) and 16 positions; the K rows are dealt to the A rows so that these are
//                  positions 8 h .. 8 h + 7 and 16 + 8 h .. + 7 of the 32 (h = lane / 32).
//   O^T = V^T P^T  A = 32 head dims x 16 positions from the transposed V copy, B = the lane's own 8 weights.
// Against 16 x 16 products with 16 tokens per wave (k_attn_prefill) a fragment read from LDS feeds twice the work
// and the fixed latencies of a chunk (barrier, fragment reads, the chain product - maximum - exponential - product) are
// paid once per CH instead of once per 32 positions and for twice the tokens.
//
// The K rows and V^T rows of a chunk are the same for the four waves: copied once, global -> LDS directly, one chunk
// ahead, double-buffered.  LDS keeps whole rows (a wave's copy is coalesced and takes no vector instruction: scalar base plus
// a per-lane offset that does not change); the 16-byte groups of a row are permuted by an exclusive or with the row's
// number, so that the lanes of a fragment read, which stand in different rows, hit different banks.  (Through registers
// the copy's address arithmetic, waits and stores cost a third of the kernel: 8B, 4080 tokens, 195 us, 131 without any copy.)
//
// SPLIT: the positions of a token block are dealt to gridDim.y workgroups, which leave un-normalised sums, maxima
// and row sums in `part`; k_attn_merge adds them up in split order.
//
// What bounds it: with two workgroups per CU a chunk of 64 positions x 128 tokens takes 1.3 us, the sum rather than
// the maximum of its parts (variants that leave one out: 40 us of 170 for the copies, 35 for the exponentials, 45 for the
// fragment reads, at 8B and 4080 tokens); the matrix cores are busy 38 %.  Measured, us per launch, k_attn_prefill / this: one
// piece, 32 heads: 584 tokens 24.2 / 20.1, 1024 40.2 / 30.8, 2032 (4B) 79.9 / 57.5, 4080 198 / 169; 16 heads: 544 19.4 / 17.9,
// 1024 31.8 / 28.3, 2032 70.5 / 50.5, 4080 149 / 102.  Two pieces, behind earlier positions, the better of k_attn_prefill and
// k_attn_small / this: 32 heads, 333 tokens behind 2048 80.1 / 55.9 (4 workgroups over the positions), 64 behind 2048 37.2 /
// 23.8 (8), 512 behind 3072 118 / 79.5 (4); 16 heads, 333 behind 2048 44.5 / 37.0 (4), 100 behind 3072 51.9 / 28.5 (8).
// Not taken: ones-products or unpacked sums for the row sums (179, 177 against 170), raised wave priority
// around the products (179), eight fragments of K in flight at once (spills).
#include "nnc_half.h"
#include "nnc_internal.h"
#include "nnc_lanes.h"

#include <type_traits>

namespace nnc {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int AB_TOKENS = 128;      // tokens per workgroup
constexpr int AB_REC = 132;         // floats per partial record: 128 sums, maximum, row sum

// LDS barrier that leaves global loads in flight
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c, Bf16*) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(Bf16::vec8, a), __builtin_bit_cast(Bf16::vec8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c, Fp16*) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(Fp16::vec8, a), __builtin_bit_cast(Fp16::vec8, b), c, 0, 0, 0);
}

// c + low + high of a packed pair
__device__ __forceinline__ float pair_sum(uint32_t w, float c, Bf16*) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(Bf16::vec2, w), __builtin_bit_cast(Bf16::vec2, Bf16::kOnes2), c, false);
}
__device__ __forceinline__ float pair_sum(uint32_t w, float c, Fp16*) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(Fp16::vec2, w), __builtin_bit_cast(Fp16::vec2, Fp16::kOnes2), c, false);
}

// The maximum of three as one v_maximum3.  It reads fresh matrix products, whose result needs 12 wait states before it may be
// read, and only the compiler puts those in: not inline assembly (v_max3 written so read two-piece scores after 3).  Not
// fmaxf either, which first quiets every operand with an instruction of its own.  A NaN score makes the maximum NaN; its
// token's weights and sums are NaN by the score itself.
__device__ __forceinline__ float max3(float x, float y, float z) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z);
}

}  // namespace

template <int PIECES, int CH, bool SPLIT, class HF>
__global__ __launch_bounds__(256, 2) void k_attn_block(const float* __restrict__ qkv, int nq, int nkv,
                                                       const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vt,
                                                       uint32_t S, uint32_t slot, uint32_t max_seq, uint32_t pos0, int n,
                                                       int half_blocks, int splits, void* __restrict__ Of, float* __restrict__ part) {
  constexpr int SUB = CH / 32;             // 32-position tiles per chunk
  constexpr int VG = CH / 8;               // 16-byte groups of a V^T row
  constexpr int VSH = VG == 8 ? 1 : 2;     // 256 bytes of LDS hold 1 << VSH rows
  constexpr uint32_t KB = CH * 256u, VB = 128u * VG * 16u;  // bytes per chunk
  __shared__ __attribute__((aligned(1024))) char Fs[2][KB + VB];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r32 = lane & 31, hf = lane >> 5;
  // Consecutive workgroups go to the 8 XCDs in turn: heads in the order that gives a kv head to one XCD (for 8 kv heads).
  // Token blocks: the longest first; where all workgroups are resident at once (half_blocks > 0) the second half of the
  // launch runs the other way, so that a CU's two workgroups add up to the same work.
  const int G = nq / nkv, hid = (int)blockIdx.x % nq, blk = (int)blockIdx.x / nq;
  const int kvh = hid % nkv, head = kvh * G + hid / nkv;
  const int NB = (n + AB_TOKENS - 1) / AB_TOKENS;
  const int tb = half_blocks > 0 && blk >= half_blocks ? blk - half_blocks : NB - 1 - blk;
  const int t0 = tb * AB_TOKENS + wave * 32;  // the wave's first token
  const bool active = t0 < n;
  const int ld = (nq + 2 * nkv) * 128;
  const int t = min(t0 + r32, n - 1);  // rows past the prompt repeat the last token (never stored)
  const uint32_t p = pos0 + (uint32_t)t;
  const uint32_t p_first = pos0 + (uint32_t)t0;
  const uint32_t p_last = pos0 + (uint32_t)min(t0 + 31, n - 1);
  const uint32_t p_last_wg = pos0 + (uint32_t)min(tb * AB_TOKENS + AB_TOKENS - 1, n - 1);
  uint32_t kv_begin = 0, kv_end = p_last_wg + 1;
  if constexpr (SPLIT) {
    const uint32_t chunks = p_last_wg / CH + 1, per = (chunks + splits - 1) / splits;
    kv_begin = min(blockIdx.y * per, chunks) * CH;
    kv_end = min(kv_end, kv_begin + per * CH);
  }

  // query fragments: lane (column r32 = token, hf) holds dims ks * 16 + hf * 8 .. + 7
  u32x4 qf[8][PIECES];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    const float* src = qkv + (size_t)t * ld + (size_t)head * 128 + ks * 16 + hf * 8;
    const float4 x0 = *reinterpret_cast<const float4*>(src), x1 = *reinterpret_cast<const float4*>(src + 4);
    float v[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
    for (int pc = 0; pc < PIECES; ++pc) {
      uint32_t b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        b[e] = HF::pack2(v[2 * e], v[2 * e + 1]);
        v[2 * e] -= HF::lo(b[e]);
        v[2 * e + 1] -= HF::hi(b[e]);
      }
      qf[ks][pc] = u32x4{b[0], b[1], b[2], b[3]};
    }
  }

  f32x16 acc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
  float mrun = -INFINITY, lrun = 0.f;  // lrun: this lane's share of its token's row sum (the other half of the positions: lane ^ 32)

  const uint16_t* kbase = kc + (((size_t)slot * nkv + kvh) * max_seq) * 128;
  const uint16_t* vbase = vt + (size_t)kvh * 128 * S;

  // Copy of a chunk: a wave's instruction takes 1 KiB of LDS, i.e. 4 K rows or 64 / VG V^T rows.
  typedef __attribute__((address_space(3))) void* lptr;
  constexpr int CK = CH / 16, CV = 128 * VG / 256;  // instructions per wave
  const uint32_t krow = (uint32_t)(wave * 4 + (lane >> 4)), kgrp = (uint32_t)(lane & 15) ^ (krow & 15);
  const uint32_t vrow = (uint32_t)(wave * (64 / VG) + lane / VG), vgrp = (uint32_t)(lane % VG) ^ ((vrow >> VSH) & (VG - 1));
  const uint32_t kvoff = krow * 256u + kgrp * 16u, vvoff = vrow * S * 2u + vgrp * 16u;
  // (inline assembly: the compiler would make every later LDS read wait for all copies; the waits are explicit)
  auto copy1 = [&](const char* base, uint32_t voff, uint32_t lds_addr) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(base)
                 : "memory", "m0");
  };
  auto copy = [&](uint32_t kv0, int buf) __attribute__((always_inline)) {  // kv0 a multiple of CH
    const uint32_t lk = (uint32_t)(size_t)(lptr)&Fs[buf][0] + (uint32_t)wave * 1024u, lv = lk + KB;
    const char* kb = reinterpret_cast<const char*>(kbase) + (size_t)kv0 * 256;
    const char* vb = reinterpret_cast<const char*>(vbase) + (size_t)kv0 * 2;
    if (kv0 + CH <= max_seq) {
#pragma unroll
      for (int j = 0; j < CK; ++j) copy1(kb + j * 4096, kvoff, lk + j * 4096u);
    } else {  // the cache ends inside the chunk: repeat its last row (those positions are masked)
#pragma unroll
      for (int j = 0; j < CK; ++j) copy1(kb, min(krow + 16u * j, max_seq - 1 - kv0) * 256u + kgrp * 16u, lk + j * 4096u);
    }
    if (kv0 + CH <= S) {
#pragma unroll
      for (int j = 0; j < CV; ++j) copy1(vb + (size_t)j * (256 / VG) * S * 2, vvoff, lv + j * 4096u);
    } else {  // likewise its last group
      const uint32_t off = vrow * S * 2u + min(vgrp * 16u, (S - 8 - kv0) * 2u);
#pragma unroll
      for (int j = 0; j < CV; ++j) copy1(vb + (size_t)j * (256 / VG) * S * 2, off, lv + j * 4096u);
    }
  };
  // byte offsets of this lane's fragment reads: K row of A row r32 (see the top), V^T row r32 of a dim tile
  const int qi = (r32 >> 3) * 4 + (r32 & 3), kpos = (qi >> 3) * 16 + ((r32 >> 2) & 1) * 8 + (qi & 7);
  const uint32_t koff = (uint32_t)(kpos * 256 + ((hf ^ (kpos & 15)) * 16));
  const uint32_t voff = KB + (uint32_t)(r32 * VG * 16 + ((hf ^ ((r32 >> VSH) & (VG - 1))) * 16));
  auto frag_k = [&](int buf, int s, int ks) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(&Fs[buf][(koff ^ (uint32_t)(ks * 32)) + (uint32_t)(s * 32 * 256)]);
  };
  auto frag_v = [&](int buf, int dt, int st) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(&Fs[buf][(voff ^ (uint32_t)(st * 32)) + (uint32_t)(dt * 32 * VG * 16)]);
  };

  // A chunk.  Fragment reads are issued well before the products that use them, and kept there by scheduling barriers:
  // left alone the compiler reads two fragments, waits for them, multiplies, and pays the LDS latency eight times.
  // DIAGONAL: the chunk reaches past the workgroup's first token, and may reach past the wave's.
  auto do_chunk = [&](auto diagonal, int buf, uint32_t kv0) __attribute__((always_inline)) {
    constexpr bool DIAGONAL = decltype(diagonal)::value;
    f32x16 sc[SUB];
    u32x4 vf[2][4];  // V^T fragments of two 16-position steps
    auto read_v = [&](int st, u32x4(&v)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) v[dt] = frag_v(buf, dt, st);
    };
    {
      u32x4 kf[3][2][SUB];  // K fragments of three pairs of k steps
      auto read_k = [&](int pr, u32x4(&v)[2][SUB]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int s = 0; s < SUB; ++s) v[q][s] = frag_k(buf, s, pr * 2 + q);
      };
#pragma unroll
      for (int pr = 0; pr < 3; ++pr) read_k(pr, kf[pr]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < SUB; ++s)
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[s][e] = 0.f;
#pragma unroll
      for (int pr = 0; pr < 4; ++pr) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int s = 0; s < SUB; ++s)
#pragma unroll
            for (int pc = 0; pc < PIECES; ++pc) sc[s] = mfma32(kf[pr % 3][q][s], qf[pr * 2 + q][pc], sc[s], (HF*)nullptr);
        __builtin_amdgcn_sched_barrier(0);
        if (pr == 0) read_k(3, kf[0]);
        if (pr == 2) read_v(0, vf[0]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (DIAGONAL && kv0 + CH - 1 > p_first) {  // mask per lane
#pragma unroll
      for (int s = 0; s < SUB; ++s)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          sc[s][e] = kv0 + s * 32 + (e >> 3) * 16 + hf * 8 + (e & 7) <= p ? sc[s][e] : -INFINITY;
    }
    // scores in units of log 2: exp(s / sqrt(128)) = exp2(s * log2(e) / sqrt(128))
    constexpr float kScale = 0.12751743082459868f;
    float m4[4 * SUB];  // (independent chains)
#pragma unroll
    for (int s = 0; s < SUB; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) m4[s * 4 + q] = max3(sc[s][q * 4], sc[s][q * 4 + 1], max3(sc[s][q * 4 + 2], sc[s][q * 4 + 3], sc[s][q * 4 + 3]));
    float mx = max3(m4[0], m4[1], max3(m4[2], m4[3], m4[3]));
    if constexpr (SUB == 2) mx = max3(mx, max3(m4[4], m4[5], m4[5]), max3(m4[6], m4[7], m4[7]));
    mx *= kScale;
    // The running maximum is the same in both lanes of a token.  It only has to bound the scores: while no lane
    // exceeds it, nothing is exchanged or rescaled.
    if (__any(mx > mrun)) {
      const float mn = fmaxf(mrun, fmaxf(mx, __shfl_xor(mx, 32, 64)));
      // (a split may hold no position a token sees: maximum -inf, sums of zero)
      const float alpha = __builtin_amdgcn_exp2f(mrun - (SPLIT && mn == -INFINITY ? 0.f : mn));
      mrun = mn;
      lrun *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[dt][e] *= alpha;
    }
    const float mn = SPLIT && mrun == -INFINITY ? 0.f : mrun;
    float l4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 2 * SUB; ++st) {
      const int s = st >> 1, ps = st & 1;
      if (DIAGONAL && kv0 + st * 16 > p_last) break;  // none of the wave's tokens sees these positions
      if (st + 1 < 2 * SUB) read_v(st + 1, vf[(st + 1) & 1]);
      uint32_t pw[PIECES][4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        float w0 = __builtin_amdgcn_exp2f(fmaf(sc[s][ps * 8 + e], kScale, -mn));
        float w1 = __builtin_amdgcn_exp2f(fmaf(sc[s][ps * 8 + e + 1], kScale, -mn));
#pragma unroll
        for (int pc = 0; pc < PIECES; ++pc) {
          const uint32_t b = HF::pack2(w0, w1);
          pw[pc][e / 2] = b;
          l4[e / 2] = pair_sum(b, l4[e / 2], (HF*)nullptr);  // the weights as they are multiplied
          if (pc + 1 < PIECES) {
            w0 -= HF::lo(b);
            w1 -= HF::hi(b);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (DIAGONAL) {
        if (kv0 + st * 16 + 15 > p_last) {
          const int keep = (int)p_last - (int)(kv0 + st * 16 + hf * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t m = column_mask(keep, e);
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) vf[st & 1][dt][e] &= m;
          }
        }
      }
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int pc = 0; pc < PIECES; ++pc)
          acc[dt] = mfma32(vf[st & 1][dt], u32x4{pw[pc][0], pw[pc][1], pw[pc][2], pw[pc][3]}, acc[dt], (HF*)nullptr);
    }
    lrun += (l4[0] + l4[1]) + (l4[2] + l4[3]);
  };

  if (kv_begin < kv_end) {
    auto copied = [&]() __attribute__((always_inline)) {  // this wave's copies have landed, then everyone's
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_barrier();
    };
    copy(kv_begin, 0);
    copied();
    int buf = 0;
    uint32_t kv0 = kv_begin;
    auto chunks_to = [&](auto diagonal, uint32_t end) __attribute__((always_inline)) {
      for (; kv0 < end; kv0 += CH, buf ^= 1) {
        if (kv0 + CH < kv_end) copy(kv0 + CH, buf ^ 1);  // (uniform over the workgroup)
        if (active && kv0 <= p_last) do_chunk(diagonal, buf, kv0);
        copied();
      }
    };
    // Whole chunks that every token of the workgroup sees, then the others.  (One loop with the column mask in it costs a 4B
    // prompt of 1040 tokens, 4 layers, 1 %: 1443 us without a mask, 1458 so, 1449 as it is.)
    const uint32_t seen = (pos0 + (uint32_t)(tb * AB_TOKENS) + 1) / CH * CH;
    chunks_to(std::false_type{}, min(seen, kv_end));
    chunks_to(std::true_type{}, kv_end);
  }
  if (!active || t0 + r32 >= n) return;
  const float l = lrun + __shfl_xor(lrun, 32, 64);

  // acc[dt] element e: head dim dt * 32 + (e / 4) * 8 + hf * 4 + e % 4 of this lane's token
  if constexpr (SPLIT) {
    float* rec = part + (((size_t)blockIdx.y * n + t) * nq + head) * AB_REC;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(rec + dt * 32 + q * 8 + hf * 4) =
            make_float4(acc[dt][q * 4], acc[dt][q * 4 + 1], acc[dt][q * 4 + 2], acc[dt][q * 4 + 3]);
    if (hf == 0) *reinterpret_cast<float2*>(rec + 128) = make_float2(mrun, l);
    return;
  } else {
    // straight into the fragment order the output projection reads: operand index k = head * 128 + dim
    const int KTQ = nq * 4, tt = t >> 4, c16 = t & 15;
    const float inv = 1.0f / l;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k0 = head * 128 + dt * 32 + q * 8 + hf * 4;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[dt][q * 4 + e] * inv;
#pragma unroll
        for (int pc = 0; pc < PIECES; ++pc) {
          const uint32_t b0 = HF::pack2(v[0], v[1]), b1 = HF::pack2(v[2], v[3]);
          v[0] -= HF::lo(b0);
          v[1] -= HF::hi(b0);
          v[2] -= HF::lo(b1);
          v[3] -= HF::hi(b1);
          const size_t el = (((size_t)(tt * PIECES + pc) * KTQ + (k0 >> 5)) * 64 + c16 + 16 * ((k0 & 31) >> 3)) * 8 + (k0 & 7);
          *reinterpret_cast<uint2*>(static_cast<uint16_t*>(Of) + el) = make_uint2(b0, b1);
        }
      }
  }
}

// The splits of a (token, head): a wave per pair, lane l the dims 2 l and 2 l + 1; four heads of a token per workgroup.
template <class HF>
__global__ __launch_bounds__(256) void k_attn_merge(const float* __restrict__ part, int splits, int n, int nq, void* __restrict__ Of) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int pair = (int)blockIdx.x * 4 + wave;
  if (pair >= n * nq) return;
  const int t = pair / nq, head = pair - t * nq;
  const float* rec0 = part + (size_t)pair * AB_REC;
  const size_t stride = (size_t)n * nq * AB_REC;
  constexpr int MAXS = ATTN_MAX_SPLITS;
  float2 ml[MAXS], o[MAXS];
#pragma unroll
  for (int s = 0; s < MAXS; ++s)
    if (s < splits) {
      ml[s] = *reinterpret_cast<const float2*>(rec0 + s * stride + 128);
      o[s] = *reinterpret_cast<const float2*>(rec0 + s * stride + 2 * lane);
    }
  float M = ml[0].x;  // finite: the first split holds position 0
#pragma unroll
  for (int s = 1; s < MAXS; ++s)
    if (s < splits) M = fmaxf(M, ml[s].x);
  float l = 0.f, a = 0.f, b = 0.f;
#pragma unroll
  for (int s = 0; s < MAXS; ++s)
    if (s < splits) {
      const float f = __builtin_amdgcn_exp2f(ml[s].x - M);
      l += f * ml[s].y;
      a += f * o[s].x;
      b += f * o[s].y;
    }
  const float inv = 1.0f / l;
  a *= inv;
  b *= inv;
  const int KTQ = nq * 4, k0 = head * 128 + 2 * lane;
#pragma unroll
  for (int pc = 0; pc < 2; ++pc) {
    const uint32_t w = HF::pack2(a, b);
    a -= HF::lo(w);
    b -= HF::hi(w);
    const size_t el = (((size_t)((t >> 4) * 2 + pc) * KTQ + (k0 >> 5)) * 64 + (t & 15) + 16 * ((k0 & 31) >> 3)) * 8 + (k0 & 7);
    *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(Of) + el) = w;
  }
}

size_t attn_split_floats(int n, int nq, int splits) { return (size_t)splits * n * nq * AB_REC; }

hipError_t launch_attn_block(hipStream_t s, bool f16, const float* qkv, int nq, int nkv, const void* kc, const void* vt, uint32_t S,
                             uint32_t slot, uint32_t max_seq, uint32_t pos0, int n, int pieces, int splits, float* part,
                             size_t part_floats, void* Of, int n_cus) {
  if (n <= 0 || nkv <= 0 || nq % nkv || S % 32 || pos0 + (uint32_t)n > max_seq || max_seq > S) return hipErrorInvalidValue;
  if (pieces == 1 ? splits != 1 : (pieces != 2 || splits < 2 || splits > ATTN_MAX_SPLITS || !part || attn_split_floats(n, nq, splits) > part_floats))
    return hipErrorInvalidValue;
  const int NB = (n + AB_TOKENS - 1) / AB_TOKENS;
  const int half = splits == 1 && NB % 2 == 0 && NB * nq <= 2 * n_cus ? NB / 2 : 0;
  const dim3 grid((unsigned)(NB * nq), (unsigned)splits);
  const uint16_t *k = static_cast<const uint16_t*>(kc), *v = static_cast<const uint16_t*>(vt);
#define AB(P, CH, SP, HF) \
  k_attn_block<P, CH, SP, HF><<<grid, 256, 0, s>>>(qkv, nq, nkv, k, v, S, slot, max_seq, pos0, n, half, splits, Of, part)
  if (pieces == 1) {
    if (f16) AB(1, 64, false, Fp16);
    else AB(1, 64, false, Bf16);
    return hipGetLastError();
  }
  if (f16) AB(2, 32, true, Fp16);
  else AB(2, 32, true, Bf16);
#undef AB
  if (hipError_t e = hipGetLastError()) return e;
  const unsigned mg = (unsigned)(((size_t)n * nq + 3) / 4);
  if (f16) k_attn_merge<Fp16><<<mg, 256, 0, s>>>(part, splits, n, nq, Of);
  else k_attn_merge<Bf16><<<mg, 256, 0, s>>>(part, splits, n, nq, Of);
  return hipGetLastError();
}

}  // namespace nnc
