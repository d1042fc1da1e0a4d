// Weights of the next GEMM brought into the L2 of the XCD that will read them, by the kernel in front of it.
//
// A short launch pays the HBM latency of its first weights in every workgroup, while the end of the kernel before it (partial
// sums through LDS, the epilogue) leaves HBM idle.  An XCD's L2 keeps clean lines across kernel boundaries (33.6 MB streamed by
// 256 workgroups take 7 us cold, 4 behind a kernel that touched one word per line on the same XCD, 6.7 on
// another), and consecutive workgroups go to the 8 XCDs in turn, so a workgroup knows by its number which share of
// the next launch will run on its own XCD.  A wrong guess costs nothing but the gain.
//
// Measured on whole prompts, us without / with: 0.6B, 14 layers, 33 tokens 650 / 641, 128 704 / 686, 256 938 / 895, 512 1365 / 1330; 1.7B, 8
// layers, 64 592 / 568, 128 733 / 691; 4B, 4 layers, 64 502 / 492; binary16 0.6B 200 1004 / 960.  In decode passes of batches it does not pay: touches by
// idle workgroups of the row-wise kernels make those last as much longer (8B, 16 sequences 504 -> 516 us per step of 4
// layers with 16 MB of them, 4B, 8 sequences 331 -> 338), at the end of the GEMMs they cost 0 - 5 %.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nnc {

// The next GEMM: row block b of nt row tiles (KT tiles of 1 KiB each) is read on XCD b % 8.
struct WeightAhead {
  const void* W = nullptr;  // NULL: nothing to do
  int n_tiles = 0, KT = 0, nt = 1;
  uint32_t nt_inv = 0;      // row / nt = row * nt_inv >> 16 for row < 65536 / nt (past that one too many for some rows: another line is touched)
  int lines_log2 = 0;       // 128-byte lines touched per row tile, from its start
};

// Up to N lines per thread of `wgs` workgroups of 256 threads, this one number wg.  In three parts, so that nothing but
// the loads themselves stands between a kernel's main loop and its epilogue (with the addresses computed there 0.6B, 128 tokens, gained
// half as much).
template <int N>
struct Ahead {
  uint32_t at[N], v[N];
  // byte offsets (past the end: nothing to touch); while the kernel's first loads are in flight
  __device__ __forceinline__ void prepare(const WeightAhead& w, int wg, int wgs) {
    const int xcd = wg & 7, slot = wg >> 3, slots = (wgs - xcd + 7) >> 3;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int item = (i * slots + slot) * 256 + (int)threadIdx.x;
      const int row = item >> w.lines_log2, line = item & ((1 << w.lines_log2) - 1);
      const int b = (int)((uint32_t)row * w.nt_inv >> 16), tile = (xcd + 8 * b) * w.nt + row - b * w.nt;
      at[i] = row < 32768 && tile < w.n_tiles && line < w.KT * 8 ? ((uint32_t)tile * w.KT * 8 + line) * 128 : 0xffffffffu;
      asm volatile("" : "+v"(at[i]));
    }
  }
  __device__ __forceinline__ void issue(const WeightAhead& w) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(w.W), 0, w.W ? w.n_tiles * w.KT * 1024 : 0, 0x00020000);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b32(r, at[i], 0, 0);
  }
  // behind everything else the workgroup does: the loads have to land before it ends
  __device__ __forceinline__ void done() {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" ::"v"(v[i]));
  }
};

// With as many lines per row tile as leave an XCD's share at no more than `lines` (whole row tiles, or the first power of two of lines).
inline WeightAhead weight_ahead(const void* W, int n_tiles, int KT, int nt, long lines) {
  WeightAhead w;
  const long rows = (long)(((n_tiles + nt - 1) / nt + 7) / 8) * nt;
  if (rows > lines || (long)n_tiles * KT >= 1L << 21) return w;  // (32-bit byte offsets, below the ones that stand for nothing)
  w.W = W; w.n_tiles = n_tiles; w.KT = KT; w.nt = nt; w.nt_inv = 65536u / nt + 1;
  while ((1 << w.lines_log2) < KT * 8 && (rows << (w.lines_log2 + 1)) <= lines) ++w.lines_log2;
  return w;
}

}  // namespace nnc
