// Device helpers shared by the streaming bf16 contractions: seq_grad_stream.hip (a work item per workgroup) and
// seq_grad_walk.hip (workgroups that walk a list of them).
#pragma once

#include "common.h"
#include "kernels.h"
#include "pair_walk.h"

namespace isopo {

typedef unsigned short u16;
typedef s16x4 __attribute__((address_space(3)))* lds_s16x4_ptr;
typedef void __attribute__((address_space(3)))* lds_void_ptr;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 32;                   // tokens per block
constexpr int NSTAGE = 4;                // token blocks in the LDS ring
constexpr int AHEAD = NSTAGE - 1;        // blocks in flight while one is multiplied

// 16 bytes per lane from a buffer straight into LDS: lane l lands at lds_addr + 16*l.
// Inline asm, so that the compiler's LDS-DMA tracking does not put a vmcnt(0) before
// every later LDS read; the kernels order them themselves with s_waitcnt vmcnt(n) + s_barrier.
__device__ __forceinline__ void load_lds16(v4i rsrc, unsigned lds_addr, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               : : "s"(lds_addr), "v"(voff), "s"(rsrc) : "memory");
}

// Two fp32 -> one dword of two bf16 (round to nearest even), one v_cvt_pk_bf16_f32.
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// Accumulator element -> VGPR at the point of use.  Without this the register allocator copies the
// whole 256-register tile out of the AGPRs before the epilogue and spills.
__device__ __forceinline__ float acc_read(float a) {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}

// Column-blocked tile order: ids run down 8-column strips of the tile grid, so the 32 workgroups an
// XCD runs at a time cover about 4 tile rows x 8 tile columns (12 operand panels) rather than
// 2 x 16 (18 panels): fewer L2 misses per flop.
struct TileGrid {
  int m, n;                              // tile rows and columns
  TileDiv strip, last;                   // tiles of a full strip; columns of the last strip, where it is narrower
};
constexpr int kStrip = 8;
inline TileGrid tile_grid(int m, int n) {
  return {m, n, tile_div_by((unsigned)(m * kStrip)), tile_div_by((unsigned)(n % kStrip ? n % kStrip : kStrip))};
}
__device__ __forceinline__ void tile_coords(int tile, const TileGrid& g, int& tile_m, int& tile_n) {
  const int s = tile_div(tile, g.strip), c0 = s * kStrip, in_strip = tile - s * (int)g.strip.d;
  if (c0 + kStrip <= g.n) {
    tile_m = in_strip / kStrip;
    tile_n = c0 + in_strip % kStrip;
  } else {
    tile_m = tile_div(in_strip, g.last);
    tile_n = c0 + in_strip - tile_m * (int)g.last.d;
  }
}

// seq_grad_walk.hip
hipError_t launch_seq_grad_walk(const SeqGradArgs& a, const ContractionPlan& pl, hipStream_t s);

}  // namespace isopo
