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

// Column-blocked tile order: ids run down strips of `width` tile columns, so that the workgroups an XCD runs at a time cover a
// compact block of tiles and few operand panels (strip_width in seq_grad_walk.hip says how wide).
constexpr int kStrip = 8;                // ... where nothing else is said
struct TileGrid {
  int m, n, width;                       // tile rows and columns; columns of a strip
  TileDiv strip, across, last;           // tiles of a full strip; its width; columns of the last strip, where it is narrower
};
inline TileGrid tile_grid(int m, int n, int width = kStrip) {
  return {m, n, width, tile_div_by((unsigned)(m * width)), tile_div_by((unsigned)width),
          tile_div_by((unsigned)(n % width ? n % width : width))};
}
// WIDTH: of a strip, where it is known (0: what the grid says)
template <int WIDTH>
__device__ __forceinline__ void tile_coords(int tile, const TileGrid& g, int& tile_m, int& tile_n) {
  const int width = WIDTH ? WIDTH : g.width, s = tile_div(tile, g.strip), c0 = s * width, in_strip = tile - s * (int)g.strip.d;
  if (WIDTH && c0 + width <= g.n) {
    tile_m = in_strip / (WIDTH ? WIDTH : 1);
    tile_n = c0 + in_strip % (WIDTH ? WIDTH : 1);
  } else {
    const TileDiv by = c0 + width <= g.n ? g.across : g.last;
    tile_m = tile_div(in_strip, by);
    tile_n = c0 + in_strip - tile_m * (int)by.d;
  }
}

// seq_grad_walk.hip
hipError_t launch_seq_grad_walk(const SeqGradArgs& a, const ContractionPlan& pl, hipStream_t s);

}  // namespace isopo
