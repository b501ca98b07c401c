// Tiles of 32 rows x 128 fp16 channels that go from global memory straight into LDS and from there into MFMA operands.
#pragma once

#include "common.h"

namespace antkv {

constexpr int kTileBytes = 32 * kD * 2;                 // 32 rows of 256 bytes

typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(3))) short4_t lds_short4;
typedef __attribute__((address_space(3))) half8_t lds_half8;
typedef __attribute__((address_space(3))) float4_t lds_float4;

// Rows of a tile are 16 chunks of 16 bytes; chunk c of row r sits at place c ^ swz(r).  The 16-byte reads of 16 rows (an
// operand with the rows on its first axis) and the 4 rows x 64 bytes of a transposed read then fall on 64 different banks.
__device__ __forceinline__ int swz(int r) { return 4 * (r & 3) + ((r >> 2) & 3); }

// byte offset of row n, channels 16 s + 8 kh .. + 7 (k-step s of an MFMA operand)
__device__ __forceinline__ uint32_t tile_at(int n, int s, int kh) { return n * 256 + (((2 * s + kh) ^ swz(n)) << 4); }

// byte offset in global memory, from the tile's first row, of the chunk that lane `lane` stages in the 1 KB of rows
// 4 part .. 4 part + 3; rows past `last_row` repeat it
__device__ __forceinline__ uint32_t stage_off(int part, int lane, int last_row)
{
    const int row = 4 * part + (lane >> 4);
    return (row < last_row ? row : last_row) * 256 + (((lane & 15) ^ swz(row)) << 4);
}

// 16 (or 4) bytes per lane from `base` + `off` to LDS address `to` + 16 (or 4) * lane.  The compiler does not count these
// loads: whoever reads the tile waits for them with vmcnt and a barrier of its own.
__device__ __forceinline__ void load_to_lds16(const void* base, uint32_t off, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void load_to_lds4(const void* base, uint32_t off, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(off), "s"(base) : "m0", "memory");
}
// Barrier behind which every wave's loads to LDS have landed except its last N.
template <int N>
__device__ __forceinline__ void landed_but()
{
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

}  // namespace antkv
