// Tiles of rows of D bf16 in shared memory, filled straight from global memory, as operands of
// v_mfma_f32_32x32x16_bf16 (gfx950).
//
// Layout: a row is 16 units of 16 bytes; unit u of tile row r sits at position u ^ (r & 15) of the
// row, so that the eight lanes that a shared-memory cycle serves read distinct banks.  Operand of
// the instruction: lane l holds row (or column) l % 32 at dimensions 16 s + 8 (l / 32) .. + 8 of step s =
// 0 .. 7, i.e. unit 2 s + l / 32; result element i of lane l is row 8 (i / 4) + 4 (l / 32) + i % 4,
// column l % 32.
#pragma once

#include "wnw_internal.h"

namespace wnw {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

__device__ inline unsigned lds_address(const void *p)
{
    return (unsigned)(size_t)(__attribute__((address_space(3))) const void *)p;
}

// 16 (4) bytes per lane from global memory, `base` (uniform) + off bytes, to shared memory at `lds`
// (uniform) + 16 (4) * lane.  In assembly, as the compiler would wait for every such load before any
// read of shared memory; the kernels wait themselves (lds_loads_wait).  There is no register output.
__device__ inline void load_to_lds(const void *base, unsigned off, unsigned lds)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}
__device__ inline void load_word_to_lds(const void *base, unsigned off, unsigned lds)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}

// Waits until at most N of this wavefront's vector memory loads are outstanding.
template <int N>
__device__ inline void lds_loads_wait()
{
    __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Work-group barrier that waits for this wavefront's shared-memory operations, not for its loads in flight.
__device__ inline void lds_tile_barrier()
{
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Loader of tiles of TILE_ROWS rows: PF 16-byte pieces per lane, wavefront `wave` (uniform) taking pieces
// 64 PF wave .. + 64 PF.  The lanes' offsets inside a tile are fixed, so a whole tile costs no vector
// arithmetic: its base is uniform.  DIRECT needs rows aligned to 16 bytes, the size of its loads; otherwise the
// pieces go through registers, for rows at any address that bf16 values may have.
template <int TILE_ROWS, int PF, bool DIRECT = true>
struct TileLoader {
    unsigned off[PF];
    int wave, lane, step;
    __device__ TileLoader(int wave_, int lane_, int step_) : wave(wave_), lane(lane_), step(step_)
    {
#pragma unroll
        for (int j = 0; j < PF; ++j) off[j] = piece(j, row(j) * step);
    }
    __device__ int row(int j) const { return ((wave * PF + j) * 64 + lane) >> 4; }
    __device__ unsigned piece(int j, int src_row) const
    {
        return (unsigned)src_row * (D * 2) + (unsigned)((lane ^ row(j)) & 15) * 16;
    }
    __device__ void copy(const uint16_t *base, unsigned byte_off, unsigned lds) const
    {
        if constexpr (DIRECT)
            load_to_lds(base, byte_off, lds);
        else {
            u32x4_t v;
            __builtin_memcpy(&v, base + byte_off / 2, sizeof(v));
            *(__attribute__((address_space(3))) u32x4_t *)(size_t)(lds + lane * 16) = v;
        }
    }
    // Rows row0, row0 + step, ... of `src` (rows of D, the last one rows - 1; row0 uniform, row0 + TILE_ROWS * step
    // < 2^31) into the tile at shared address `lds`.  Past the last row that row comes again.
    __device__ void load(const uint16_t *src, int row0, int rows, unsigned lds) const
    {
        lds += (unsigned)(wave * PF) * 1024;
        if (row0 + step * TILE_ROWS <= rows) {
            const uint16_t *base = src + (size_t)row0 * D;
#pragma unroll
            for (int j = 0; j < PF; ++j) copy(base, off[j], lds + j * 1024);
        } else {
            const int first = min(row0, rows - 1);
            const uint16_t *base = src + (size_t)first * D;
#pragma unroll
            for (int j = 0; j < PF; ++j)
                copy(base, piece(j, min(row(j) * step, rows - 1 - first)), lds + j * 1024);
        }
    }
};

// Byte offsets in a tile of this lane's eight fragments of rows 0 .. 31 (those of rows 32 n .. are 32 n rows
// further: the swizzle repeats).
struct FragOffsets {
    unsigned o[8];
    __device__ explicit FragOffsets(int lane)
    {
        const unsigned col = lane & 31, half = lane >> 5;
#pragma unroll
        for (int s = 0; s < 8; ++s) o[s] = col * (D * 2) + ((2 * s + half) ^ (col & 15)) * 16;
    }
};
__device__ inline bf16x8_t frag_read(unsigned lds)
{
    return __builtin_bit_cast(bf16x8_t, *(const __attribute__((address_space(3))) u32x4_t *)(size_t)lds);
}

__device__ inline f32x16_t mfma32(bf16x8_t a, bf16x8_t b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

}  // namespace wnw
