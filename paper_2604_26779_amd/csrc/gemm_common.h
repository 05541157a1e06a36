// What the GEMM kernels share: operand vector types, the K slab of the tiled weights, and the order of the tiles over the dies.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace specv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2v_t __attribute__((ext_vector_type(2)));

constexpr int GEMM_KS = 4;          // k-steps (of 16) per slab of the tiled weights
constexpr int GEMM_XCDS = 8;        // accelerator dies, each with its own L2; workgroup i of a launch runs on die i % 8
constexpr int GEMM_THREADS = 256;
constexpr int GEMM_EPI_PLAIN = 0, GEMM_EPI_SWIGLU = 1, GEMM_EPI_STREAM = 2, GEMM_EPI_STREAM_SHARED = 3;

// 64 x 16 bytes from memory straight into LDS (no staging registers, no LDS store instructions): lane i's 16 bytes at base + offset + 16 i go
// to dst + 16 i.  base, offset and dst are the wavefront's; offset < 2^31.
// A buffer load, not global_load ... lds: the compiler takes the latter for a flat access that may touch either memory and, while one is
// outstanding, turns each of its counted waits into vmcnt(0) lgkmcnt(0) - every LDS read and every weight fragment would be waited
// for together with all that was requested after it.
__device__ inline void load_to_lds(const u32x4_t* base, int offset, u32x4_t* dst)
{
    constexpr int RAW = 0x00020000;                     // word 3 of the descriptor: 32-bit data format, no stride, no swizzle
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xffffffffu, RAW);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void __attribute__((address_space(3)))*)dst, 16, (threadIdx.x & 63) * 16, offset, 0, 0);
}

// s_waitcnt operand: at most n vector-memory operations outstanding, the other counters not waited for
constexpr int vmcnt_imm(int n) { return (n & 15) | 0x70 | 0xF00 | ((n >> 4) << 14); }

// eight E4M3 codes (two words) -> eight fp16 or bf16, exact
template <bool F16>
__device__ inline u32x4_t widen_e4m3x8(unsigned int wa, unsigned int wb)
{
    if constexpr (F16)
        return u32x4_t{__builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wa, 1.0f, false)),
                       __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wa, 1.0f, true)),
                       __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wb, 1.0f, false)),
                       __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wb, 1.0f, true))};
    else
        return u32x4_t{__builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(wa, 1.0f, false)),
                       __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(wa, 1.0f, true)),
                       __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(wb, 1.0f, false)),
                       __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(wb, 1.0f, true))};
}

// entry of the grouped GEMM's tile list: first 32-row block of the tile (24 bits) and how many of its rows are not padding
__host__ __device__ inline int moe_tile_pack(int first_block, int rows) { return first_block | (rows << 24); }
__device__ inline int moe_tile_block(int t) { return t & 0xffffff; }
__device__ inline int moe_tile_rows(int t) { return t >> 24; }

// Which tile a workgroup computes.  Workgroups go to the dies round robin in launch order, so the launch index is re-mapped:
// die j takes a contiguous stretch of the tiles in the order (row tile fastest, then column tile, then k-split).  The workgroups
// that share a weight tile then share an L2, and a die reads the activations of one or two k-splits instead of all of them.
struct GemmTile { int bx, by, bz; };       // column tile, k-split, row tile
__device__ inline GemmTile gemm_tile_of_workgroup()
{
    const int nx = gridDim.x, ny = gridDim.y, nz = gridDim.z;
    const int total = nx * ny * nz, lin = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
    const int xcd = lin % GEMM_XCDS, slot = lin / GEMM_XCDS;
    const int v = xcd * (total / GEMM_XCDS) + (xcd < total % GEMM_XCDS ? xcd : total % GEMM_XCDS) + slot;
    // (the divisions run in the vector unit; without the hint the compiler keeps what follows from them there too)
    return GemmTile{__builtin_amdgcn_readfirstlane((v / nz) % nx), __builtin_amdgcn_readfirstlane(v / (nz * nx)), __builtin_amdgcn_readfirstlane(v % nz)};
}

}  // namespace specv
