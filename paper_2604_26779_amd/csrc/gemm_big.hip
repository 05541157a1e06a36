// MFMA GEMM with 192- or 256-row x 256-column tiles, for launches of more than 128 rows (layouts and operand formats as in
// gemm_bf16.hip; the tile is chosen there).
//
// Here the MFMAs are the bound, and what keeps them waiting is the CU's vector-memory path: a tile needs MB + 8 KiB per
// 16-wide k-step (twice the MB part for hi + lo operands) for MB * 64 MFMA cycles, as long as nothing is fetched twice.  So both
// operands go from memory straight into LDS (global_load ... lds) exactly once per workgroup, and the four wavefronts (2 x 2,
// MB/2 x 4 accumulator blocks of 32 x 32 each) read their fragments from there.
//   * A slab is two k-steps.  NBUF slabs sit in LDS (80-144 KiB, one workgroup per CU): while one is multiplied, the others
//     are in flight, so a transfer has two or three slabs' worth of MFMAs (1 000 or 2 000 cycles each) to arrive.
//   * LDS reads run one k-step ahead of the MFMAs that use them, across the slab boundary too: the barrier between slabs sits
//     before the last k-step's MFMAs, when every wavefront has its last fragments in registers and the next slab has arrived.
//     Behind it the freed buffer is refilled and the next slab's first fragments are read, under those MFMAs.
// 8B shapes, before (weights streamed into registers, every fragment by two wavefronts; activations staged through registers) and
// with the ring: gate/up 103 -> 93 us at 384 rows and 248 -> 229 at 1024 (1 050 TFLOP/s), QKV and output projection 41 -> 38.5 and
// 91 -> 82.  What bounds it is the clock under the MFMAs' load: the 384-row gate/up takes 90 us alone, 73 with the MFMAs only, and
// with operands of zeros 73 and 60.  Re-reading one slab instead of streaming gains 2 us: the transfers are hidden.
#include <type_traits>

#include "common.h"
#include "gemm_common.h"
#include "lds_limit.h"
#include "operand.h"

namespace specv {

template <int MB, int EPI, bool W8, int XF>
struct GemmBig {
    static constexpr int KS = 2;                                      // k-steps per LDS slab
    static constexpr int A_CHUNKS = KS * MB * XF;                     // 1 KiB chunks (64 lanes x 16 bytes) per slab
    static constexpr int W_CHUNKS = W8 ? 8 : KS * 8;
    static constexpr int CHUNKS = A_CHUNKS + W_CHUNKS;
    static constexpr int NBUF = CHUNKS <= 32 ? 4 : 3;
    static constexpr int EPI_BYTES = EPI == GEMM_EPI_SWIGLU ? (MB / 2) * 32 * 129 * 4 : 0;
    static constexpr int LDS_BYTES = NBUF * CHUNKS * 1024 > EPI_BYTES ? NBUF * CHUNKS * 1024 : EPI_BYTES;
};

template <int MB, int EPI, bool W8, int XF>
__global__ __launch_bounds__(GEMM_THREADS, 1) void gemm_big_kernel(
    const u32x4_t* __restrict__ Wp, const u32x4_t* __restrict__ Xp, float* __restrict__ out, int n_blocks, int k_steps,
    int ksteps_per_split, int mb_pad, int M, int N, int ldo, int64_t split_stride, const float* __restrict__ wscale)
{
    typedef GemmBig<MB, EPI, W8, XF> C;
    constexpr int KS = C::KS, NBUF = C::NBUF, MBW = MB / 2, NBW = 4;
    constexpr int SLAB = C::CHUNKS * 64;                               // u32x4_t per slab
    constexpr int LPS = C::CHUNKS / 4;                                 // transfers per wavefront and slab
    constexpr int A_LPS = C::A_CHUNKS / 4;
    static_assert(C::A_CHUNKS % 4 == 0 && C::W_CHUNKS % 4 == 0, "the chunks must divide over the wavefronts");
    static_assert((NBUF - 1) * LPS <= 63, "the wait below counts transfers in six bits");
    extern __shared__ u32x4_t lds[];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int mh = wave & 1, np = wave >> 1;
    const GemmTile tile_of = gemm_tile_of_workgroup();
    const int bx = tile_of.bx, by = tile_of.by;
    const int ks0 = by * ksteps_per_split;
    const int ks1 = ks0 + ksteps_per_split < k_steps ? ks0 + ksteps_per_split : k_steps;
    const int n_slabs = (ks1 - ks0) / KS;                              // even, and at least 4
    const int mblk0 = tile_of.bz * MB, nb_first = bx * 8, nb0 = nb_first + np * NBW;

    // chunk wave + 4 j of a slab: activations [k-step][row block][part], then weights [column block][k-step]
    // (8 bit: [column block], both k-steps in one word)
    const u32x4_t* src[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        if (j < A_LPS) {
            const int c = wave + 4 * j, kl = c / (MB * XF), rem = c % (MB * XF);
            src[j] = Xp + (((int64_t)(ks0 + kl) * mb_pad + mblk0) * XF + rem) * 64;
        } else {
            const int c = wave + 4 * (j - A_LPS), blk = W8 ? c : c >> 1;
            const int nb = nb_first + blk < n_blocks ? nb_first + blk : 0;
            src[j] = Wp + (((int64_t)(ks0 / GEMM_KS) * n_blocks + nb) * (W8 ? 2 : GEMM_KS) + (W8 ? 0 : c & 1)) * 64;
        }
    }
    const int64_t x_step = (int64_t)KS * mb_pad * XF * 64;
    const int64_t w_half = W8 ? 64 : 128, w_step = (int64_t)n_blocks * (W8 ? 2 : GEMM_KS) * 64;
    auto stage = [&](int s, int buf) {
#pragma unroll
        for (int j = 0; j < LPS; ++j) {
            const u32x4_t* p = src[j] + (j < A_LPS ? s * x_step : (s >> 1) * w_step + (s & 1) * w_half) + lane;
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)p,
                                             (void __attribute__((address_space(3)))*)(lds + buf * SLAB + (wave + 4 * j) * 64), 16, 0, 0);
        }
    };

    f32x16_t acc[MBW][NBW];
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < NBW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    u32x4_t a[2][MBW][XF], w[2][NBW];
    u32x2v_t w8[2][NBW];
    auto read_frags = [&](int buf, auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        const u32x4_t* base = lds + buf * SLAB;
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
            const u32x4_t* wl = base + C::A_CHUNKS * 64;
            if constexpr (W8) w8[kk][j] = *((const u32x2v_t*)(wl + (np * NBW + j) * 64 + lane) + kk);
            else w[kk][j] = wl[((np * NBW + j) * KS + kk) * 64 + lane];
        }
#pragma unroll
        for (int i = 0; i < MBW; ++i)
#pragma unroll
            for (int part = 0; part < XF; ++part) a[kk][i][part] = base[((kk * MB + mh * MBW + i) * XF + part) * 64 + lane];
    };
    auto multiply = [&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        u32x4_t wk[NBW];
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
            if constexpr (W8) wk[j] = widen_e4m3x8<XF == XF_F16>(w8[kk][j].x, w8[kk][j].y);
            else wk[j] = w[kk][j];
        }
        // hi products of all blocks first, then the lo products: two MFMAs on one accumulator are never adjacent
#pragma unroll
        for (int part = 0; part < XF; ++part)
#pragma unroll
            for (int i = 0; i < MBW; ++i)
#pragma unroll
                for (int j = 0; j < NBW; ++j) {
                    if constexpr (XF == XF_F16)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a[kk][i][part]),
                                                                           __builtin_bit_cast(f16x8_t, wk[j]), acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[kk][i][part]),
                                                                            __builtin_bit_cast(bf16x8_t, wk[j]), acc[i][j], 0, 0, 0);
                }
    };
    // one MFMA, one LDS read, one MFMA, one LDS read, ...: the reads (and the transfers) go out under the MFMAs
    auto interleave = [&](auto transfers_c) {
        constexpr int READS = MBW * XF + NBW, T = decltype(transfers_c)::value ? LPS : 0;
#pragma unroll
        for (int i = 0; i < READS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if constexpr (T > 0) {
#pragma unroll
            for (int i = 0; i < T && i < MBW * NBW * XF - READS - 1; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        }
    };
    using k0_t = std::integral_constant<int, 0>;
    using k1_t = std::integral_constant<int, 1>;
    int buf = 0;
    // slab s; REST = slabs behind it that are still to come or in flight, capped at NBUF (then buffer `buf` is refilled)
    auto slab = [&](auto rest_c, int s) {
        constexpr int REST = decltype(rest_c)::value;
        const int next = buf + 1 < NBUF ? buf + 1 : 0;
        read_frags(buf, k1_t{});
        multiply(k0_t{});
        interleave(std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (REST > 0) {
            // this wavefront's last reads of the slab are done and its share of the next slab has arrived (the slabs after
            // that stay in flight); behind the barrier the same holds for all four
            constexpr int FLIGHT = (REST < NBUF - 1 ? REST : NBUF - 1) - 1;
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(FLIGHT * LPS) & ~0xF00);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            read_frags(next, k0_t{});
            if constexpr (REST >= NBUF) stage(s + NBUF, buf);
        }
        multiply(k1_t{});
        if constexpr (REST > 0) interleave(std::integral_constant<bool, (REST >= NBUF)>{});
        __builtin_amdgcn_sched_barrier(0);
        buf = next;
    };

    float wsc[NBW];                                     // 8-bit weights: this lane's column scales
#pragma unroll
    for (int j = 0; j < NBW; ++j) wsc[j] = 1.0f;
    if constexpr (W8) {
#pragma unroll
        for (int j = 0; j < NBW; ++j)
            if (nb0 + j < n_blocks) wsc[j] = wscale[(nb0 + j) * 32 + (lane & 31)];
#pragma unroll
        for (int j = 0; j < NBW; ++j) asm volatile("" : "+v"(wsc[j]));       // arrived before the transfers are counted
    }
#pragma unroll
    for (int i = 0; i < NBUF; ++i) stage(i, i);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NBUF - 1) * LPS));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_frags(0, k0_t{});
    int s = 0;
    for (; s < n_slabs - NBUF; ++s) slab(std::integral_constant<int, NBUF>{}, s);
    if constexpr (NBUF > 3) { slab(std::integral_constant<int, 3>{}, s); ++s; }
    slab(std::integral_constant<int, 2>{}, s);
    slab(std::integral_constant<int, 1>{}, s + 1);
    slab(std::integral_constant<int, 0>{}, s + 2);

    if constexpr (EPI == GEMM_EPI_SWIGLU) {
        // Gate and up column blocks are interleaved in the tiling, so a wavefront's four accumulator columns are (gate, up) of
        // two groups of 32 hidden channels: silu(gate) * up in registers, transposed through LDS into rows one half of the rows
        // at a time, and written in the operand order the down projection reads.
        float* tile = (float*)lds;                              // [MBW*32 rows][129]
        uint4* xo = (uint4*)out;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            __syncthreads();
            if (mh == half) {
#pragma unroll
                for (int i = 0; i < MBW; ++i)
#pragma unroll
                    for (int cg = 0; cg < 2; ++cg)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            float g = acc[i][2 * cg][r], u = acc[i][2 * cg + 1][r];
                            if constexpr (W8) {
                                g *= wsc[2 * cg];
                                u *= wsc[2 * cg + 1];
                            }
                            int row = i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                            tile[row * 129 + (np * 2 + cg) * 32 + (lane & 31)] = g / (1.0f + __expf(-g)) * u;
                        }
            }
            __syncthreads();
            for (int e = threadIdx.x; e < MBW * 32 * 16; e += GEMM_THREADS) {
                int row = e >> 4, g8 = e & 15;
                int m = (mblk0 + half * MBW) * 32 + row, f = bx * 128 + g8 * 8;
                if (m >= M || f >= N / 2) continue;
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = tile[row * 129 + g8 * 8 + j];
                xp_store8_t<XF>(xo, m, f, mb_pad, v);
            }
        }
        return;
    }
    float* o = out + (int64_t)by * split_stride;
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
        const int n = (nb0 + j) * 32 + (lane & 31);
        if (nb0 + j >= n_blocks || n >= N) continue;
        const float sc = wsc[j];
#pragma unroll
        for (int i = 0; i < MBW; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                int m = (mblk0 + mh * MBW + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (m < M) o[(int64_t)m * ldo + n] = W8 ? acc[i][j][r] * sc : acc[i][j][r];
            }
    }
}

template <int MB, int EPI, bool W8, int XF>
static spec_status launch_one(const PackedW& W, const bf16_t* Xp, int M, int mb_pad, float* out, int ldo, int kps, dim3 grid, hipStream_t s)
{
    auto kern = gemm_big_kernel<MB, EPI, W8, XF>;
    constexpr int lds_bytes = GemmBig<MB, EPI, W8, XF>::LDS_BYTES;        // beyond the 64 KiB a kernel gets by default
    static LdsLimit limit;
    const hipError_t raised = limit.raise((const void*)kern, lds_bytes);
    if (raised != hipSuccess) { set_error("gemm: cannot reserve %d bytes of LDS: %s", lds_bytes, hipGetErrorString(raised)); return SPEC_EHIP; }
    kern<<<grid, GEMM_THREADS, lds_bytes, s>>>((const u32x4_t*)W.data, (const u32x4_t*)Xp, out, W.n_blocks, W.k_steps, kps, mb_pad, M, W.N, ldo,
                                               (int64_t)M * ldo, W.scale);
    SPEC_LAUNCH_CHECK("gemm_big_kernel");
    return SPEC_OK;
}

template <int MB, int EPI>
static spec_status launch_by_type(const PackedW& W, const bf16_t* Xp, int M, int mb_pad, float* out, int ldo, int kps, dim3 grid, hipStream_t s)
{
    if (W.w8) return W.f16 ? launch_one<MB, EPI, true, XF_F16>(W, Xp, M, mb_pad, out, ldo, kps, grid, s)
                           : launch_one<MB, EPI, true, XF_HILO>(W, Xp, M, mb_pad, out, ldo, kps, grid, s);
    return W.f16 ? launch_one<MB, EPI, false, XF_F16>(W, Xp, M, mb_pad, out, ldo, kps, grid, s)
                 : launch_one<MB, EPI, false, XF_HILO>(W, Xp, M, mb_pad, out, ldo, kps, grid, s);
}

// grid = (256-column tiles, k-splits, tiles of mb * 32 rows); mb = 6 or 8; every split holds a multiple of 8 k-steps
spec_status launch_gemm_big(const PackedW& W, const bf16_t* Xp, int M, int mb, int mb_pad, float* out, int ldo, int kps, bool swiglu,
                            dim3 grid, hipStream_t s)
{
    if ((mb != 6 && mb != 8) || kps % 8 || W.k_steps % 8) { set_error("gemm: bad shape for the 256-column tile"); return SPEC_EINVAL; }
    if (mb == 6) return swiglu ? launch_by_type<6, GEMM_EPI_SWIGLU>(W, Xp, M, mb_pad, out, ldo, kps, grid, s)
                               : launch_by_type<6, GEMM_EPI_PLAIN>(W, Xp, M, mb_pad, out, ldo, kps, grid, s);
    return swiglu ? launch_by_type<8, GEMM_EPI_SWIGLU>(W, Xp, M, mb_pad, out, ldo, kps, grid, s)
                  : launch_by_type<8, GEMM_EPI_PLAIN>(W, Xp, M, mb_pad, out, ldo, kps, grid, s);
}

}  // namespace specv
