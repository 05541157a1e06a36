// bf16 MFMA GEMM for the verify step's projections:  out[m][n] = sum_k x[m][k] * W[n][k],
// fp32 accumulation, M = B*(k+1) rows (a few dozen to a few hundred), N and K in the thousands.
// At these shapes the weights are streamed once from HBM and everything else is noise, so the
// kernel is organised around the weight stream:
//
//   * W is re-tiled once (at model creation) into MFMA operand order: for every block of 32
//     output columns and every 16-wide k-step, the 64 lanes' 16-byte operands are contiguous
//     (1 KiB).  A wavefront owns one 32-column block and reads its stream with perfectly
//     coalesced 16-byte loads straight into registers; no LDS round trip for the weights.
//     The fragments are ordered [k-slab][column block][k-step in slab]: all wavefronts of a
//     launch move through K together, so at any moment the chip reads one contiguous region
//     (spread evenly over the HBM channels) instead of thousands of streams a power of two apart.
//   * the activations are written by the producing kernel in the same operand order, as hi + lo
//     bf16 pairs ([k-step][32-row block][hi|lo][lane][8], see operand.h), staged through LDS in
//     slabs of KS k-steps (two or three in flight, one barrier per slab) and shared by the 4 wavefronts
//     of the workgroup; each weight fragment feeds two MFMAs per row block (hi and lo).
//   * v_mfma_f32_32x32x16_bf16: A = activation fragment (rows m), B = weight fragment
//     (columns n), so a lane ends up with one output column and 16 rows: stores are
//     128-byte row segments.
//   * K is split across workgroups (grid.y) when N alone gives too few workgroups to keep
//     256 CUs streaming; partial sums go to separate fp32 slices that the consumer adds up
//     in a fixed order (deterministic).
#include <type_traits>

#include "common.h"
#include "gemm_common.h"
#include "operand.h"

namespace specv {

constexpr int GEMM_WD = 2;          // slabs of weight fragments each wavefront keeps in flight: the LDS slabs behind them allow no more
constexpr int GEMM_KUNIT = GEMM_KS * 4;             // K is a multiple of 16 times this

// how many slabs ahead the activations of a tile of mb row blocks are requested.  Two, but one for the large slabs of two hi + lo row blocks and more
// (QKV / output projection of the 8B shape at 64 rows 14.2 / 10.9 us with two, 14.0 / 10.7 with one; at 4 rows 10.9 / 8.1 and 11.2 / 8.2), and
// one in an unsplit launch that crowds the chip: workgroups on one CU cover each other's waits, and requests further ahead only hold up the weight
// stream.  With 16-bit weights that is from one workgroup per CU to three (gate/up of 2 x 18944 and 2 x 28672 columns at 64 rows 71.5 -> 69.5,
// 80.3 -> 78.1 us, heads of 48000 at 4 rows and 64000 at 64 68.8 -> 66.0, 86.7 -> 84.1; with one each or less 45.6 -> 46.5; with four and five either way
// within 2 %: 128256 at 32 and 96 rows 163.8 -> 161.4, 189.5 -> 191.7); with 8-bit ones at 65 rows and more from one on (18944 columns at 96 rows 57.6 ->
// 54.4), below, where few bytes are in flight, from 7/4 on (heads of 96000 columns at 48 rows 76.9 -> 73.5, 128256 at 4, 16 and 32 rows 84.0 -> 80.5,
// 90.7 -> 85.4, 91.9 -> 87.2; 18944 columns at 4 rows 38.1 -> 39.8, 32000 26.0 -> 30.8).  Of the 256-column tiles only the 8-bit ones of 64 rows gain
// (128256 at 64 rows 89.6 -> 87.5).  All at K = 4096.
constexpr int gemm_slabs_ahead(int mb, int xf) { return mb == 1 || xf == XF_F16 ? 2 : 1; }
static bool gemm_crowded(int64_t workgroups, bool w8, int mb, bool one_block)
{
    constexpr int CUS = 256;
    if (!w8) return workgroups > CUS && workgroups <= 3 * CUS;
    return workgroups * 4 > CUS * (one_block && mb <= 2 ? 7 : 4);
}

// from gemm_big.hip
spec_status launch_gemm_big(const PackedW& W, const bf16_t* Xp, int M, int mb, int mb_pad, float* out, int ldo, int kps, bool swiglu,
                            dim3 grid, hipStream_t s);

size_t bf16_packed_elems(int N, int K) { return (size_t)cdiv(N, 32) * 32 * (size_t)K; }

// ------------------------------------------------------------------ weight re-tiling
struct PackParts { const bf16_t* ptr[4]; int row_end[4]; int n; int interleave; int to_f16; };

// bf16 pair -> fp16 pair.  Exact for magnitudes from 2^-14 up to 65504 (bf16 has fewer mantissa bits than fp16);
// below 2^-14 the fp16 grid has steps of 2^-24 (absolute error at most 2^-25, nothing for a weight matrix);
// beyond 65504 the value saturates.
__device__ inline unsigned int bf16x2_to_f16x2(unsigned int w)
{
    return pack_f16x2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
}

__global__ void pack_w_kernel(PackParts parts, int N, int K, int k_steps, int64_t total, uint4* __restrict__ out)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;     // one 16-byte operand per thread
    if (idx >= total) return;
    int lane = (int)(idx & 63);
    int64_t frag = idx >> 6;
    // frag = (slab * n_blocks + nb) * KS + kk
    int kk = (int)(frag % GEMM_KS);
    int n_blocks = (N + 31) / 32;
    int nb = (int)((frag / GEMM_KS) % n_blocks);
    int ks = (int)(frag / GEMM_KS / n_blocks) * GEMM_KS + kk;
    int n = nb * 32 + (lane & 31);
    int k0 = ks * 16 + (lane >> 5) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (parts.interleave) {
        // two equal parts (gate, up): column block 2j holds rows 32j.. of part 0, block 2j+1 the same rows of part 1
        int row = (nb >> 1) * 32 + (lane & 31);
        if (row < parts.row_end[0]) v = *(const uint4*)(parts.ptr[nb & 1] + (int64_t)row * K + k0);
    } else if (n < N) {
        int start = 0;
        for (int p = 0; p < parts.n; ++p) {
            if (n < parts.row_end[p]) {
                v = *(const uint4*)(parts.ptr[p] + (int64_t)(n - start) * K + k0);
                break;
            }
            start = parts.row_end[p];
        }
    }
    if (parts.to_f16) v = make_uint4(bf16x2_to_f16x2(v.x), bf16x2_to_f16x2(v.y), bf16x2_to_f16x2(v.z), bf16x2_to_f16x2(v.w));
    out[idx] = v;
}

spec_status bf16_pack_matrix(const bf16_t* const* dev_parts, const int* part_rows, int n_parts, int K, bf16_t* dev_out,
                             PackedW* out, bool interleave, bool to_f16, hipStream_t s)
{
    if (n_parts < 1 || n_parts > 4 || K % (16 * GEMM_KUNIT)) { set_error("bf16_pack_matrix: bad shape"); return SPEC_EINVAL; }
    PackParts pp;
    pp.n = n_parts;
    pp.interleave = interleave ? 1 : 0;
    pp.to_f16 = to_f16 ? 1 : 0;
    if (interleave && (n_parts != 2 || part_rows[0] != part_rows[1] || part_rows[0] % 32)) { set_error("bf16_pack_matrix: interleaving needs two equal parts of a multiple of 32 rows"); return SPEC_EINVAL; }
    int N = 0;
    for (int i = 0; i < n_parts; ++i) {
        if (((uintptr_t)dev_parts[i] & 15) != 0) { set_error("bf16 weights must be 16-byte aligned"); return SPEC_EINVAL; }
        N += part_rows[i];
        pp.ptr[i] = dev_parts[i];
        pp.row_end[i] = N;
    }
    out->data = dev_out;
    out->N = N;
    out->K = K;
    out->n_blocks = (int)cdiv(N, 32);
    out->k_steps = K / 16;
    out->f16 = to_f16 ? 1 : 0;
    int64_t total = (int64_t)out->n_blocks * out->k_steps * 64;
    pack_w_kernel<<<(unsigned)cdiv(total, 256), 256, 0, s>>>(pp, N, K, out->k_steps, total, (uint4*)dev_out);
    SPEC_LAUNCH_CHECK("pack_w_kernel");
    return SPEC_OK;
}

// 8-bit weights (E4M3 codes, one fp32 scale per output row): the same tiling with two k-steps per 16-byte word,
// [k_steps / KS][n_blocks][KS / 2][64 lanes][2 fragments of 8 codes], and the scales in tiled column order.
struct PackParts8 { const unsigned char* ptr[4]; const float* scale[4]; int row_end[4]; int n; int interleave; };

__device__ inline bool pack8_source(const PackParts8& parts, int nb, int col, int N, int* part, int* row)
{
    if (parts.interleave) {
        *part = nb & 1;
        *row = (nb >> 1) * 32 + col;
        return *row < parts.row_end[0];
    }
    const int n = nb * 32 + col;
    if (n >= N) return false;
    int start = 0;
    for (int p = 0; p < parts.n; ++p) {
        if (n < parts.row_end[p]) { *part = p; *row = n - start; return true; }
        start = parts.row_end[p];
    }
    return false;
}

__global__ void pack_w8_kernel(PackParts8 parts, int N, int K, int64_t total, uint4* __restrict__ out, float* __restrict__ scale_out)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;     // one 16-byte word (two fragments) per thread
    const int n_blocks = (N + 31) / 32;
    if (idx < (int64_t)n_blocks * 32) {                                // the scales, tiled column order; padding columns 0
        int part, row;
        scale_out[idx] = pack8_source(parts, (int)(idx >> 5), (int)(idx & 31), N, &part, &row) ? parts.scale[part][row] : 0.f;
    }
    if (idx >= total) return;
    const int lane = (int)(idx & 63);
    const int64_t frag2 = idx >> 6;                                    // (slab * n_blocks + nb) * (KS / 2) + pair
    const int pair = (int)(frag2 % (GEMM_KS / 2));
    const int nb = (int)((frag2 / (GEMM_KS / 2)) % n_blocks);
    const int ks = (int)(frag2 / (GEMM_KS / 2) / n_blocks) * GEMM_KS + 2 * pair;
    const int k0 = ks * 16 + (lane >> 5) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    int part, row;
    if (pack8_source(parts, nb, lane & 31, N, &part, &row)) {
        const unsigned char* src = parts.ptr[part] + (int64_t)row * K + k0;
        const uint2 a = *(const uint2*)src, b = *(const uint2*)(src + 16);
        v = make_uint4(a.x, a.y, b.x, b.y);
    }
    out[idx] = v;
}

size_t w8_packed_bytes(int N, int K) { return align_up((size_t)cdiv(N, 32) * 32 * ((size_t)K + sizeof(float)), 256); }

// dev_out: w8_packed_bytes(N, K) bytes: the tiled codes, then the tiled scales
spec_status w8_pack_matrix(const unsigned char* const* dev_parts, const float* const* dev_scales, const int* part_rows, int n_parts,
                           int K, void* dev_out, PackedW* out, bool interleave, bool x_f16, hipStream_t s)
{
    if (n_parts < 1 || n_parts > 4 || K % (16 * GEMM_KUNIT)) { set_error("w8_pack_matrix: bad shape"); return SPEC_EINVAL; }
    PackParts8 pp;
    pp.n = n_parts;
    pp.interleave = interleave ? 1 : 0;
    if (interleave && (n_parts != 2 || part_rows[0] != part_rows[1] || part_rows[0] % 32)) { set_error("w8_pack_matrix: interleaving needs two equal parts of a multiple of 32 rows"); return SPEC_EINVAL; }
    int N = 0;
    for (int i = 0; i < n_parts; ++i) {
        if (((uintptr_t)dev_parts[i] & 7) != 0 || ((uintptr_t)dev_scales[i] & 3) != 0) { set_error("8-bit weights must be 8-byte aligned"); return SPEC_EINVAL; }
        N += part_rows[i];
        pp.ptr[i] = dev_parts[i];
        pp.scale[i] = dev_scales[i];
        pp.row_end[i] = N;
    }
    out->data = (const bf16_t*)dev_out;
    out->N = N;
    out->K = K;
    out->n_blocks = (int)cdiv(N, 32);
    out->k_steps = K / 16;
    out->w8 = 1;
    out->f16 = x_f16 ? 1 : 0;           // the codes are the same either way; the kernel widens them to the activations' type
    out->scale = (const float*)((const char*)dev_out + (size_t)out->n_blocks * 32 * K);
    int64_t total = (int64_t)out->n_blocks * (out->k_steps / 2) * 64;
    pack_w8_kernel<<<(unsigned)cdiv(total, 256), 256, 0, s>>>(pp, N, K, total, (uint4*)dev_out, (float*)out->scale);
    SPEC_LAUNCH_CHECK("pack_w8_kernel");
    return SPEC_OK;
}

// ------------------------------------------------------------------ the GEMM
// Wp : [k_steps / KS][n_blocks][KS][64] u32x4_t   Xp : [k_steps][mb_pad][hi|lo][64] u32x4_t
// out: [splits][M][ldo] fp32 (slice stride = split_stride floats)
// MB row blocks (of 32) per workgroup tile; the 4 wavefronts are arranged WM along the rows x 4/WM
// along the columns.  A wavefront owns MB/WM row blocks and WM column blocks (the tile is always 128
// columns), so with WM = 2 every activation fragment read from LDS feeds two MFMAs and every weight
// fragment is read by two wavefronts (the second read hits the CU's L1): half the LDS traffic per MFMA.
// GROUPED (mixture of experts): blockIdx.z walks a device-side list of row tiles, tiles[0] = number of
// tiles, then (group, first row block and rows in use) pairs; group g multiplies by the matrix at Wp + g * w_group_stride
// (all groups have the same shape).  Tiles past the list's end exit at once.
// (Large row counts take the 192- and 256-row x 256-column tiles of gemm_big.hip.)
// W8: the weights are E4M3 codes, two k-steps per 16-byte word (half the weight bytes and load instructions); a
// fragment is widened to bf16 in registers right before its MFMAs (exact) and the output column's scale is applied to
// the accumulators in the epilogue.
// XF: the activations' operand format (operand.h): XF_HILO = hi + lo bf16 pairs against bf16 weights, two MFMAs per
// weight fragment and row block; XF_F16 = one fp16 value against fp16 weights, one MFMA.  The fused SwiGLU epilogue
// writes its output in the same format (gate/up and down projection take the same one).
// The activation slabs are requested LA slabs ahead (LA + 1 of them in LDS), so that waiting for one - vector loads return in order - does
// not also wait for the weights requested just before it.  What bounds a launch is how much of the weight stream is in flight, so every
// wait in the loop counts (load_to_lds says why that takes buffer loads), and nothing is fetched twice.  8B shape, us with every wait draining the
// queue and the last slab of the weights re-read past the end / now: QKV, output, gate/up and down projection at 4 rows 12.2, 8.9, 36.6, 19.9 /
// 10.6, 7.8, 35.0, 19.0; at 64 rows 14.3, 10.8, 40.0, 21.3 / 13.7, 10.1, 37.2, 20.3; at 96 rows 18.5, 14.3, 44.5, 24.5 / 16.2, 11.8, 42.3, 22.2; at 128
// rows 20.0, 15.3, 48.1, 26.7 / 19.1, 14.5, 46.5, 25.5.  With 8-bit weights at 4 rows 10.0, 7.1, 27.5, 14.3 / 8.5, 6.1, 21.6, 11.7, at 128 rows 17.8, 13.7, 40.7,
// 23.2 / 16.5, 12.9, 35.0, 21.1.
// EPI: PLAIN, SWIGLU (fused), or for an output that is not split along K - in the first place the head's logits, tens of megabytes that
// nobody reads before the launch ends - STREAM: stored past the L2s, it does not push out what the workgroups share there (head of 128256
// rows at 64, 74 and 128 rows: 171 -> 164, 198 -> 177, 184 -> 172 us; slices of a split output are small and gain nothing).  STREAM_SHARED: the
// same with several row tiles of 64 rows, whose workgroups also share the weights: ordinary instead of nontemporal loads (two 8B layers and a head of
// 40960 columns at 160 and 256 rows 625 -> 615, 769 -> 746 us; QKV of 10240 x 2048 and the attention's prologue at 256 rows 54.6 -> 52.7).  Not with tall
// tiles, of which two share them (a draft pass with a head of 32000 columns at 140 and 256 rows 492 -> 505, 624 -> 650), with one row tile
// (164 -> 181 at 64 rows) or where K is split.
template <int MB, int WM, int EPI, bool GROUPED = false, int NBW_T = WM, bool W8 = false, int XF = XF_HILO, int WD = GEMM_WD,
          int LA = gemm_slabs_ahead(MB, XF)>
__global__ __launch_bounds__(GEMM_THREADS, (MB >= 3 && WM == 1 && NBW_T == 2) ? 1 : 2) void gemm_bf16_kernel(
    const u32x4_t* __restrict__ Wp, const u32x4_t* __restrict__ Xp, float* __restrict__ out, int n_blocks, int k_steps,
    int ksteps_per_split, int mb_pad, int M, int N, int ldo, int64_t split_stride,
    const int32_t* __restrict__ tiles = nullptr, int64_t w_group_stride = 0, const float* __restrict__ wscale = nullptr)
{
    constexpr int KS = GEMM_KS;
    constexpr int KSW = W8 ? KS / 2 : KS;               // 16-byte words of one column block per lane and slab
    constexpr int MBW = MB / WM, NBW = NBW_T;
    constexpr int TILE_NB = (4 / WM) * NBW;             // 32-column blocks per workgroup tile
    static_assert(MB % WM == 0, "row blocks must divide over the wavefronts");
    constexpr int SLAB = KS * MB * 64 * XF;             // u32x4_t per slab (XF operand words per lane and k-step)
    constexpr int XPT = SLAB / GEMM_THREADS;            // u32x4_t per thread per slab
    static_assert(SLAB % GEMM_THREADS == 0, "a slab must divide over the threads");
    constexpr int NX = LA + 1;
    static_assert(LA <= WD && (WD == 2 || WD == 4), "the waits below count the weight loads behind an activation slab");
    // the fused SwiGLU epilogue re-uses the slabs as an fp32 transpose tile, which may be the larger of the two
    constexpr int EPI_WORDS = EPI != GEMM_EPI_SWIGLU ? 0 : (WM == 1 ? 32 * 129 : MB * 32 * 65) / 4 + 1;
    constexpr int LDS_WORDS = NX * SLAB > EPI_WORDS ? NX * SLAB : EPI_WORDS;
    __shared__ u32x4_t lds[LDS_WORDS];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int mh = wave % WM, np = wave / WM;
    int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if constexpr (!GROUPED) {
        const GemmTile tile_of = gemm_tile_of_workgroup();
        bx = tile_of.bx;
        by = tile_of.by;
        bz = tile_of.bz;
    }
    const int nb0 = bx * TILE_NB + np * NBW;
    const int ks0 = by * ksteps_per_split;
    int ks1 = ks0 + ksteps_per_split;
    if (ks1 > k_steps) ks1 = k_steps;
    const int n_slabs = (ks1 - ks0) / KS;
    int mblk0 = bz * MB;                        // first 32-row block of this tile
    if constexpr (GROUPED) {
        if (bz >= tiles[0]) return;
        Wp += (int64_t)tiles[1 + 2 * bz] * w_group_stride;
        if constexpr (W8) wscale += (int64_t)tiles[1 + 2 * bz] * w_group_stride * 4;   // a group's scales sit in its own region
        mblk0 = moe_tile_block(tiles[2 + 2 * bz]);
        M = mblk0 * 32 + moe_tile_rows(tiles[2 + 2 * bz]);                 // padding rows are not stored
    }

    // slab s of column block j of this wavefront: wptr[j] + s * wslab (+ the lane), all scalar
    const u32x4_t* wptr[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
        wptr[j] = Wp + (((int64_t)(ks0 / KS) * n_blocks + (nb0 + j < n_blocks ? nb0 + j : 0)) * KSW) * 64;
    const int64_t wslab = (int64_t)n_blocks * KSW * 64;
    float wsc[NBW];                                     // 8-bit weights: this lane's column scales
#pragma unroll
    for (int j = 0; j < NBW; ++j) wsc[j] = 1.0f;
    const u32x4_t* xbase = Xp + ((int64_t)ks0 * mb_pad + (int64_t)mblk0) * (64 * XF);

    f32x16_t acc[MBW][NBW];
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < NBW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // the weight stream runs WD slabs ahead of the MFMAs: a register ring, each entry refilled
    // right after its last use
    u32x4_t w[WD][KSW][NBW];
    auto load_w = [](const u32x4_t* p) {
        if constexpr (EPI == GEMM_EPI_STREAM_SHARED) return *p;
        else return __builtin_nontemporal_load(p);
    };

    // The activation slabs go from memory straight into LDS.  The offsets are scalar, and the base moves with the slab, so none grows with K.
    auto stage_x = [&](int slab, int tobuf) {
        const u32x4_t* src = xbase + (int64_t)slab * KS * mb_pad * (64 * XF);
#pragma unroll
        for (int j = 0; j < XPT; ++j) {
            const int c = wave + 4 * j, kl = c / (MB * XF), rem = c % (MB * XF);       // 1 KiB chunk c of the slab
            load_to_lds(src, (kl * mb_pad * XF + rem) * 1024, lds + tobuf * SLAB + c * 64);
        }
    };
    int buf = 0;
    // No branch may sit between the loads and their use: the compiler can only count outstanding
    // loads (s_waitcnt vmcnt(n)) along straight-line code, and falls back to draining the whole
    // queue otherwise.  So every slab issues its prefetches unconditionally; past the end they read
    // activations that are in the caches (results unused; the last slab of the weights would come from HBM once more).
    auto slab_body = [&](auto slot_c, int s) {
        constexpr int SLOT = decltype(slot_c)::value;
        const int s_x = s + LA < n_slabs ? s + LA : n_slabs - 1;
        // the oldest loads of this slab, into the buffer that the last slab has freed
        stage_x(s_x, buf > 0 ? buf - 1 : NX - 1);
        // keep these loads HERE: left alone, the scheduler sinks them to the end of the slab, next to the LDS
        // stores that consume them, and the whole round trip to L2 is then paid once per slab
        const u32x4_t* w_src[NBW];
#pragma unroll
        for (int j = 0; j < NBW; ++j) w_src[j] = s + WD < n_slabs ? wptr[j] + (int64_t)(s + WD) * wslab : xbase;
        __builtin_amdgcn_sched_barrier(0);
        // LDS reads run one k-step ahead of the MFMAs that use them (two register sets): with one or two
        // wavefronts per SIMD nothing else would hide the LDS latency.  The scheduling barriers keep that order.
        u32x4_t a[2][MBW][XF];
        auto read_a = [&](int set, int kk) {
#pragma unroll
            for (int i = 0; i < MBW; ++i)
#pragma unroll
                for (int part = 0; part < XF; ++part)
                    a[set][i][part] = lds[buf * SLAB + ((kk * MB + mh * MBW + i) * XF + part) * 64 + lane];
        };
        read_a(0, 0);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            if (kk + 1 < KS) read_a((kk + 1) & 1, kk + 1);
            __builtin_amdgcn_sched_barrier(0);
            u32x4_t wk[NBW];                             // this k-step's weight fragments in the activations' 16-bit type
#pragma unroll
            for (int j = 0; j < NBW; ++j) {
                if constexpr (W8) {
                    wk[j] = widen_e4m3x8<XF == XF_F16>(w[SLOT][kk >> 1][j][(kk & 1) * 2], w[SLOT][kk >> 1][j][(kk & 1) * 2 + 1]);
                } else {
                    wk[j] = w[SLOT][kk][j];
                }
            }
            // hi products of all blocks first, then the lo products: two MFMAs on one accumulator are never adjacent
#pragma unroll
            for (int part = 0; part < XF; ++part)
#pragma unroll
                for (int i = 0; i < MBW; ++i)
#pragma unroll
                    for (int j = 0; j < NBW; ++j) {
                        if constexpr (XF == XF_F16)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a[kk & 1][i][part]),
                                                                               __builtin_bit_cast(f16x8_t, wk[j]), acc[i][j], 0, 0, 0);
                        else
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[kk & 1][i][part]),
                                                                                __builtin_bit_cast(bf16x8_t, wk[j]), acc[i][j], 0, 0, 0);
                    }
            if (!W8 || (kk & 1)) {                       // (8-bit: a word serves two k-steps and is refilled after the second)
#pragma unroll
                for (int j = 0; j < NBW; ++j)
                    w[SLOT][W8 ? kk >> 1 : kk][j] = load_w(w_src[j] + (W8 ? kk >> 1 : kk) * 64 + lane);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ... and the weight loads of this slab stay above the LDS stores, so that waiting for the (older)
        // activation loads does not drain the weight stream
        __builtin_amdgcn_sched_barrier(0);
        // Wait for the next slab's transfers into LDS only: the weight reloads (KSW * NBW a slab) and the transfers that were issued
        // after them stay in flight (__syncthreads would drain the whole queue).  No wavefront reads the next buffer
        // before this barrier, and all have finished reading this one when they pass it.
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(KSW * NBW + (LA - 1) * (KSW * NBW + XPT)));
        __builtin_amdgcn_s_barrier();
        buf = buf + 1 < NX ? buf + 1 : 0;
    };

    // n_slabs is a multiple of WD (K % (16 * GEMM_KUNIT) == 0, split sizes are rounded to two slabs, and a ring of four is taken
    // where they are multiples of four)
    if (n_slabs > 0) {
        if constexpr (W8) {
            // Fetched before anything else and known to have arrived (the first wait below, then the empty asm behind the loop that
            // ties the values to that point) on every path into the epilogue: a load the compiler may still count as
            // outstanding there makes it wait with vmcnt(0) before each of the 64 stores, which serialises them.
#pragma unroll
            for (int j = 0; j < NBW; ++j)
                if (nb0 + j < n_blocks) wsc[j] = wscale[(nb0 + j) * 32 + (lane & 31)];
        }
#pragma unroll
        for (int d = 0; d < LA; ++d) stage_x(d, d);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < WD; ++d)
#pragma unroll
            for (int i = 0; i < KSW; ++i)
#pragma unroll
                for (int j = 0; j < NBW; ++j) w[d][i][j] = load_w(wptr[j] + (int64_t)d * wslab + i * 64 + lane);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((LA - 1) * XPT + KSW * NBW * WD));
        __builtin_amdgcn_s_barrier();
        // The loop runs at least once, has no remainder and is not peeled: every load is then used on the only way on from it.  Otherwise the compiler
        // drops those that nobody reads, or moves them behind a wait that counts them (tests/test_gemm_waits.py walks the built code for that; draining
        // the queue at the end instead costs 0.1 us a launch, 10 us of a step at batch 1).
        int s = 0;
#pragma clang loop unroll(disable)
        do {
            slab_body(std::integral_constant<int, 0>{}, s);
            slab_body(std::integral_constant<int, 1>{}, s + 1);
            if constexpr (WD == 4) {
                slab_body(std::integral_constant<int, 2>{}, s + 2);
                slab_body(std::integral_constant<int, 3>{}, s + 3);
            }
            s += WD;
        } while (s < n_slabs);
        if constexpr (W8) {
#pragma unroll
            for (int j = 0; j < NBW; ++j) asm volatile("" : "+v"(wsc[j]));
        }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(KSW * NBW));       // no transfer into LDS is left when the epilogue re-uses it or the workgroup ends
    }

    if constexpr (EPI == GEMM_EPI_SWIGLU && WM == 1 && NBW == 1) {
        // 128-column tile of the 1 x 4 arrangement with one column block per wavefront: wavefronts 0 and 2 hold the gates,
        // 1 and 3 the ups of 2 x 32 hidden channels (the column blocks of a pair are both inside the matrix or both outside).  The raw accumulators go through LDS one row block at a time, and
        // silu(gate) * up is formed on the way out.  Odd row-block counts use expf as swiglu_pack_kernel does, which they take where K
        // is split: fused or not, the result is the same bits.  (Even ones are never split while the fusion is on.)
        float* tile = (float*)lds;                              // [32 rows][129]
        uint4* xo = (uint4*)out;
#pragma unroll
        for (int i = 0; i < MBW; ++i) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                tile[row * 129 + np * 32 + (lane & 31)] = W8 ? acc[i][0][r] * wsc[0] : acc[i][0][r];
            }
            __syncthreads();
            {
                const int e = threadIdx.x;                      // 32 rows x 8 groups of 8 hidden channels
                const int row = e >> 3, g8 = e & 7;
                const int m = (mblk0 + i) * 32 + row, f = bx * 64 + g8 * 8;
                if (m < M && f < N / 2) {
                    const float* src = tile + row * 129 + (g8 >> 2) * 64 + (g8 & 3) * 8;
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) { const float g = src[j], u = src[32 + j]; v[j] = g / (1.0f + (MB % 2 ? expf(-g) : __expf(-g))) * u; }
                    xp_store8_t<XF>(xo, m, f, mb_pad, v);
                }
            }
        }
        return;
    } else if constexpr (EPI == GEMM_EPI_SWIGLU && WM == 1) {
        // 256-column tile of the 1 x 4 arrangement (each wavefront: all MB row blocks, gate and up of 32 hidden channels):
        // the same transpose through LDS, one row block (32 rows x 128 channels) at a time.
        static_assert(EPI != GEMM_EPI_SWIGLU || WM != 1 || NBW == 2, "fused SwiGLU needs two column blocks per wavefront");
        float* tile = (float*)lds;                              // [32 rows][129]
        uint4* xo = (uint4*)out;
#pragma unroll
        for (int i = 0; i < MBW; ++i) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float g = acc[i][0][r], u = acc[i][NBW - 1][r];
                if constexpr (W8) {
                    g *= wsc[0];
                    u *= wsc[NBW - 1];
                }
                const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                tile[row * 129 + np * 32 + (lane & 31)] = g / (1.0f + __expf(-g)) * u;
            }
            __syncthreads();
            for (int e = threadIdx.x; e < 32 * 16; e += GEMM_THREADS) {
                const int row = e >> 4, g8 = e & 15;
                const int m = (mblk0 + i) * 32 + row, f = bx * 128 + g8 * 8;
                if (m >= M || f >= N / 2) continue;
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = tile[row * 129 + g8 * 8 + j];
                xp_store8_t<XF>(xo, m, f, mb_pad, v);
            }
        }
        return;
    } else if constexpr (EPI == GEMM_EPI_SWIGLU) {
        // The weights of the gate/up projection are tiled with gate and up column blocks interleaved,
        // so this wavefront's two accumulators hold gate and up of the same 32 hidden channels:
        // silu(gate) * up in registers, transposed through LDS (free after the main loop) into rows,
        // and written as hi + lo bf16 in the operand order the down projection reads.
        static_assert(EPI != GEMM_EPI_SWIGLU || NBW == 2, "fused SwiGLU needs two column blocks per wavefront");
        float* tile = (float*)lds;                              // [MB*32 rows][65]
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MBW; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float g = acc[i][0][r], u = acc[i][NBW - 1][r];
                if constexpr (W8) {
                    g *= wsc[0];
                    u *= wsc[NBW - 1];
                }
                int row = (mh * MBW + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                tile[row * 65 + np * 32 + (lane & 31)] = g / (1.0f + __expf(-g)) * u;
            }
        __syncthreads();
        uint4* xo = (uint4*)out;
        for (int e = threadIdx.x; e < MB * 32 * 8; e += GEMM_THREADS) {
            int row = e >> 3, g8 = e & 7;
            int m = mblk0 * 32 + row, f = bx * 64 + g8 * 8;
            if (m >= M || f >= N / 2) continue;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = tile[row * 65 + g8 * 8 + j];
            xp_store8_t<XF>(xo, m, f, mb_pad, v);
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
                if (m >= M) continue;
                const float v = W8 ? acc[i][j][r] * sc : acc[i][j][r];
                if constexpr (EPI >= GEMM_EPI_STREAM) __builtin_nontemporal_store(v, o + (int64_t)m * ldo + n);
                else o[(int64_t)m * ldo + n] = v;
            }
    }
}

// Tile shapes.  Up to 4 row blocks (128 rows) a launch has one kind of tile: MB = min(row blocks, gemm_max_mb) x 128
// columns.  From gemm_big_min_blocks row blocks on (0 = never) the 256-column tile with 8 or 6 row blocks is available
// too, and each GEMM takes it when it still fills the chip: at least gemm_big_min_tiles (200) tiles, or - K split, two or more tiles of
// rows - at least 192 workgroups of 32 or more k-steps each (a 256 x 256 tile with a short K spends its time in prologue
// and epilogue; with one tile of rows the extra split-K slices cost the consumers more than the GEMM gains; and a fused
// SwiGLU epilogue cannot split K at all).  Both kinds read the same activation buffer, so its rows are padded
// to a multiple of both tile heights: 8 blocks, or 12 where that pads less (then the big tile has 6 row blocks).
static int gemm_big_mb(int M)
{
    const int nb = (int)cdiv(M, 32), from = tune("gemm_big_min_blocks");
    if (from <= 0 || nb < from || nb < 5) return 0;
    return cdiv(nb, 12) * 12 < cdiv(nb, 8) * 8 ? 6 : 8;
}
int gemm_mb(int M) { int mb = (int)cdiv(M, 32), cap = tune("gemm_max_mb"); cap = cap < 1 ? 1 : (cap > 4 ? 4 : cap); return mb > cap ? cap : mb; }
int gemm_mb_pad(int M)
{
    const int nb = (int)cdiv(M, 32), big = gemm_big_mb(M);
    if (big) return (int)cdiv(nb, big == 6 ? 12 : 8) * (big == 6 ? 12 : 8);
    const int mb = gemm_mb(M);
    return (int)cdiv(nb, mb) * mb;
}

struct GemmShape { int mb, tile_nb, kunit, m_tiles, n_tiles; bool wide = false, one_block = false; };
GemmShape gemm_shape(const PackedW& W, int M, bool fused_swiglu)      // (not static: the dispatch has a test)
{
    GemmShape g;
    const int pad = gemm_mb_pad(M), big = gemm_big_mb(M);
    if (big) {
        const int64_t tiles = (int64_t)cdiv(W.n_blocks, 8) * (pad / big);
        int64_t splits = tune("gemm_wg_target") / tiles;
        if (splits > W.k_steps / 32) splits = W.k_steps / 32;
        if (splits < 1) splits = 1;
        if (tiles >= tune("gemm_big_min_tiles") || (!fused_swiglu && pad / big >= 2 && tiles * splits >= 192)) {
            g.mb = big; g.tile_nb = 8; g.kunit = GEMM_KS * 2;
            g.m_tiles = pad / big; g.n_tiles = (int)cdiv(W.n_blocks, 8);
            if (big == 8 && cdiv(M, 32) <= 6) g.mb = 6;                 // 129..192 rows: the one tile needs 6 row blocks only
            return g;
        }
    }
    g.mb = big ? 4 : gemm_mb(M);
    g.tile_nb = 4;
    g.kunit = GEMM_KS * 2;                              // k-steps per split: whole pairs of slabs
    g.m_tiles = pad / g.mb; g.n_tiles = (int)cdiv(W.n_blocks, 4);
    // One tile of 64 or 128 rows, plain epilogue, K unsplit because the columns alone give enough workgroups (the LM head): 256-column
    // tiles with the wavefronts 1 x 4 - no weight fragment fetched twice, the activation slab serves twice the columns.
    // (With K split to make up the workgroups the extra slices cost the consumers what the GEMM gains.)
    if ((g.mb == 4 || g.mb == 2) && g.m_tiles == 1 && !fused_swiglu && tune("gemm_wide4") > 0 && W.n_blocks % 8 == 0 && W.n_blocks / 8 >= tune("gemm_wide4")) {
        g.wide = true; g.tile_nb = 8; g.n_tiles = W.n_blocks / 8; g.kunit = GEMM_KS * 2;
        return g;
    }
    // 97..128 rows: two tiles of 64 rows x 256 columns (wavefronts 1 x 4) instead of one of 128 x 128 (2 x 2): the same
    // number of workgroups and K splits, the same MFMAs per workgroup and slab, but no weight fragment fetched twice and half
    // the activation slab per workgroup; the second row tile's weights come from L2 (the two are neighbours on one XCD).
    // The same holds for up to gemm_split_rows 128-row tiles (129..256 rows at 2); a 64-row tile that would hold padding
    // only is not launched.
    // 129..256 rows where K is not split (the fused gate/up projection): two tiles of 96 or 128 rows instead of three or four of
    // 64 - 2 x 112 workgroups fit the chip at once, 3 x 112 and 4 x 112 do not.
    // 97..128 rows with fp16 activations: one tile of 128 rows x 128 columns with the wavefronts 1 x 4, each its own column
    // block over all four row blocks.  Every weight fragment is then fetched by exactly one wavefront of one workgroup
    // (the pair of 64-row tiles fetches each twice: the second time as an L2 hit, but through the same L1 and memory
    // pipeline as the weight stream), at the price of one LDS read per MFMA, which the single fp16 MFMA per fragment leaves room for:
    // gate/up 56 -> 50 us, down 31 -> 26 us at the 8B shape.  With hi + lo operands the pair stays ahead.
    // 33..64 rows: the same arrangement instead of 2 x 2, in either format (at 64 rows of the 8B shape gate/up 56.3 -> 42.1 us,
    // down 29.0 -> 24.6, QKV and output projection 16.3 -> 14.7 on average): the activation slab is half as large and the second
    // fetch of every weight fragment was what the 2 x 2 arrangement waited for.
    if ((g.mb == 2 || (g.mb == 4 && W.f16)) && g.m_tiles == 1 && tune("gemm_one_block") != 0 && W.n_blocks % 4 == 0) {
        g.one_block = true; g.tile_nb = 4; g.n_tiles = W.n_blocks / 4; g.kunit = GEMM_KS * 2;
        return g;
    }
    if (g.mb == 4 && g.m_tiles <= tune("gemm_split_rows") && W.n_blocks % 8 == 0) {
        const int nb = (int)cdiv(M, 32);
        // 129..256 rows, plain epilogue: the tall tiles too (K = 4096 unless stated; us, 64-row / tall)
        //  - where K stays whole in either and their workgroups fill the chip in one round, which the 64-row ones exceed: two 8B layers and a head of 24576
        //    columns at 160 and 256 rows 564 / 557, 681 / 658, of 32000 598 / 569, 698 / 669; a draft pass with 32000 at 256 rows 666 / 624.  Not with 8-bit
        //    weights and four row blocks: 602 / 609, 616 / 618;
        //  - where the 64-row ones leave K whole on part of the chip and the tall ones get enough slices to do less each (1.5 or 2 times the rows in 1/2 or
        //    1/3 of K; projection and the reader of its slices): 9216, 10240 columns at 256 rows 78.0 / 67.7, 78.5 / 69.6; 12288, 16384 at 160 88.7 / 75.9, 97.4 /
        //    86.1; with two slices for twice the rows 92.5 / 89.7 at best (K = 4096), 72.8 / 74.1 (K = 2560).  The slices cost the same whatever K: 9216 columns at
        //    256 rows 64.0 / 60.2 at K = 3072, 57.7 / 57.0 at 2560, 50.1 / 53.0 at 2048.  Never the head, which is not split (with
        //    one of 16384 columns at 160 and 256 rows 530 / 552, 627 / 653);
        //  - K split either way, fp16 inputs against 16-bit weights, from an eighth of the chip on (down projection and the norm, K = 3.5 N: 4096 columns at 160
        //    and 256 rows 61.3 / 57.7, 69.9 / 65.6, 8192 columns 192 / 144, 200 / 162; 3072 at 160 46.2 / 45.4, 2048 at 256 38.7 / 40.7, 1024 28.8 / 32.5).
        //    Hi + lo (20.3 / 23.0) and 8-bit weights (49.4 / 49.4, 58.4 / 60.2) lose by the additional slices.
        const int cols = W.n_blocks / 8, mb_tall = nb <= 6 ? 3 : 4, target = tune("gemm_wg_target");
        const int n_tall = (int)cdiv(nb, mb_tall) * cols, n_64 = (int)cdiv(nb, 2) * cols, slices = std::max(1, target / n_tall);
        const bool fills = n_tall * 4 >= target * 3 && n_tall <= target && !(W.w8 && mb_tall == 4);
        const bool idle = !W.whole && n_64 * 2 > target && n_64 <= target && mb_tall < 2 * slices && W.k_steps >= 160;
        const bool split = !W.whole && W.f16 && !W.w8 && n_64 * 8 > target && n_64 <= target;
        g.mb = nb >= 5 && (fused_swiglu || fills || idle || split) && tune("gemm_tiles_96") != 0 ? mb_tall : 2;
        g.m_tiles = (int)cdiv(nb, g.mb); g.wide = true; g.tile_nb = 8; g.n_tiles = W.n_blocks / 8; g.kunit = GEMM_KS * 2;
        return g;
    }
    return g;
}

int gemm_pick_splits(const PackedW& W, int M, int forced)
{
    const GemmShape g = gemm_shape(W, M, false);
    const int unit = g.kunit;
    int max_splits = W.k_steps / (tune("gemm_min_ksteps") > unit ? tune("gemm_min_ksteps") : unit);
    if (max_splits < 1) max_splits = 1;
    int splits = forced > 0 ? forced : tune("gemm_wg_target") / (g.n_tiles * g.m_tiles);
    if (splits < 1) splits = 1;
    if (splits > max_splits) splits = max_splits;
    int kps = (int)cdiv(cdiv(W.k_steps, splits), unit) * unit;
    return (int)cdiv(W.k_steps, kps);
}

// Whether the gate/up projection forms silu(gate) * up in its epilogue.
bool gemm_can_fuse_swiglu(const PackedW& W, int M, int splits)
{
    if (splits != 1) return false;
    const GemmShape g = gemm_shape(W, M, true);
    // odd row-block counts (a tile with one column block per wavefront): where K would not be split anyway, by the tile count or by
    // splits_gu - with few column tiles the split projection and its pass over the slices keep more of the chip busy.  (At 4 rows of
    // the 8B shape the fused launch takes the 37.5 us of the plain one and saves the 4.6 us pass per layer.)
    if (g.mb % 2 != 0 && !g.wide) return gemm_pick_splits(W, M, tune("splits_gu")) == 1;
    return true;
}

// out must hold splits * M * ldo floats; with swiglu (gate/up projection, splits == 1) out is instead the operand buffer of
// silu(gate) * up, [N/2] channels wide, in the format the matrix takes (hi + lo or fp16).
// Returns SPEC_EUNSUPPORTED (nothing launched) if swiglu is asked for a shape it cannot fuse.
spec_status launch_gemm_bf16(const PackedW& W, const bf16_t* Xp, int M, float* out, int ldo, int splits, bool swiglu, hipStream_t s)
{
    const GemmShape g = gemm_shape(W, M, swiglu);
    const int mb = g.mb, mb_pad = gemm_mb_pad(M);
    int kps = (int)cdiv(cdiv(W.k_steps, splits), g.kunit) * g.kunit;
    dim3 grid((unsigned)g.n_tiles, (unsigned)cdiv(W.k_steps, kps), (unsigned)g.m_tiles);
    int64_t stride = (int64_t)M * ldo;
    const u32x4_t* wp = (const u32x4_t*)W.data;
    const u32x4_t* xp = (const u32x4_t*)Xp;
    if (swiglu && !gemm_can_fuse_swiglu(W, M, splits)) { set_error("gemm: SwiGLU cannot be fused for this shape"); return SPEC_EUNSUPPORTED; }
    const int epi = swiglu ? GEMM_EPI_SWIGLU : (grid.y > 1 ? GEMM_EPI_PLAIN : (grid.z > 1 ? GEMM_EPI_STREAM_SHARED : GEMM_EPI_STREAM));
    const bool crowded = gemm_crowded((int64_t)grid.x * grid.z, W.w8, mb, g.one_block || mb == 1);
#define SPEC_GEMM_CALL(...) gemm_bf16_kernel<__VA_ARGS__><<<grid, GEMM_THREADS, 0, s>>>(wp, xp, out, W.n_blocks, W.k_steps, kps, mb_pad, M, W.N, ldo, stride, nullptr, 0, W.scale)
    // MB row blocks, WM wavefronts along the rows, NBW column blocks per wavefront.  One column block and 8-bit weights, half the bytes a slab: a weight ring
    // of four slabs where the split allows it and the launch does not crowd the chip (gate/up of the 8B shape at 4 and 128 rows 26.3 -> 22.9, 39.6 -> 36 us;
    // heads of 64000 and 151936 columns, K = 2048, at 64 and 32 rows 32.7 / 31.9, 61.4 / 59.3 with four / two)
#define SPEC_GEMM_TILE(MB, WM, NBW, E, W8, XF) do { \
        constexpr int FAR = gemm_slabs_ahead(MB, XF), NEAR = (NBW == 1 || WM == 2 || (W8 && MB == 2)) && E != GEMM_EPI_PLAIN ? 1 : FAR; \
        if (crowded) SPEC_GEMM_CALL(MB, WM, E, false, NBW, W8, XF, 2, NEAR); \
        else if (W8 && NBW == 1 && kps % (4 * GEMM_KS) == 0) SPEC_GEMM_CALL(MB, WM, E, false, NBW, W8, XF, W8 && NBW == 1 ? 4 : 2, FAR); \
        else SPEC_GEMM_CALL(MB, WM, E, false, NBW, W8, XF, 2, FAR); } while (0)
    // the four combinations of 8-bit or 16-bit weights and hi + lo or fp16 activations
#define SPEC_GEMM_BY_TYPE(MB, WM, NBW, E) do { \
        if (W.w8) { if (W.f16) SPEC_GEMM_TILE(MB, WM, NBW, E, true, XF_F16); else SPEC_GEMM_TILE(MB, WM, NBW, E, true, XF_HILO); } \
        else { if (W.f16) SPEC_GEMM_TILE(MB, WM, NBW, E, false, XF_F16); else SPEC_GEMM_TILE(MB, WM, NBW, E, false, XF_HILO); } } while (0)
#define SPEC_GEMM_F16(MB, WM, NBW, E) do { if (W.w8) SPEC_GEMM_TILE(MB, WM, NBW, E, true, XF_F16); else SPEC_GEMM_TILE(MB, WM, NBW, E, false, XF_F16); } while (0)
#define SPEC_GEMM_BY_EPI(BY_TYPE, MB, WM, NBW, SHARED) do { \
        if (epi == GEMM_EPI_SWIGLU) BY_TYPE(MB, WM, NBW, GEMM_EPI_SWIGLU); \
        else if (epi == GEMM_EPI_PLAIN) BY_TYPE(MB, WM, NBW, GEMM_EPI_PLAIN); \
        else if (epi == GEMM_EPI_STREAM_SHARED) BY_TYPE(MB, WM, NBW, SHARED); \
        else BY_TYPE(MB, WM, NBW, GEMM_EPI_STREAM); } while (0)
    switch (mb) {
        case 1: SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 1, 1, 1, GEMM_EPI_STREAM); break;
        case 2:
            if (g.one_block) SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 2, 1, 1, GEMM_EPI_STREAM);
            else if (g.wide) SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 2, 1, 2, GEMM_EPI_STREAM_SHARED);
            else SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 2, 2, 2, GEMM_EPI_STREAM);
            break;
        case 3:
            if (g.wide) SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 3, 1, 2, GEMM_EPI_STREAM);
            else SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 3, 1, 1, GEMM_EPI_STREAM);
            break;
        case 6: case 8: return launch_gemm_big(W, Xp, M, mb, mb_pad, out, ldo, kps, swiglu, grid, s);
        default:
            if (g.one_block) SPEC_GEMM_BY_EPI(SPEC_GEMM_F16, 4, 1, 1, GEMM_EPI_STREAM);
            else if (g.wide) SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 4, 1, 2, GEMM_EPI_STREAM);
            else SPEC_GEMM_BY_EPI(SPEC_GEMM_BY_TYPE, 4, 2, 2, GEMM_EPI_STREAM);
            break;
    }
#undef SPEC_GEMM_BY_EPI
#undef SPEC_GEMM_F16
#undef SPEC_GEMM_BY_TYPE
#undef SPEC_GEMM_TILE
#undef SPEC_GEMM_CALL
    SPEC_LAUNCH_CHECK("gemm_bf16_kernel");
    return SPEC_OK;
}

// Grouped GEMM over a device-side tile list (see the kernel): 64-row tiles, group g uses the matrix g *
// group_stride elements after W0; Xp and the output cover rows_pad rows (a multiple of 64).  With swiglu
// the output is the hi + lo operand buffer of silu(gate) * up (rows_pad / 32 row blocks per k-step).
spec_status launch_gemm_bf16_grouped(const PackedW& W0, int64_t group_stride, const bf16_t* Xp, int rows_pad, int max_tiles,
                                     const int32_t* tiles, float* out, int ldo, bool swiglu, hipStream_t s)
{
    if (rows_pad % 64 || max_tiles < 1 || W0.k_steps % GEMM_KUNIT) { set_error("grouped gemm: bad shape"); return SPEC_EINVAL; }
    dim3 grid((unsigned)cdiv(W0.n_blocks, 4), 1, (unsigned)max_tiles);
    const u32x4_t* wp = (const u32x4_t*)W0.data;
    const u32x4_t* xp = (const u32x4_t*)Xp;
    // distance between the groups' matrices in 16-byte words (group_stride: bf16 elements, or bytes of a whole 8-bit region,
    // codes and scales, so that the scales of group g sit g * stride behind those of group 0 as well)
    const int64_t stride16 = W0.w8 ? group_stride / 16 : group_stride / 8;
    // Two tile shapes of 64 rows: 128 columns with the wavefronts 2 x 2, or 256 columns with the wavefronts 1 x 4 (each
    // its own two column blocks: no weight fragment is fetched twice and the activation slab serves twice the columns,
    // which is what the expert GEMMs - few rows, all weights touched - are bound by).
    const bool wide = tune("moe_wide_tiles") != 0 && W0.n_blocks % 8 == 0;
    if (wide) grid.x = (unsigned)cdiv(W0.n_blocks, 8);
#define SPEC_GROUPED_LAUNCH(WMV, E, W8V, XFV) gemm_bf16_kernel<2, WMV, E, true, 2, W8V, XFV><<<grid, GEMM_THREADS, 0, s>>>( \
        wp, xp, out, W0.n_blocks, W0.k_steps, W0.k_steps, rows_pad / 32, rows_pad, W0.N, ldo, 0, tiles, stride16, W0.scale)
#define SPEC_GROUPED_BY_TYPE(WMV, E) do { \
        if (W0.w8) { if (W0.f16) SPEC_GROUPED_LAUNCH(WMV, E, true, XF_F16); else SPEC_GROUPED_LAUNCH(WMV, E, true, XF_HILO); } \
        else { if (W0.f16) SPEC_GROUPED_LAUNCH(WMV, E, false, XF_F16); else SPEC_GROUPED_LAUNCH(WMV, E, false, XF_HILO); } } while (0)
#define SPEC_GROUPED_LAUNCH_E(E) do { if (wide) SPEC_GROUPED_BY_TYPE(1, E); else SPEC_GROUPED_BY_TYPE(2, E); } while (0)
    if (swiglu) SPEC_GROUPED_LAUNCH_E(GEMM_EPI_SWIGLU); else SPEC_GROUPED_LAUNCH_E(GEMM_EPI_PLAIN);
#undef SPEC_GROUPED_LAUNCH_E
#undef SPEC_GROUPED_BY_TYPE
#undef SPEC_GROUPED_LAUNCH
    SPEC_LAUNCH_CHECK("gemm_bf16_kernel (grouped)");
    return SPEC_OK;
}

}  // namespace specv
