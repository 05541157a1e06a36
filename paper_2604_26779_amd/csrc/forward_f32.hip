// Generic fp32 verify forward: plain kernels for any model shape (the tiny fp32 configuration and
// a bring-up reference for shapes the MFMA path does not cover).  Same step order as the bf16
// path: embed -> per layer [RMSNorm, QKV, rotary + speculative KV write, causal attention over the
// paged cache, O + residual, RMSNorm, gate/up, SwiGLU, down + residual] -> final RMSNorm -> head.
#include <initializer_list>
#include <type_traits>
#include <utility>

#include "common.h"

namespace specv {

// ------------------------------------------------------------------ small kernels
// x = embed[token]; and, once per forward pass, every input row's position and where its key and value go: row_at[m] = (position, page *
// SPEC_PAGE_SIZE + position in the page, or -1 if the entry was dropped or its sequence holds no page for it)
__global__ void f32_embed_kernel(const int32_t* __restrict__ tokens, const float* __restrict__ embed, int d, int vocab, int T, KvView kv,
                                 float* __restrict__ x, int2* __restrict__ row_at)
{
    int m = blockIdx.x;
    if (threadIdx.x == 0) {
        const int seq = kv.entry_seq[m / T];           // -1: the entry was dropped (id out of range or named twice)
        const int pos = seq >= 0 ? kv.ctx_len[seq] + m % T : 0, lp = pos / SPEC_PAGE_SIZE;
        const bool writable = seq >= 0 && lp < kv.n_held[seq];
        row_at[m] = make_int2(pos, writable ? kv.page_table[(int64_t)seq * kv.max_pages + lp] * SPEC_PAGE_SIZE + pos % SPEC_PAGE_SIZE : -1);
    }
    int t = tokens[m];
    t = t < 0 ? 0 : (t >= vocab ? vocab - 1 : t);
    for (int c = threadIdx.x; c < d; c += blockDim.x) x[(int64_t)m * d + c] = embed[(int64_t)t * d + c];
}

__global__ __launch_bounds__(256) void f32_rmsnorm_kernel(const float* __restrict__ x, const float* __restrict__ gain,
                                                          int d, float eps, float* __restrict__ y)
{
    int m = blockIdx.x;
    const float* xr = x + (int64_t)m * d;
    float ss = 0.f;
    for (int c = threadIdx.x; c < d; c += 256) ss += xr[c] * xr[c];
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    __shared__ float part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = part[0] + part[1] + part[2] + part[3];
    float r = 1.0f / sqrtf(tot / (float)d + eps);
    for (int c = threadIdx.x; c < d; c += 256) y[(int64_t)m * d + c] = xr[c] * r * gain[c];
}

// y[m][n] (+)= sum_k a[m][k] * w[n][k], y has leading dimension ldy;
// 32x32 output tile per workgroup, 16x16 threads, 2x2 outputs per thread
template <bool ACCUM>
__global__ __launch_bounds__(256) void f32_gemm_kernel(const float* __restrict__ a, const float* __restrict__ w, int M,
                                                       int N, int K, float* __restrict__ y, int ldy)
{
    __shared__ float sa[32][33], sw[32][33];
    int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
    for (int k0 = 0; k0 < K; k0 += 32) {
        for (int i = threadIdx.x; i < 32 * 32; i += 256) {
            int r = i >> 5, c = i & 31;
            int kk = k0 + c;
            sa[r][c] = (m0 + r < M && kk < K) ? a[(int64_t)(m0 + r) * K + kk] : 0.f;
            sw[r][c] = (n0 + r < N && kk < K) ? w[(int64_t)(n0 + r) * K + kk] : 0.f;
        }
        __syncthreads();
#pragma unroll 8
        for (int c = 0; c < 32; ++c) {
            float a0 = sa[ty][c], a1 = sa[ty + 16][c], w0 = sw[tx][c], w1 = sw[tx + 16][c];
            acc[0][0] += a0 * w0; acc[0][1] += a0 * w1; acc[1][0] += a1 * w0; acc[1][1] += a1 * w1;
        }
        __syncthreads();
    }
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            int m = m0 + ty + 16 * i, n = n0 + tx + 16 * j;
            if (m < M && n < N) {
                float* dst = y + (int64_t)m * ldy + n;
                *dst = ACCUM ? *dst + acc[i][j] : acc[i][j];
            }
        }
}

// The same product for few rows: up to three matrices over the same input side by side (their columns follow each other in y).
// A wavefront computes 8 rows x 4 columns with K spread over its lanes, so that a narrow projection still gives hundreds of
// wavefronts, every load is 16 bytes and the only wait is one trip to memory per 256 of K; the 32 sums are folded over the
// lanes by exchanging halves (32 shuffles).  K % 4 == 0, rows and matrices 16-byte aligned.  Bound by the launch and two trips to memory
// at the sizes of the tiny configuration (3.8 us for N = 1024, K = 256 at 16 rows; the tiled kernel 15.2).
// Around the product (FORM; at these sizes a kernel of its own costs more than what it computes: norm 2.9 us, SwiGLU 2.4, rotary 4.4):
//   NORM    the rows are RMS-normalised: the sum of squares is folded beside the products, the gain goes to the weights, 1 / rms to the result;
//   SWIGLU  two matrices, gate and up; a wavefront takes two columns of each and writes silu(gate) * up;
//   ROPE    the three matrices are q, k and v; a wavefront takes two adjacent columns of the lower half of a q or k head and their partners of
//           the upper one (v: four adjacent columns), rotates them, writes q to y and k, v to their slots of the cache.  head_dim % 4 == 0.
struct F32Parts { const float* w[3]; int end[3]; int n; };
struct F32Fused {
    const float* gain = nullptr;               // NORM
    float eps = 0.f;
    const int2* row_at = nullptr;              // ROPE
    KvView kv;
    int layer_pool = 0, Hq = 0, Hkv = 0, dh = 0;
    float theta = 0.f;
};
constexpr int F32_ACCUM = 1, F32_NORM = 2, F32_SWIGLU = 4, F32_ROPE = 8;

// the rotation of one pair: cos and sin of pos * theta^(-2 j / dh)
__device__ inline float2 f32_rope_angle(int pos, int j, int dh, float theta)
{
    const float inv_freq = powf(theta, -2.0f * (float)j / (float)dh), ang = (float)pos * inv_freq;
    return make_float2(cosf(ang), sinf(ang));
}

template <int FORM>
__global__ __launch_bounds__(256) void f32_gemm_rows_kernel(const float* __restrict__ a, F32Parts parts, int M, int N, int K,
                                                            float* __restrict__ y, int ldy, F32Fused f)
{
    constexpr bool ACCUM = FORM & F32_ACCUM, NORM = FORM & F32_NORM, SWIGLU = FORM & F32_SWIGLU, ROPE = FORM & F32_ROPE;
    const int lane = threadIdx.x & 63, n0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * 4, m0 = blockIdx.y * 8;
    if (n0 >= N) return;
    // column of the output (ROPE: of the projection) that the wavefront's sum j belongs to
    const int half = f.dh >> 1, in_head = ROPE ? n0 % f.dh : 0;
    const bool rotated = ROPE && n0 < (f.Hq + f.Hkv) * f.dh;
    auto column = [&](int j) {
        if (SWIGLU) return n0 / 2 + (j & 1);
        if (rotated) return n0 - in_head + in_head / 2 + (j & 1) + (j >> 1) * half;
        return n0 + j;
    };
    const float *wr[4], *ar[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (SWIGLU) {
            const int n = column(j) < N / 2 ? column(j) : N / 2 - 1;
            wr[j] = parts.w[j >> 1] + (int64_t)n * K;
        } else {
            const int n = column(j) < N ? column(j) : N - 1;
            const int p = n < parts.end[0] ? 0 : (n < parts.end[1] ? 1 : 2);
            wr[j] = parts.w[p] + (int64_t)(n - (p > 0 ? parts.end[p - 1] : 0)) * K;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) ar[i] = a + (int64_t)(m0 + i < M ? m0 + i : M - 1) * K;
    float acc[32], ss[8];
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) ss[i] = 0.f;
    const int m = m0 + (lane >> 3), jl = (lane >> 1) & 3;
    int2 at = make_int2(0, -1);
    if constexpr (ROPE) at = f.row_at[m < M ? m : M - 1];
    for (int k = lane * 4; k < K; k += 256) {
        float4 wv[4], av[8], gv;
#pragma unroll
        for (int j = 0; j < 4; ++j) wv[j] = *(const float4*)(wr[j] + k);
        if constexpr (NORM) gv = *(const float4*)(f.gain + k);
#pragma unroll
        for (int i = 0; i < 8; ++i) av[i] = *(const float4*)(ar[i] + k);
        __builtin_amdgcn_sched_barrier(0);                 // all the loads before the first use of one
        if constexpr (NORM) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { wv[j].x *= gv.x; wv[j].y *= gv.y; wv[j].z *= gv.z; wv[j].w *= gv.w; }
#pragma unroll
            for (int i = 0; i < 8; ++i) { ss[i] += av[i].x * av[i].x; ss[i] += av[i].y * av[i].y; ss[i] += av[i].z * av[i].z; ss[i] += av[i].w * av[i].w; }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float& r = acc[i * 4 + j];
                r += av[i].x * wv[j].x; r += av[i].y * wv[j].y; r += av[i].z * wv[j].z; r += av[i].w * wv[j].w;
            }
    }
    // a lane keeps the half of its sums that its bit selects and hands the other half over: sum lane / 2 ends up in lanes
    // 2 r and 2 r + 1
    // (a compile-time size for every step: the array has to stay in registers)
    auto fold = [&](auto& v, auto half_c, auto off_c) {
        constexpr int HALF = decltype(half_c)::value, OFF = decltype(off_c)::value;
        const bool up = lane & OFF;
#pragma unroll
        for (int r = 0; r < HALF; ++r) {
            const float give = up ? v[r] : v[r + HALF], keep = up ? v[r + HALF] : v[r];
            v[r] = keep + __shfl_xor(give, OFF);
        }
    };
    fold(acc, std::integral_constant<int, 16>{}, std::integral_constant<int, 32>{});
    fold(acc, std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
    fold(acc, std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
    fold(acc, std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    fold(acc, std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
    float v = acc[0] + __shfl_xor(acc[0], 1);
    if constexpr (NORM) {
        fold(ss, std::integral_constant<int, 4>{}, std::integral_constant<int, 32>{});
        fold(ss, std::integral_constant<int, 2>{}, std::integral_constant<int, 16>{});
        fold(ss, std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
        float tot = ss[0];
        for (int off = 4; off > 0; off >>= 1) tot += __shfl_xor(tot, off);
        v *= 1.0f / sqrtf(tot / (float)K + f.eps);
    }
    const int n = column(jl);
    if constexpr (SWIGLU) {
        const float u = __shfl_xor(v, 4);                  // the up column's sum sits with the lane whose bit 2 is set
        if ((lane & 5) == 0 && m < M && n < N / 2) y[(int64_t)m * ldy + n] = v / (1.0f + expf(-v)) * u;
        return;
    }
    if constexpr (ROPE) {
        const int slot = at.y, head = n / f.dh, c = n - head * f.dh;
        if (rotated) {
            const float o = __shfl_xor(v, 4);              // the partner half's sum
            const float2 cs = f32_rope_angle(at.x, in_head / 2 + (jl & 1), f.dh, f.theta);
            v = jl < 2 ? v * cs.x - o * cs.y : v * cs.x + o * cs.y;
        }
        if ((lane & 1) || m >= M) return;
        if (head < f.Hq) { y[(int64_t)m * ldy + n] = v; return; }
        if (slot < 0) return;
        const int kind = head < f.Hq + f.Hkv ? 0 : 1, kh = head - f.Hq - kind * f.Hkv;
        const int64_t block = (int64_t)SPEC_PAGE_SIZE * f.dh, page = slot / SPEC_PAGE_SIZE;
        ((float*)f.kv.pool)[((((int64_t)f.layer_pool * f.kv.n_pages + page) * 2 + kind) * f.Hkv + kh) * block + (int64_t)(slot % SPEC_PAGE_SIZE) * f.dh + c] = v;
        return;
    }
    if ((lane & 1) == 0 && m < M && n < N) {
        float* dst = y + (int64_t)m * ldy + n;
        *dst = ACCUM ? *dst + v : v;
    }
}

// rotary embedding of q (in place) and k, and the speculative write of k, v into the paged cache.
// one workgroup per input row; qkv row = [q heads | k heads | v heads]
__global__ void f32_rope_kv_write_kernel(float* __restrict__ qkv, const int2* __restrict__ row_at,
                                         KvView kv, int layer_pool, int Hq, int Hkv, int dh, float theta)
{
    int m = blockIdx.x;
    const int pos = row_at[m].x, slot = row_at[m].y;
    int half = dh >> 1;
    float* row = qkv + (int64_t)m * (Hq + 2 * Hkv) * dh;
    const bool writable = slot >= 0;
    const int64_t page = slot / SPEC_PAGE_SIZE;
    const int t = slot % SPEC_PAGE_SIZE;
    float* pool = (float*)kv.pool;
    int64_t block = (int64_t)SPEC_PAGE_SIZE * dh;
    for (int e = threadIdx.x; e < (Hq + Hkv) * half; e += blockDim.x) {
        int h = e / half, j = e % half;
        const float2 cs = f32_rope_angle(pos, j, dh, theta);
        float* v = row + (int64_t)h * dh;
        float lo = v[j], hi = v[j + half];
        float rlo = lo * cs.x - hi * cs.y, rhi = hi * cs.x + lo * cs.y;
        if (h < Hq) { v[j] = rlo; v[j + half] = rhi; }
        else if (writable) {
            int kh = h - Hq;
            float* dst = pool + ((((int64_t)layer_pool * kv.n_pages + page) * 2 + 0) * Hkv + kh) * block;
            dst[(int64_t)t * dh + j] = rlo;
            dst[(int64_t)t * dh + j + half] = rhi;
        }
    }
    if (writable)
        for (int e = threadIdx.x; e < Hkv * dh; e += blockDim.x) {
            int kh = e / dh, c = e % dh;
            float* dst = pool + ((((int64_t)layer_pool * kv.n_pages + page) * 2 + 1) * Hkv + kh) * block;
            dst[(int64_t)t * dh + c] = row[(int64_t)(Hq + Hkv + kh) * dh + c];
        }
}

// one wavefront per (input row, query head): online softmax over the visible cache positions
__global__ __launch_bounds__(64) void f32_attention_kernel(const float* __restrict__ qkv, int T,
                                                           const int32_t* __restrict__ seq_ids, KvView kv,
                                                           int layer_pool, int Hq, int Hkv, int dh, float scale,
                                                           float* __restrict__ out)
{
    int m = blockIdx.x, j = blockIdx.y;
    int b = m / T, i = m % T;
    int seq = kv.entry_seq[b];
    int visible = seq >= 0 ? kv.ctx_len[seq] + i + 1 : 0;
    int cap = seq >= 0 ? kv.n_held[seq] * SPEC_PAGE_SIZE : 0;
    if (visible > cap) visible = cap;
    int g = j / (Hq / Hkv);
    const float* q = qkv + (int64_t)m * (Hq + 2 * Hkv) * dh + (int64_t)j * dh;
    const float* pool = (const float*)kv.pool;
    int64_t block = (int64_t)SPEC_PAGE_SIZE * dh;
    int lane = threadIdx.x;
    __shared__ float sq[256];
    __shared__ float sp[64];
    for (int c = lane; c < dh; c += 64) sq[c] = q[c];
    __syncthreads();
    float mx = -INFINITY, sum = 0.f;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};                  // channels lane, lane+64, ... (dh <= 256)
    for (int p0 = 0; p0 < visible; p0 += 64) {
        int pos = p0 + lane;
        float s = -INFINITY;
        int my_page = 0;                                  // page of this lane's position
        if (pos < visible) {
            my_page = kv.page_table[(int64_t)seq * kv.max_pages + pos / SPEC_PAGE_SIZE];
            const int64_t page = my_page;
            const float* kr = pool + ((((int64_t)layer_pool * kv.n_pages + page) * 2 + 0) * Hkv + g) * block +
                              (int64_t)(pos % SPEC_PAGE_SIZE) * dh;
            float d = 0.f;
#pragma unroll 16
            for (int c = 0; c < dh; ++c) d += kr[c] * sq[c];
            s = d * scale;
        }
        float cm = s;
        for (int off = 32; off > 0; off >>= 1) cm = fmaxf(cm, __shfl_xor(cm, off));
        float nm = fmaxf(mx, cm);
        float corr = expf(mx - nm);
        float p = (pos < visible) ? expf(s - nm) : 0.f;
        float ps = p;
        for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off);
        sum = sum * corr + ps;
        mx = nm;
        __syncthreads();
        sp[lane] = p;
        __syncthreads();
        int cnt = visible - p0 < 64 ? visible - p0 : 64;
        for (int a = 0; a < 4; ++a) {
            if (64 * a < dh) {
                // every lane stays on, as the page ids are handed round between them: those beyond the last channel repeat it (not stored)
                const int c = lane + 64 * a < dh ? lane + 64 * a : dh - 1;
                float o = acc[a] * corr;
                // a page of positions at a time (p0 is a multiple of the page size), its loads in flight together: the
                // slots past the last visible position re-read that one and are left out of the sum
                for (int t0 = 0; t0 < cnt; t0 += SPEC_PAGE_SIZE) {
                    const int64_t page = __builtin_amdgcn_readlane(my_page, t0);
                    const int n_t = cnt - t0 < SPEC_PAGE_SIZE ? cnt - t0 : SPEC_PAGE_SIZE;
                    const float* vb = pool + ((((int64_t)layer_pool * kv.n_pages + page) * 2 + 1) * Hkv + g) * block + c;
                    float v[SPEC_PAGE_SIZE];
#pragma unroll
                    for (int t = 0; t < SPEC_PAGE_SIZE; ++t) v[t] = vb[(int64_t)(t < n_t ? t : n_t - 1) * dh];
#pragma unroll
                    for (int t = 0; t < SPEC_PAGE_SIZE; ++t)
                        if (t < n_t) o += sp[t0 + t] * v[t];
                }
                acc[a] = o;
            }
        }
    }
    for (int a = 0; a < 4; ++a) {
        int c = lane + 64 * a;
        if (c < dh) out[(int64_t)m * Hq * dh + (int64_t)j * dh + c] = sum > 0.f ? acc[a] / sum : 0.f;
    }
}

// The same for head_dim % 4 == 0: four wavefronts per (input row, query head), each every fourth piece of 64 positions.  A piece is two trips to memory:
// keys with a lane per position (16 bytes at a time), values with a lane per four channels and 64 / (head_dim / 4) positions side by
// side, asked for before the softmax.  The wavefronts' results are merged through LDS.  Bound by those trips and the merge: 128 positions of 4 heads x 64
// channels, 16 rows: 17.1 us as one wavefront with a piece after the other and a trip per page of values, 8.8 us now.
constexpr int F32_ATT_WAVES = 4, F32_VQ = 16;             // values (float4) in flight per lane

__global__ __launch_bounds__(256) void f32_attention_split_kernel(const float* __restrict__ q_rows, int ldq, int T, KvView kv, int layer_pool,
                                                                  int Hq, int Hkv, int dh, float scale, float* __restrict__ out)
{
    const int m = blockIdx.x, head = blockIdx.y, b = m / T, g = head / (Hq / Hkv);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int seq = kv.entry_seq[b];
    int visible = seq >= 0 ? kv.ctx_len[seq] + m % T + 1 : 0;
    const int cap = seq >= 0 ? kv.n_held[seq] * SPEC_PAGE_SIZE : 0;
    if (visible > cap) visible = cap;
    const int64_t block = (int64_t)SPEC_PAGE_SIZE * dh;
    const float* pool = (const float*)kv.pool + (int64_t)layer_pool * kv.n_pages * 2 * Hkv * block;
    __shared__ float4 s_q[64];
    __shared__ float s_p[F32_ATT_WAVES][64], s_m[F32_ATT_WAVES], s_l[F32_ATT_WAVES];
    __shared__ int s_page[F32_ATT_WAVES][64 / SPEC_PAGE_SIZE];
    __shared__ float4 s_o[F32_ATT_WAVES][64];
    const int quads = dh >> 2, groups = 64 / quads;       // dh <= 256
    if ((int)threadIdx.x < quads) s_q[threadIdx.x] = *(const float4*)(q_rows + (int64_t)m * ldq + (int64_t)head * dh + threadIdx.x * 4);
    __syncthreads();
    const int vg = lane / quads, vc = (lane - vg * quads) * 4;
    const bool v_lane = vg < groups;
    float mx = -INFINITY, sum = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int p0 = wave * 64; p0 < visible; p0 += 64 * F32_ATT_WAVES) {
        const int cnt = visible - p0 < 64 ? visible - p0 : 64, pos = p0 + (lane < cnt ? lane : cnt - 1);
        const int page = kv.page_table[(int64_t)seq * kv.max_pages + pos / SPEC_PAGE_SIZE];
        if (lane % SPEC_PAGE_SIZE == 0) s_page[wave][lane / SPEC_PAGE_SIZE] = page;      // (written and read by this wavefront only)
        __builtin_amdgcn_wave_barrier();
        // positions vg, vg + groups, ... of the piece; those past the end read the last one and weigh nothing
        auto value = [&](int t) {
            const int tc = t < cnt ? t : cnt - 1;
            return *(const float4*)(pool + ((int64_t)s_page[wave][tc / SPEC_PAGE_SIZE] * 2 * Hkv + Hkv + g) * block + (int64_t)(tc % SPEC_PAGE_SIZE) * dh + (v_lane ? vc : 0));
        };
        const float* kr = pool + ((int64_t)page * 2 * Hkv + g) * block + (int64_t)(pos % SPEC_PAGE_SIZE) * dh;
        float d = 0.f;
        for (int c0 = 0; c0 < quads; c0 += 16) {
            float4 kq[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) kq[c] = *(const float4*)(kr + 4 * (c0 + c < quads ? c0 + c : 0));
#pragma unroll
            for (int c = 0; c < 16; ++c)
                if (c0 + c < quads) {
                    const float4 qq = s_q[c0 + c];
                    d += kq[c].x * qq.x; d += kq[c].y * qq.y; d += kq[c].z * qq.z; d += kq[c].w * qq.w;
                }
        }
        float4 vv[F32_VQ];
#pragma unroll
        for (int u = 0; u < F32_VQ; ++u) vv[u] = value(vg + u * groups);
        const float sc = lane < cnt ? d * scale : -INFINITY;
        float cm = sc;
        for (int off = 32; off > 0; off >>= 1) cm = fmaxf(cm, __shfl_xor(cm, off));
        const float nm = fmaxf(mx, cm), corr = expf(mx - nm);
        const float p = lane < cnt ? expf(sc - nm) : 0.f;
        float ps = p;
        for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off);
        sum = sum * corr + ps;
        mx = nm;
        s_p[wave][lane] = p;
        __builtin_amdgcn_wave_barrier();
        acc.x *= corr; acc.y *= corr; acc.z *= corr; acc.w *= corr;
        for (int t0 = vg; t0 < 64; t0 += F32_VQ * groups) {
            if (t0 > vg) {
#pragma unroll
                for (int u = 0; u < F32_VQ; ++u) vv[u] = value(t0 + u * groups);
            }
#pragma unroll
            for (int u = 0; u < F32_VQ; ++u) {
                const int t = t0 + u * groups;
                const float w = t < cnt ? s_p[wave][t] : 0.f;
                const float4 x = t < cnt ? vv[u] : make_float4(0.f, 0.f, 0.f, 0.f);      // (whatever the last position holds)
                acc.x += w * x.x; acc.y += w * x.y; acc.z += w * x.z; acc.w += w * x.w;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    s_o[wave][lane] = acc;
    if (lane == 0) { s_m[wave] = mx; s_l[wave] = sum; }
    __syncthreads();
    if ((int)threadIdx.x < dh) {
        float M = -INFINITY, L = 0.f, o = 0.f;
        const int waves = visible > 64 * (F32_ATT_WAVES - 1) ? F32_ATT_WAVES : (visible + 63) >> 6;      // those with positions of their own
        for (int w = 0; w < waves; ++w) M = fmaxf(M, s_m[w]);
        for (int w = 0; w < waves; ++w) {
            const float f = s_m[w] > -INFINITY ? expf(s_m[w] - M) : 0.f;      // (0 where all scores are NaN: the NaN sums come through)
            L += f * s_l[w];
            for (int i = 0; i < groups; ++i) o += f * ((const float*)&s_o[w][i * quads])[threadIdx.x];
        }
        out[(int64_t)m * Hq * dh + (int64_t)head * dh + threadIdx.x] = L > 0.f ? o / L : 0.f;
    }
}

__global__ void f32_swiglu_kernel(const float* __restrict__ gu, int M, int F, float* __restrict__ act)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)M * F) return;
    int m = idx / F, f = idx % F;
    float g = gu[(int64_t)m * 2 * F + f], u = gu[(int64_t)m * 2 * F + F + f];
    act[idx] = g / (1.0f + expf(-g)) * u;
}

// ------------------------------------------------------------------ host side
struct F32Ws { float *x, *h, *qkv, *attn, *gu, *act; int2* row_at; };

static size_t f32_carve(const spec_model_desc& d, int M, char* base, F32Ws* w)
{
    size_t off = 0;
    auto take = [&](size_t elems) { size_t o = off; off = align_up(off + elems * sizeof(float), 256); return base ? (float*)(base + o) : nullptr; };
    int nqkv = (d.n_q_heads + 2 * d.n_kv_heads) * d.head_dim;
    F32Ws t;
    t.x = take((size_t)M * d.d_model);
    t.h = take((size_t)M * d.d_model);
    t.qkv = take((size_t)M * nqkv);
    t.attn = take((size_t)M * d.n_q_heads * d.head_dim);
    t.gu = take((size_t)M * 2 * d.ffn_dim);
    t.act = take((size_t)M * d.ffn_dim);
    t.row_at = (int2*)take((size_t)M * 2);
    if (w) *w = t;
    return off;
}

size_t f32_workspace_bytes(const spec_model_desc& d, int B, int k) { return f32_carve(d, B * (k + 1), nullptr, nullptr); }

// f32_gemm_rows_kernel takes a trip to memory per 256 of K, but fetches a matrix again for every 8 rows; the tiled kernel takes a trip per
// 32 of K (3.6 us each), and its tile is 32 rows.  Tiled / rows, us:
//   matrices that stay in the 256 MB memory-side cache: N = 1024, K = 256: 15.2 / 3.8 at 16 rows, 18.4 / 12.1 at 512; N = 1024, K = 704:
//   38.8 / 5.1 and 45.7 / 20.9; N = 4096, K = 256: 15.2 / 4.2 and 41.1 / 37.6; N = K = 4096: 319 / 20 and 669 / 547; two of 16384 x 2048 (256
//   MB): 716 / 626 at 128 rows, 2509 / 2353 at 512.  The lead shrinks with the rows, and beyond 512 nothing was measured;
//   beyond the cache every 8 rows fetch the matrices from HBM: up to 24 rows that is still the faster (98304 x 1024: 286 / 174 at 16 rows,
//   335 / 349 at 32, 1129 / 1384 at 128; 131072 x 4096: 1389 / 869, 1532 / 1725, 5707 / 6804).  With more, it is so while the tiled kernel has too few
//   tiles to hide its trips, that is up to some number of outputs per matrix: N = 4096, K = 28672: 3286 / 2970 at 256 rows, 3938 / 4494
//   at 384; N = 8192, K = 16384: 1912 / 1653 at 128, 2361 / 2484 at 192; two of 11008 x 4096: 1026 / 860 at 96, 1949 / 2253 at 256; two of 28672 x
//   4096: 1216 / 770 at 32, 1381 / 1526 at 64.  (70000 x 1024, 273 MB, is even from 64 rows on.)
static bool rows_kernel_is_ahead(int M, int N, int K, int n_matrices)
{
    if (M > 512) return false;
    if ((int64_t)N * K * 4 <= (int64_t)288 << 20) return true;
    return M <= 24 || (int64_t)M * N <= (int64_t)n_matrices * 1300000;
}

// Whether the norm and what follows a projection are better done in its kernel, which repeats them for every few columns (a third more vector work),
// than by launches of their own.  Forward pass of two layers, separate / fused, us: 16 rows of d = 256, 512, 1024, 2048: 83 / 65, 126 / 104, 203 / 174,
// 333 / 302; 64 rows: 90 / 72, 156 / 141, 332 / 312, 764 / 743; 256 rows: 130 / 120, 405 / 412, 1071 / 1111, 2825 / 2854 (d = 256: products of up to 92 M
// multiplications, d = 512: up to 369 M).
static bool rows_kernel_fuses(int M, int N, int K) { return M <= 64 || (int64_t)M * N * K <= 128 << 20; }

// y = a w^T for up to three matrices over the same rows, side by side in y.  FORM other than 0 and ACCUM: what f32_gemm_rows_kernel does around
// it; false and nothing launched where that kernel is not the one to take, or where its larger inner loop would cost more than the launches it saves.
template <int FORM = 0>
static bool gemm(const float* a, std::initializer_list<std::pair<const float*, int>> ws, int M, int K, float* y, int ldy, hipStream_t s,
                 const F32Fused& f = F32Fused())
{
    constexpr bool FUSED = FORM & ~F32_ACCUM;
    F32Parts parts{};
    int N = 0;
    bool aligned = K % 4 == 0 && ((uintptr_t)a & 15) == 0 && ((uintptr_t)f.gain & 15) == 0;
    for (auto& w : ws) {
        N += w.second;
        parts.w[parts.n] = w.first;
        parts.end[parts.n++] = N;
        aligned = aligned && ((uintptr_t)w.first & 15) == 0;
    }
    for (int i = parts.n; i < 3; ++i) { parts.w[i] = parts.w[parts.n - 1]; parts.end[i] = N; }
    const bool rows = aligned && rows_kernel_is_ahead(M, N, K, parts.n);
    if (FUSED && (!rows || !rows_kernel_fuses(M, N, K))) return false;
    if (rows) {
        dim3 grid((unsigned)cdiv(N, 16), (unsigned)cdiv(M, 8));
        f32_gemm_rows_kernel<FORM><<<grid, 256, 0, s>>>(a, parts, M, N, K, y, ldy, f);
        return true;
    }
    for (auto& w : ws) {
        dim3 grid((unsigned)cdiv(w.second, 32), (unsigned)cdiv(M, 32));
        f32_gemm_kernel<(FORM & F32_ACCUM) != 0><<<grid, 256, 0, s>>>(a, w.first, M, w.second, K, y, ldy);
        y += w.second;
    }
    return true;
}

spec_status f32_forward(spec_model* mdl, spec_kv* kv, int B, int k, const int32_t* dev_seq_ids,
                        const int32_t* dev_tokens, float* dev_logits, void* ws, hipStream_t s)
{
    const spec_model_desc& d = mdl->desc;
    if (d.head_dim > 256 || (d.head_dim & 1)) { set_error("fp32 path needs an even head_dim <= 256"); return SPEC_EUNSUPPORTED; }
    int T = k + 1, M = B * T;
    int Hq = d.n_q_heads, Hkv = d.n_kv_heads, dh = d.head_dim, D = d.d_model, F = d.ffn_dim;
    int nq = Hq * dh, nkv = Hkv * dh, nqkv = nq + 2 * nkv;
    F32Ws w;
    f32_carve(d, M, (char*)ws, &w);
    KvView view = kv->view();
    float scale = 1.0f / sqrtf((float)dh);

    f32_embed_kernel<<<M, 256, 0, s>>>(dev_tokens, (const float*)mdl->embed(), D, d.vocab, T, view, w.x, w.row_at);
    const bool quads = dh % 4 == 0;
    // Four wavefronts per row and head while one each would not give every SIMD of the chip one.  Forward pass of two layers at contexts of 128, 700 and
    // 3000, one / four, us: 128 rows x 8 heads 173 / 171, 291 / 254, 925 / 592; 192 x 8 213 / 220, 375 / 355, 1016 / 844; 256 x 8 242 / 261, 428 / 437,
    // 1128 / 1085; 256 x 16 at 128 and 700 527 / 566, 870 / 896.  (The contexts are not known here.)
    const bool split_attention = quads && ((uintptr_t)view.pool & 15) == 0 && (int64_t)M * Hq <= 1024;
    F32Fused f;
    f.eps = d.rms_eps;
    f.row_at = w.row_at;
    f.kv = view;
    f.Hq = Hq; f.Hkv = Hkv; f.dh = dh; f.theta = d.rope_theta;
    for (int l = 0; l < d.n_layers; ++l) {
        int lp = kv->alias_mod > 0 ? l % kv->alias_mod : l;
        auto W = [&](int i) { return (const float*)mdl->layer_w(l, i); };
        f.layer_pool = lp;
        f.gain = W(0);
        if (!quads || !gemm<F32_NORM | F32_ROPE>(w.x, {{W(1), nq}, {W(2), nkv}, {W(3), nkv}}, M, D, w.qkv, nqkv, s, f)) {
            f32_rmsnorm_kernel<<<M, 256, 0, s>>>(w.x, W(0), D, d.rms_eps, w.h);
            gemm(w.h, {{W(1), nq}, {W(2), nkv}, {W(3), nkv}}, M, D, w.qkv, nqkv, s);
            f32_rope_kv_write_kernel<<<M, 256, 0, s>>>(w.qkv, w.row_at, view, lp, Hq, Hkv, dh, d.rope_theta);
        }
        if (split_attention) f32_attention_split_kernel<<<dim3(M, Hq), 256, 0, s>>>(w.qkv, nqkv, T, view, lp, Hq, Hkv, dh, scale, w.attn);
        else f32_attention_kernel<<<dim3(M, Hq), 64, 0, s>>>(w.qkv, T, dev_seq_ids, view, lp, Hq, Hkv, dh, scale, w.attn);
        gemm<F32_ACCUM>(w.attn, {{W(4), D}}, M, nq, w.x, D, s);
        f.gain = W(5);
        if (!gemm<F32_NORM | F32_SWIGLU>(w.x, {{W(6), F}, {W(7), F}}, M, D, w.act, F, s, f)) {
            f32_rmsnorm_kernel<<<M, 256, 0, s>>>(w.x, W(5), D, d.rms_eps, w.h);
            gemm(w.h, {{W(6), F}, {W(7), F}}, M, D, w.gu, 2 * F, s);
            f32_swiglu_kernel<<<(unsigned)cdiv((int64_t)M * F, 256), 256, 0, s>>>(w.gu, M, F, w.act);
        }
        gemm<F32_ACCUM>(w.act, {{W(8), D}}, M, F, w.x, D, s);
    }
    f.gain = (const float*)mdl->final_norm();
    if (!gemm<F32_NORM>(w.x, {{(const float*)mdl->head_w(), head_rows(d)}}, M, D, dev_logits, head_rows(d), s, f)) {
        f32_rmsnorm_kernel<<<M, 256, 0, s>>>(w.x, (const float*)mdl->final_norm(), D, d.rms_eps, w.h);
        gemm(w.h, {{(const float*)mdl->head_w(), head_rows(d)}}, M, D, dev_logits, head_rows(d), s);
    }
    SPEC_LAUNCH_CHECK("fp32 forward");
    return SPEC_OK;
}

}  // namespace specv
