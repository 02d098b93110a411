// k_attn_f32.hip -- chunk attention over the compressed cache (Eq. 2 / Eq. 4)
// for fp32 tensors, on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32
// products and sums, 64 cycles each).
//
// Workgroup = 8 waves = 32 query rows of one head; the waves take the 32-key
// tiles in turn (tile t goes to wave t mod 8) and their partial results are
// combined in LDS at the end.  Splitting the keys inside the workgroup gives
// short chunks enough waves: a quarter-480P layer (F = 390, 3 frames) has only
// 37 row blocks per head.
//
// Per wave and tile:
//   S^T = K . Q^T   (A = key rows, B = the wave's query rows, in VGPRs; 2 x
//                   d/4 products in all, the contraction index permuted so that
//                   a lane's operands of four products are 16 adjacent bytes);
//   online softmax in fp32, one query column per lane (lanes l and l^32 share
//                   a query and hold different keys);
//   O^T += V^T . P^T (B = P straight from the S^T accumulators: entry i of lane
//                   half hl is key 8(i/4) + 4hl + i%4, so product i contracts
//                   exactly these two keys; A = the matching V rows, output row
//                   block mb of lane l32 being dim (d/32) l32 + mb so that the
//                   lane's operands of all blocks are adjacent).
//
// What bounds it: the matrix cores.  A tile is d products of 64 cycles per
// wave, and both operands come straight from global memory (16-byte loads into
// one of two register buffers, half a tile ahead of their use -- 2048 cycles at
// d = 128, longer than any memory latency), so there is no LDS staging and no
// barrier in the loop.  12 heads, F = 390, 21-frame window, d = 128 (33.6
// GFLOP): 395 us, 85 TFLOP/s of the 154 a large fp32 matrix product reaches,
// against 3.3 ms for the vector-arithmetic kernel this replaced; MFMA busy 70%
// of the cycles a CU is occupied, and the 444 workgroups fill 256 CUs 1.7
// times.  64 or 128 query rows per workgroup (4 or 2 waves sharing the keys)
// measured 441 and 791 us; items dealt XCD by XCD instead of round robin 438.
#include "fkv_internal.h"

namespace fkv {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int TN = 32;  // keys per tile

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000u);
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, uint32_t off, u32x4 &x) {
    x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, uint32_t off, u32x2_t &x) {
    x = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

// The vector of one V row's operands (d / 32 adjacent dims).
template <int D>
struct VecOf;
template <>
struct VecOf<128> {
    typedef f32x4_t f;
    typedef u32x4 u;
};
template <>
struct VecOf<64> {
    typedef f32x2_t f;
    typedef u32x2_t u;
};

template <int D>
__global__ __launch_bounds__(kThreads, 2) void attn_f32_kernel(AttnArgs a) {
    constexpr int MB = D / 32;           // 32-row blocks of O^T
    constexpr int KV = D / 8;            // 16-byte vectors of a lane's K operand per tile
    constexpr int KH = KV / 2;           // per half
    typedef typename VecOf<D>::f vvec;
    typedef typename VecOf<D>::u uvec;
    // partial results: O^T in the accumulator layout, row maxima, row sums
    __shared__ float Os[kWaves][16 * MB][64];
    __shared__ float Ms[kWaves][32], Ls[kWaves][32];

    const int item = blockIdx.x;
    const int li = item / a.n_qtiles;
    const int h = a.heads.head[li];
    const int qt = item - li * a.n_qtiles;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, hl = lane >> 5;
    const int Lq = a.Lq;
    const int row = qt * kAttnRowsF32 + l32;
    const bool rok = row < Lq;

    const float *Qr = (const float *)a.Q + ((size_t)h * Lq + (rok ? row : 0)) * D + 4 * hl;
    f32x4_t qf[KV];
#pragma unroll
    for (int t = 0; t < KV; ++t) qf[t] = rok ? *(const f32x4_t *)(Qr + 8 * t) : f32x4_t{};

    int kvl = a.kv_len[h];
    kvl = __builtin_amdgcn_readfirstlane(kvl < 0 ? 0 : (kvl > a.slab ? (int)a.slab : kvl));
    const int Lk = kvl + Lq;
    const int T = (Lk + TN - 1) / TN;
    const float *Kc = (const float *)a.Kc + (size_t)h * a.slab * D;
    const float *Vc = (const float *)a.Vc + (size_t)h * a.slab * D;
    const float *Kq = (const float *)a.K_cur + (size_t)h * Lq * D;
    const float *Vq = (const float *)a.V_cur + (size_t)h * Lq * D;

    // This lane's operands of the tile at j0 through range-checked buffers
    // (32-bit offsets; the host keeps a head's cache and chunk below 2^31
    // bytes).  A tile inside one source needs one buffer; in the tile that
    // straddles history and chunk each row comes from the one buffer that holds
    // it, the other reads zero.  Rows past the last key read zero.
    const uint32_t koff = (uint32_t)(l32 * D + 4 * hl) * 4u;
    const uint32_t voff = (uint32_t)(4 * hl * D + MB * l32) * 4u;
    // 4 * NG vectors at byte offsets off + g * gstep + e * step of the tile (the
    // group's base is opaque, or the compiler keeps every offset in a register)
    auto tile_load = [&](const float *hist, const float *chunk, int j0, auto &x, uint32_t off, uint32_t gstep,
                         uint32_t step) {
        constexpr int NG = sizeof(x) / sizeof(x[0]) / 4;
        if (j0 + TN <= kvl || j0 >= kvl) {
            const bool in_hist = j0 < kvl;
            const auto r = rsrc(in_hist ? hist + (size_t)j0 * D : chunk + (size_t)(j0 - kvl) * D,
                                (uint32_t)(in_hist ? TN : min(TN, Lk - j0)) * D * 4);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                uint32_t b = off + g * gstep;
                __asm__ volatile("" : "+v"(b));
#pragma unroll
                for (int e = 0; e < 4; ++e) bload(r, b + e * step, x[4 * g + e]);
            }
        } else {
            const uint32_t nh = (uint32_t)(kvl - j0) * D * 4;
            const auto rh = rsrc(hist + (size_t)j0 * D, nh);
            const auto rc = rsrc(chunk, (uint32_t)min(TN - (kvl - j0), Lq) * D * 4);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    auto y = x[4 * g + e];
                    uint32_t b = off + g * gstep + e * step, c = b - nh;   // a history row's c wraps: out of range
                    __asm__ volatile("" : "+v"(b), "+v"(c));
                    bload(rh, b, x[4 * g + e]);
                    bload(rc, c, y);
                    x[4 * g + e] |= y;
                }
            }
        }
    };
    auto load_k = [&](int j0, int half, u32x4 (&x)[KH]) {
        tile_load(Kc, Kq, j0, x, koff + 32u * (half * KH), 128, 32);
    };
    // V rows of products 8*half .. 8*half + 7
    auto load_v = [&](int j0, int half, uvec (&x)[8]) {
        tile_load(Vc, Vq, j0, x, voff + half * (16 * D * 4), 8 * D * 4, D * 4);
    };
    auto f = [](uint32_t w) { return __uint_as_float(w); };

    f32x16_t o[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) o[mb] = f32x16_t{};
    float m_run = -__builtin_inff(), l_run = 0.f;

    u32x4 ka[KH], kb[KH];
    uvec va[8], vb[8];
    if (wave < T) load_k(wave * TN, 0, ka);
    for (int t = wave; t < T; t += kWaves) {
        const int j0 = t * TN;
        f32x16_t s = {};
        load_k(j0, 1, kb);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < KH; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(f(ka[u][e]), qf[u][e], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_v(j0, 0, va);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < KH; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(f(kb[u][e]), qf[KH + u][e], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_v(j0, 1, vb);
        __builtin_amdgcn_sched_barrier(0);

        s *= a.scale;
        if (j0 + TN > Lk) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (j0 + 8 * (i >> 2) + 4 * hl + (i & 3) >= Lk) s[i] = -__builtin_inff();
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        if (__ballot(m_new != m_run)) {
            const float alpha = m_new == m_run ? 1.f : expf(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) o[mb] *= alpha;
        }
        // a row whose scores are all -inf so far weighs nothing (-inf - -inf would be NaN)
        const float m_ref = m_run == -__builtin_inff() ? 0.f : m_run;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = expf(s[i] - m_ref);
            l_run += s[i];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) o[mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(f(va[i][mb]), s[i], o[mb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (t + kWaves < T) load_k(j0 + kWaves * TN, 0, ka);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                o[mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(f(vb[i][mb]), s[8 + i], o[mb], 0, 0, 0);
    }

    // Combine the waves' partial results: every wave leaves its accumulators,
    // maxima and sums in LDS, then combines an eighth of the accumulator
    // entries.  A part without keys has maximum -inf and weight 0.
    l_run += __shfl_xor(l_run, 32);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) Os[wave][16 * mb + i][lane] = o[mb][i];
    if (hl == 0) {
        Ms[wave][l32] = m_run;
        Ls[wave][l32] = l_run;
    }
    __syncthreads();
    float M = Ms[0][l32];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) M = fmaxf(M, Ms[k][l32]);
    float L = 0.f, wt[kWaves];
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const float m = Ms[k][l32];
        wt[k] = m == -__builtin_inff() ? 0.f : expf(m - M);
        L = fmaf(wt[k], Ls[k][l32], L);
    }
    if (!rok) return;
    const float inv = 1.f / L;
    float *Or = (float *)a.O + ((size_t)h * Lq + row) * D;
    // accumulator entry i of lane half hl is output row 8(i/4) + 4hl + i%4 of
    // every block; wave w combines entries 2w and 2w + 1
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int i = 2 * wave + e;
        vvec x = {};
#pragma unroll
        for (int k = 0; k < kWaves; ++k)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) x[mb] = fmaf(wt[k], Os[k][16 * mb + i][lane], x[mb]);
        *(vvec *)(Or + MB * (8 * (i >> 2) + 4 * hl + (i & 3))) = x * inv;
    }
    if (a.lse && hl == 0 && wave == 0) a.lse[(size_t)h * Lq + row] = M + logf(L);
}

}  // namespace

hipError_t launch_attention_f32(const AttnArgs &a, int head_dim, hipStream_t s) {
    if (head_dim == 128)
        hipLaunchKernelGGL(attn_f32_kernel<128>, dim3(a.n_items), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL(attn_f32_kernel<64>, dim3(a.n_items), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace fkv
