// k_attn.hip -- chunk attention over each head's compressed cache (Eq. 2 for
// static heads, Eq. 4 for dynamic heads), bf16 inputs, gfx950 MFMA.
//
// For head h the key sequence is [Kc[h][0:kv_len[h]]; K_cur[h]] (the retained
// history, then the current chunk) and likewise for values; every query row of
// the chunk attends to all of it with no mask.  The per-head key count is
// ragged (it comes from the device-side kv_len), and one key tile may straddle
// the history/chunk boundary.  The PAGED instantiation attends heads in place:
// their retained history -- the kept frames of Eq. 2 for static heads, the
// kept segments of Eq. 3 for dynamic heads -- is read straight from the
// slot-permuted cache through a per-head page table (paged_tile), with no
// compressed copy.
//
// Workgroup = 8 waves = 256 query rows of one head (32 per wave); one workgroup
// fills a CU.  Keys are processed in tiles of 64.  Per wave and tile, with v_mfma_f32_32x32x16_bf16:
//   S^T = K . Q^T   (A = K rows from LDS, B = the wave's Q rows, held in VGPRs),
//                   2 x (d/16) MFMAs;
//   softmax in fp32 (exp2 with the scale folded into log2 units; the
//                   row sum adds the bf16-rounded probabilities with v_dot2);
//   O^T += V^T . P^T (A = rows of a V^T tile in LDS, B = P taken straight from
//                    the S^T accumulators, rounded to bf16), 4 x (d/32) MFMAs.
// Computing S transposed makes each lane own one query column, so P needs no
// data movement between the two products: in the 32x32 accumulator layout a
// lane holds 16 keys of its query, which are exactly the 8-element k-slices the
// B operand of the value product takes (any consistent permutation of the
// contraction index is allowed; the V^T tile is stored with the same
// permutation).  Both operands are read from LDS with 16-byte reads; V is
// transposed on its way into LDS (measured faster than the LDS transpose
// reads).
//
// Per 64-key tile a wave issues 32 products (D = 128), 32 operand reads and the
// tile's 32 exponentials with their scaling, rounding and sums.  The loop
// (attn_segment) interleaves them in one pinned order: products of one tile's
// scores and the previous one's values alternate, a few VALU instructions behind
// each, so the exponentials of a key block run while 16 other products do, and
// nothing in a wave waits for a row maximum: the exponentials' reference is the
// row maximum of the segment's first tile.  Probabilities may then exceed one,
// in bf16 and fp32 by 2^100 and more without loss (their relative rounding is
// the same); a segment in which a sum passes 2^100 or an output is not finite is
// computed again with a running maximum (it moves where a tile's exceeds it by
// more than 8 in log2 units).  That costs the segment twice and more, and a NaN
// or an infinity in Q or V always brings it about: 480P step 509 us, 967 with one
// NaN in one static head's V, 1086 with one in every head's.
// Bound: at 1080P the clock, which the power of the products holds at 1.73-1.85
// GHz (a 8192^3 library product reaches 1.2 PFLOP/s on this card, a bare loop of
// these products, reads and exponentials 1.44), and 65% of the cycles issue a
// product (60% before, when the softmax of one wave group ran beside the
// products of the other: its row maximum, its scalar page arithmetic of some 70
// instructions per tile and its wait for the second part of a straddling tile
// were in the way).  Layer steps, both kernels in turn on one card and then on
// another: 1080P 13.28 -> 12.52 and 12.97 -> 12.39 ms, 480P 541 -> 519 and 528 ->
// 507 us, with quarter-frame segments, where every sixth tile straddles, 461 ->
// 430 and 449 -> 419 us.  A segment's fixed cost went the other way (a launch of one
// tile per item takes 9.7 us at d = 128, 7.9 before, 8.1 and 6.9 at d = 64), so
// those with segments of up to ten tiles take up to 9% longer.
// Measured beside it, 480P step: the wave groups half an iteration apart 544
// against 527 us; every tile's source found anew by scalar branches 527 against
// 508 us (a run of full tiles now costs a scalar add); all exponentials in the
// second half of an iteration 571 against 557 us of the kernel before.
//
// Global K/V rows come in through buffer loads whose per-lane offsets are loop
// invariant; rows past the end of a source fall outside the buffer's range and
// read as zero.
//
// Schedules: a work item is (entry of the launch's head list, query tile);
// one workgroup per item, or the balanced schedule (attn_common.h) that splits
// the key tiles of all items evenly, or every item in as many parts as there are
// workgroups to spare, over one workgroup per CU; the parts of a
// split item are merged by the workgroup that completes the last of them
// (merge_rows).  Heads with longer caches make the per-item
// schedule uneven (at 480P a dynamic head has 342 key tiles per query tile, a
// static head 245, on 228 items for 256 CUs).
#include "attn_common.h"
#include "attn_merge.h"
#include "handover.h"

namespace fkv {
namespace {

using namespace attn;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kThreads = 512;      // 8 waves
constexpr int kBufs = 4;           // K and V^T tiles in LDS
constexpr float kSumLimit = 0x1p100f; // a larger sum of probabilities redoes the segment with a running max
constexpr float kFarMove = 64.f;      // largest move by whole powers of two
constexpr float kLowest = 0x1.fffffep127f;  // largest finite value
constexpr float kRescaleSlack = 8.f;  // log2 units the running max of a redone segment may lag behind
constexpr uint32_t kRsrcWord3 = 0x00020000u;  // raw 32-bit buffer, range checked
constexpr bf16x2_t kOnes2 = {(__bf16)1.f, (__bf16)1.f};

template <int D>
struct Cfg {
    static constexpr int RSE = D + 8;           // K row stride in LDS (16-byte pad), elements
    static constexpr int TRSE = BN + 8;         // V^T row stride in LDS (16-byte pad), elements
    static constexpr int CPR = D / 8;           // 16-byte chunks per row
    static constexpr int RPP = kThreads / CPR;  // rows one pass of the workgroup covers
    static constexpr int NV = BN / RPP;         // 16-byte vectors per thread per staged K tile
    static constexpr int VW = D / 64;           // 4-byte words (2 dims) per thread and key of a staged V tile
    static constexpr int KS = D / 16;           // k-steps of S^T = K Q^T
    static constexpr int MB = D / 32;           // 32-row blocks of O^T
    static constexpr int TILE = BN * RSE;       // elements per K tile
    static constexpr int VTILE = D * TRSE;      // elements per V^T tile
    static_assert(NV >= 1 && BN % RPP == 0, "tile shape");
    static_assert((BN / 4) * (D / (2 * VW)) == kThreads, "one V unit (4 keys x 2 VW dims) per thread");
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, kRsrcWord3);
}

__device__ __forceinline__ u32x4 bload(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff = 0) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}

// Rows of the key tile starting at j0 of [hist (kvl rows); chunk (Lq rows)] into
// registers, zeros past Lk = kvl + Lq: N 16-byte vectors at byte offsets
// off0 + i*step within the tile.  Rows past the end of a source fall outside
// its buffer range and read as zero; the tile straddling the history/chunk
// boundary merges both sources that way.
template <int D, int N>
__device__ __forceinline__ void load_tile(const uint16_t *hist, const uint16_t *chunk, int j0, int kvl,
                                          int Lk, int Lq, u32x4 *dst, uint32_t off0, uint32_t step) {
    if (j0 + BN <= kvl) {
        const auto r = rsrc(hist + (size_t)j0 * D, BN * D * 2);
#pragma unroll
        for (int i = 0; i < N; ++i) dst[i] = bload(r, off0 + i * step);
    } else if (j0 >= kvl) {
        const auto r = rsrc(chunk + (size_t)(j0 - kvl) * D, (uint32_t)(Lk - j0) * D * 2);
#pragma unroll
        for (int i = 0; i < N; ++i) dst[i] = bload(r, off0 + i * step);
    } else {
        const int nh = kvl - j0;
        const int nc = min(BN - nh, Lq);
        const auto rh = rsrc(hist + (size_t)j0 * D, (uint32_t)nh * D * 2);
        const auto rc = rsrc(chunk, (uint32_t)nc * D * 2);
        const uint32_t shift = (uint32_t)nh * D * 2;  // chunk rows start at tile row nh
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t o = off0 + i * step;
            // below tile row nh, o - shift wraps to a huge offset: out of range, reads 0
            dst[i] = bload(rh, o) | bload(rc, o - shift);
        }
    }
}

// Page table of a head read in place: the cache position of each kept piece
// (pg_P tokens), one byte per piece -- piece y's entry sits in byte y >> 6 of
// lane y & 63, up to 256 pieces in one VGPR, looked up with v_readlane, so the
// tile loop never waits on a scalar load (whose counter it shares with the LDS
// reads).  Piece y starts at cache row entry(y) * pg_P of the head, entry =
// slot * pg_ppf + (piece within its frame).
//   static entry: the pieces of kept frame y / pg_ppf, which is logical frame
//                 y' (y' < st_first) or y' + st_gap;
//   dynamic entry: the pieces of the segments in kept_seg[h] (ascending, as
//                 the selection wrote them).
// The host has checked that every entry fits in a byte.
__device__ __forceinline__ uint32_t kept_piece_table(const AttnArgs &a, int li, int kvl, int lane) {
    uint32_t tab = 0;
    const int ppf = a.pg_ppf;
    const int n = a.st_kept[li];
    if (n >= 0) {
        const int first = a.st_first[li], gap = a.st_gap[li];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int y = lane + 64 * k;
            if (y < n * ppf) {
                const int fy = y / ppf, u = y - fy * ppf;
                tab |= (uint32_t)(a.slots.slot[fy < first ? fy : fy + gap] * ppf + u) << (8 * k);
            }
        }
        return tab;
    }
    const int m = a.pg_L > a.F ? a.pg_L / a.F : 1;           // pieces per segment
    const int n_pieces = kvl / a.pg_P;
    const int32_t *ks = a.kept_seg + (size_t)a.heads.head[li] * a.pg_nseg;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int y = lane + 64 * k;
        if (y < n_pieces) {
            // a kept_seg row and kv_len that disagree must not address outside
            // the head's cache: clamp the segment id
            const int q = y / m, g = min(max(ks[q], 0), a.pg_nseg - 1);
            int t, u;
            if (a.pg_L <= a.F) {
                t = g / ppf;
                u = g - t * ppf;
            } else {
                t = min(g * m + (y - q * m), (int)(a.slab / a.F) - 1);   // a short last segment ends at H
                u = 0;
            }
            tab |= (uint32_t)(a.slots.slot[t] * ppf + u) << (8 * k);
        }
    }
    return tab;
}
__device__ __forceinline__ int kept_piece(uint32_t tab, int y) {
    return (int)((uint32_t)__builtin_amdgcn_readlane((int)tab, y & 63) >> (8 * (y >> 6))) & 255;
}

// j0 / P for 0 <= j0 < 2^31 with the launch's 64-bit reciprocal M = floor(2^64 / P) + 1
// (= magic_hi * 2^32 + magic_lo): floor(j0 * M / 2^64) exactly, since j0 * M / 2^64
// exceeds j0 / P by less than 2^-33 < 1 / P.  A few scalar multiplies instead of
// the generic division sequence in every tile load.
__device__ __forceinline__ int div_piece(const AttnArgs &a, int j0) {
    const uint64_t p = (uint64_t)(uint32_t)j0 * a.pg_magic_hi + __umulhi((uint32_t)j0, a.pg_magic_lo);
    return (int)(p >> 32);
}

// Position of a key tile: its first key j0 and, read in place while j0 is in the
// history, the kept piece y it starts in, the row r within that piece
// (j0 = y * P + r) and that row's offset in the cache.  It moves from run to run
// of full tiles (attn_segment), where the page table is read.
struct PageCursor {
    int j0, y, r;
    uint32_t off;  // element offset of history row j0 in the head's cache (j0 < kvl)
};

// A 64-key tile's rows: part `a`, and where the tile crosses from one source to
// the next (a kept piece to another, or the history to the chunk) part `b`,
// whose first row is `shift` bytes into the tile.  Rows past the last part fall
// outside its buffer's range and read as zero.
struct TileSrc {
    __amdgpu_buffer_rsrc_t a, b;
    uint32_t shift;
    bool two;
};

// Read in place: the history length kvl is a whole number of pieces of P >= 64
// rows, so a tile starting in piece y holds min(P - r, BN) rows of it, then the
// next piece's rows while history lasts, then the chunk's.
template <int D>
__device__ __forceinline__ TileSrc paged_tile(const uint16_t *hist, uint32_t tab, int P, const PageCursor &c,
                                              const uint16_t *chunk, int kvl, int Lk, int Lq) {
    if (c.j0 >= kvl) {
        const auto r = rsrc(chunk + (size_t)(c.j0 - kvl) * D, (uint32_t)(Lk - c.j0) * D * 2);
        return TileSrc{r, r, 0u, false};
    }
    const int na = min(P - c.r, BN);
    const bool more = c.j0 + na < kvl;  // another kept piece follows, else the chunk
    const auto ra = rsrc(hist + c.off, (uint32_t)na * D * 2);
    if (na == BN) return TileSrc{ra, ra, 0u, false};
    return TileSrc{ra,
                   rsrc(more ? hist + (size_t)kept_piece(tab, c.y + 1) * P * D : chunk,
                        (uint32_t)(more ? BN - na : min(BN - na, Lq)) * D * 2),
                   (uint32_t)na * D * 2, true};
}

// Over a compact copy: [hist (kvl rows); chunk (Lq rows)].
template <int D>
__device__ __forceinline__ TileSrc compact_tile(const uint16_t *hist, const uint16_t *chunk, int j0, int kvl, int Lk,
                                                int Lq) {
    if (j0 >= kvl) {
        const auto r = rsrc(chunk + (size_t)(j0 - kvl) * D, (uint32_t)(Lk - j0) * D * 2);
        return TileSrc{r, r, 0u, false};
    }
    const int na = min(kvl - j0, BN);
    const auto ra = rsrc(hist + (size_t)j0 * D, (uint32_t)na * D * 2);
    if (na == BN) return TileSrc{ra, ra, 0u, false};
    return TileSrc{ra, rsrc(chunk, (uint32_t)min(BN - na, Lq) * D * 2), (uint32_t)na * D * 2, true};
}

template <int W>
struct Words;
template <>
struct Words<1> {
    uint32_t w[1];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
        w[0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0);
    }
};
template <>
struct Words<2> {
    uint32_t w[2];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
        w[0] = (uint32_t)v[0];
        w[1] = (uint32_t)v[1];
    }
};

constexpr int kPrefetch = 4;   // operand reads in flight ahead of the product that takes them

// S^T = K Q^T for one key tile in LDS (KS products per key block), the operand
// reads kPrefetch products ahead.
template <int D>
__device__ __forceinline__ void score_block(const uint16_t *ks, int kbase, const bf16x8_t (&qf)[D / 16],
                                            f32x16_t (&s)[2]) {
    using C = Cfg<D>;
    constexpr int NSTEP = 2 * C::KS;
    auto read_a = [&](int i) {
        return __builtin_bit_cast(bf16x8_t, *(const u32x4 *)(ks + kbase + (i & 1) * 32 * C::RSE + (i >> 1) * 16));
    };
    s[0] = f32x16_t{};
    s[1] = f32x16_t{};
    bf16x8_t fr[kPrefetch];
#pragma unroll
    for (int i = 0; i < kPrefetch; ++i) fr[i] = read_a(i);
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
        const bf16x8_t x = fr[st % kPrefetch];
        if (st + kPrefetch < NSTEP) fr[st % kPrefetch] = read_a(st + kPrefetch);
        s[st & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[st >> 1], s[st & 1], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < kPrefetch; ++i) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (st + kPrefetch < NSTEP) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
}

// One segment: positions [t0, t1) of item (h, qt), where position j is key
// tile (j + rot) mod T of the item's T tiles (the order of key tiles does not
// change the result beyond rounding).  slot == nullptr means the segment is the
// whole item and the normalised output (and lse) is written; otherwise the
// partial result goes to the slot.  Uses every thread of the workgroup and
// leaves no LDS read pending.
template <int D, bool PAGED>
__device__ __forceinline__ void attn_segment(const AttnArgs &a, uint16_t *Ks, uint16_t *Vs, uint32_t *redo, int li,
                                             int qt, int t0, int t1, int rot, float *slot) {
    using C = Cfg<D>;
    const int h = a.heads.head[li];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hl = lane >> 5;
    const int Lq = a.Lq;
    const int n = t1 - t0;       // >= 1

    // The wave's 32 query rows, in the B-operand layout: lane holds row l32,
    // dims [16*kk + 8*hl, +8).
    const int qrow = qt * BM + wave * 32 + l32;
    const bool qok = qrow < Lq;
    const uint16_t *Qh = (const uint16_t *)a.Q + (size_t)h * Lq * D;
    bf16x8_t qf[C::KS];
#pragma unroll
    for (int kk = 0; kk < C::KS; ++kk) {
        const u32x4 v = qok ? *(const u32x4 *)(Qh + (size_t)qrow * D + kk * 16 + hl * 8) : u32x4{0, 0, 0, 0};
        qf[kk] = __builtin_bit_cast(bf16x8_t, v);
    }

    const int kvl = entry_kvl<PAGED>(a, li);
    const int Lk = kvl + Lq;
    const uint16_t *Kc = PAGED ? (const uint16_t *)a.K_hist + (size_t)h * a.cap * a.F * D
                               : (const uint16_t *)a.Kc + (size_t)h * a.slab * D;
    const uint16_t *Vc = PAGED ? (const uint16_t *)a.V_hist + (size_t)h * a.cap * a.F * D
                               : (const uint16_t *)a.Vc + (size_t)h * a.slab * D;
    const uint16_t *Kq = (const uint16_t *)a.K_cur + (size_t)h * Lq * D;
    const uint16_t *Vq = (const uint16_t *)a.V_cur + (size_t)h * Lq * D;
    const uint32_t ktab = PAGED ? kept_piece_table(a, li, kvl, lane) : 0u;

    // Loop-invariant per-thread staging geometry.  K: rows r0 + RPP*i, 16-byte
    // chunk c.  V: keys 4*vq .. 4*vq+3 of the tile, dims 2*VW*vc .. +2*VW, stored
    // transposed: row d of the V^T tile holds the tile's 64 keys, and within each
    // 16-key group the key quads sit in the order 0, 2, 1, 3 so that the 8 keys a
    // lane feeds to the value product (16t + 4hl + 0..3 and 16t + 8 + 4hl + 0..3)
    // are contiguous.
    const int c = tid % C::CPR, r0 = tid / C::CPR;
    const uint32_t voff = (uint32_t)(r0 * D + c * 8) * 2u;    // + i*RPP*D*2 bytes
    const int wofs = r0 * C::RSE + c * 8;                      // + i*RPP*RSE elements
    // (lanes of a wave: four key quads by sixteen dim groups, so a V load reads whole
    // 128-byte halves of four rows at D = 128; sixteen quads by four groups, free of
    // bank conflicts in the stores, took 43.3 against 42.4 us on 16 heads of 64 and
    // the same at 480P and 1080P)
    const int vq = (tid & 3) | ((tid >> 6) & 3) << 2, vc = ((tid >> 2) & 15) | ((tid >> 8) & 1) << 4;
    const uint32_t voffv = (uint32_t)(4 * vq * D + vc * 2 * C::VW) * 2u;  // + r*D*2 bytes
    const int vofs = 2 * C::VW * vc * C::TRSE + 16 * (vq >> 2) + 4 * (((vq & 1) << 1) | ((vq >> 1) & 1));

    // The segment's key tiles: kt0, kt0 + 1, ... (mod T); where the keys end inside
    // tile T - 1 and it is one of them, it comes first (the first tile's row maxima
    // are taken, with the keys past Lk masked); the others are full ones.
    const int T = (Lk + BN - 1) / BN;
    const int kt0 = (t0 + rot) % T;
    const bool ragged = Lk % BN != 0 && T - 1 - kt0 < n;
    // The full tiles, which the order wraps over; none where nothing follows the first
    // one: the prologue's later loads then come from an empty buffer (a part of one
    // tile 1.2 us sooner; for D = 64, half the bytes, it measured 0.2 us the other way).
    const int Tw = D == 128 && n == 1 ? 0 : Lk / BN;
    const int P = PAGED ? a.pg_P : 0;
    auto piece_off = [&](int y, int r) { return (uint32_t)(kept_piece(ktab, y) * P + r) * (uint32_t)D; };
    // the next tile of the rotated order: read in place, the offset moves on by a
    // tile inside a piece, and the page table is read where a piece ends
    auto advance = [&](PageCursor &cu) {
        cu.j0 += BN;
        if (cu.j0 >= Tw * BN) {         // the order wraps to the first tile
            cu = PageCursor{0, 0, 0, PAGED && kvl > 0 ? piece_off(0, 0) : 0u};
        } else if (PAGED) {
            cu.r += BN;
            cu.off += BN * D;
            if (cu.r >= P) {
                cu.r -= P;
                ++cu.y;
                if (cu.j0 < kvl) cu.off = piece_off(cu.y, cu.r);
            }
        }
    };

    u32x4 kst[C::NV];
    Words<C::VW> vst[4];
    // Sources of the next tile's loads.  Full tiles that follow one another in one
    // source (a piece, the compact history, the chunk) are a run: `left` more of them
    // at soff, for which a tile's loads take a scalar add.  Any other tile is a run of
    // one, of up to two parts.
    __amdgpu_buffer_rsrc_t krun = rsrc(Kq, 0), vrun = krun, k2 = krun, v2 = krun;
    uint32_t soff = 0, shift = 0;
    int left = 0;
    bool two = false;
    auto one_tile = [&](const PageCursor &cu) {
        const TileSrc k = PAGED ? paged_tile<D>(Kc, ktab, P, cu, Kq, kvl, Lk, Lq)
                                : compact_tile<D>(Kc, Kq, cu.j0, kvl, Lk, Lq);
        const TileSrc v = PAGED ? paged_tile<D>(Vc, ktab, P, cu, Vq, kvl, Lk, Lq)
                                : compact_tile<D>(Vc, Vq, cu.j0, kvl, Lk, Lq);
        krun = k.a;
        vrun = v.a;
        k2 = k.b;
        v2 = v.b;
        shift = k.shift;
        two = k.two;
        soff = 0;
        left = 1;
    };
    // the run that starts at cu, and cu past it
    auto next_run = [&](PageCursor &cu) {
        const int end = Tw * BN;
        const bool hist = cu.j0 < kvl;
        const int lim = !hist ? end : min(end, PAGED ? cu.j0 + P - cu.r : kvl);
        left = (lim - cu.j0) / BN;
        if (PAGED && hist) left = min(left, (kvl - cu.j0 + BN - 1) / BN);
        left = min(left, 1 << 16);    // (soff stays below 2^31)
        if (left > 0) {
            const size_t off = hist && PAGED ? (size_t)cu.off : (size_t)(hist ? cu.j0 : cu.j0 - kvl) * D;
            krun = rsrc((hist ? Kc : Kq) + off, (uint32_t)left * (BN * D * 2));
            vrun = rsrc((hist ? Vc : Vq) + off, (uint32_t)left * (BN * D * 2));
            soff = 0;
            const int m = left - 1;   // (advance adds the last one)
            cu.j0 += m * BN;
            cu.r += m * BN;
            cu.off += (uint32_t)(m * BN * D);
        } else {
            one_tile(cu);
        }
        advance(cu);
    };
    // one tile of the run into registers
    auto load = [&]() {
        if (!two) {
#pragma unroll
            for (int i = 0; i < C::NV; ++i) kst[i] = bload(krun, voff + i * (C::RPP * D * 2), soff);
#pragma unroll
            for (int r = 0; r < 4; ++r) vst[r].load(vrun, voffv + r * (D * 2), soff);
        } else {
            // each lane from the part that holds its row: no load waits for another
#pragma unroll
            for (int i = 0; i < C::NV; ++i) {
                const uint32_t o = voff + i * (C::RPP * D * 2);
                if (o < shift) kst[i] = bload(krun, o, 0);
                else kst[i] = bload(k2, o - shift, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t o = voffv + r * (D * 2);
                if (o < shift) vst[r].load(vrun, o, 0);
                else vst[r].load(v2, o - shift, 0);
            }
            two = false;
        }
        soff += BN * D * 2;
        --left;
    };
    constexpr int kStores = C::NV + 2 * C::VW;
    // store x of the staged tile: the K vectors, then the V^T rows (4 keys each)
    auto store = [&](int x, int b, const u32x4 (&kst)[C::NV], const Words<C::VW> (&vst)[4]) {
        if (x < C::NV) {
            *(u32x4 *)(Ks + b * C::TILE + wofs + x * C::RPP * C::RSE) = kst[x];
            return;
        }
        const int e = x - C::NV, j = e >> 1;
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;   // high or low halves
        *(uint2 *)(Vs + b * C::VTILE + vofs + e * C::TRSE) =
            make_uint2(__builtin_amdgcn_perm(vst[1].w[j], vst[0].w[j], sel),
                       __builtin_amdgcn_perm(vst[3].w[j], vst[2].w[j], sel));
    };

    // LDS read bases of the MFMA operands.
    // K (A of S^T): lane reads row 32*kb + l32, dims 16*kk + 8*hl.
    const int kbase = l32 * C::RSE + hl * 8;
    // V^T (A of O^T): lane reads row 32*mb + l32, keys 16t + 8hl .. +8 of the
    // permuted V^T tile.
    const int vbase = l32 * C::TRSE + 8 * hl;

    // Steps of iteration `it`, in four runs of products:
    //   A  score products of key block 0 of tile it        (KS)
    //   B  value products of key block 1 of tile it - 1    (2 MB: key group t, then dim block)
    //   C  score products of key block 1 of tile it        (KS)
    //   D  value products of key block 0 of tile it        (2 MB)
    // so the exponentials of a key block have two runs of other products between
    // its scores and its value products.  Operand A of step x (x >= NSTEP: the
    // next iteration's run A).
    constexpr int xB = C::KS, xC = xB + 2 * C::MB, xD = xC + C::KS, NSTEP = xD + 2 * C::MB;
    static_assert(NSTEP % kPrefetch == 0 && kPrefetch <= C::KS, "operand ring");
    auto buf = [](int tile) { return tile & (kBufs - 1); };
    auto read_a = [&](int x, int it) -> bf16x8_t {
        const bool score = x < xB || (x >= xC && x < xD) || x >= NSTEP;
        if (score) {
            const int kb = x >= xC && x < xD, kk = x >= NSTEP ? x - NSTEP : kb ? x - xC : x;
            return __builtin_bit_cast(bf16x8_t, *(const u32x4 *)(Ks + buf(x >= NSTEP ? it + 1 : it) * C::TILE + kbase +
                                                                kb * 32 * C::RSE + kk * 16));
        }
        const int y = x >= xD ? x - xD : x - xB + 2 * C::MB, t = y / C::MB, mb = y % C::MB;
        return __builtin_bit_cast(bf16x8_t, *(const u32x4 *)(Vs + buf(x >= xD ? it : it - 1) * C::VTILE + vbase +
                                                            (32 * mb) * C::TRSE + 16 * t));
    };

    f32x16_t o[C::MB];
    float m_run, l_run;   // reference of the exponentials (log2 units); this lane's share of the running sum
    const float c2 = a.scale_log2;

    bool every = false;   // take every tile's row maximum
    for (;;) {
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb) o[mb] = f32x16_t{};
        m_run = -__builtin_inff();
        l_run = 0.f;
        f32x16_t s[2];
        bf16x8_t pb[4];
        bf16x8_t fr[kPrefetch];

        // Prologue: the first two tiles into LDS, the third into registers.
        auto cursor_at = [&](int j0) {
            PageCursor cu{j0, 0, 0, 0u};
            if (PAGED && j0 < kvl) {
                cu.y = div_piece(a, j0);
                cu.r = j0 - cu.y * P;
                cu.off = piece_off(cu.y, cu.r);
            }
            return cu;
        };
        PageCursor cu = cursor_at(ragged ? (T - 1) * BN : kt0 * BN);
        one_tile(cu);
        // the others go on at kt0 + 1, or at kt0 where the last tile came first
        if (ragged && kt0 < T - 1) cu = cursor_at(kt0 * BN);
        else advance(cu);
        // (past the segment's end the order goes on over valid tiles, never used; where
        // the keys fill no tile, over an empty buffer)
        auto fetch = [&]() {
            if (left == 0) {
                if (Tw > 0) {
                    next_run(cu);
                } else {
                    krun = vrun = rsrc(Kq, 0);
                    soff = 0;
                    left = 1;
                }
            }
            load();
        };
        // (both tiles' loads in flight together)
        load();
        u32x4 k0[C::NV];
        Words<C::VW> v0[4];
#pragma unroll
        for (int i = 0; i < C::NV; ++i) k0[i] = kst[i];
#pragma unroll
        for (int r = 0; r < 4; ++r) v0[r] = vst[r];
        fetch();
#pragma unroll
        for (int x = 0; x < kStores; ++x) store(x, 0, k0, v0);
#pragma unroll
        for (int x = 0; x < kStores; ++x) store(x, 1, kst, vst);
        fetch();
        __syncthreads();
        // Let every outstanding load (the Q fragments included) land once here, so
        // the loop's score products carry no wait on the staging loads in flight.
        __builtin_amdgcn_s_waitcnt(0);

        auto product = [&](int x, const bf16x8_t &f) {
            if (x < xB || (x >= xC && x < xD)) {
                const int kb = x >= xC, kk = kb ? x - xC : x;
                s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[kk], kk == 0 ? f32x16_t{} : s[kb], 0, 0, 0);
            } else {
                const int y = x >= xD ? x - xD : x - xB + 2 * C::MB, t = y / C::MB, mb = y % C::MB;
                o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pb[t], o[mb], 0, 0, 0);
            }
        };
        // P^T as the B operand: k-step t covers keys 16t + {4hl..4hl+3, 8+4hl..8+4hl+3},
        // i.e. accumulator entries s[t/2][8*(t%2) + j]; pair p is entries 2p, 2p + 1 in that order.
        float e0, e1, m_exp;
        auto exp_pair = [&](int p) {
            const int t = p >> 2, j = 8 * (t & 1) + 2 * (p & 3);
            e0 = __builtin_amdgcn_exp2f(fmaf(s[t >> 1][j], c2, -m_exp));
            e1 = __builtin_amdgcn_exp2f(fmaf(s[t >> 1][j + 1], c2, -m_exp));
        };
        auto round_pair = [&](int p) {
            const int t = p >> 2, j = 2 * (p & 3);
            pb[t][j] = (__bf16)e0;
            pb[t][j + 1] = (__bf16)e1;
        };
        // The row sum adds the bf16-rounded probabilities -- exactly the P the
        // value product consumes -- two at a time, in two chains.
        float l2 = 0.f;
        auto sum_pair = [&](int p) {
            const int t = p >> 2, j = 2 * (p & 3);
            const bf16x2_t pr = {pb[t][j], pb[t][j + 1]};
            if (t & 1) l2 = __builtin_amdgcn_fdot2_f32_bf16(pr, kOnes2, l2, false);
            else l_run = __builtin_amdgcn_fdot2_f32_bf16(pr, kOnes2, l_run, false);
        };
        int it = 0;
        // Row maximum of the tile whose scores s holds, in log2 units.
        auto row_max = [&](const f32x16_t &s0, const f32x16_t &s1) {
            float mx = fmaxf(s0[0], s0[1]);
#pragma unroll
            for (int i = 2; i < 16; ++i) mx = fmaxf(mx, s0[i]);
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s1[i]);
            return fmaxf(mx, __shfl_xor(mx, 32)) * c2;
        };
        // A finite reference above every score of a row maximum mx: the rounding of a
        // score times c2 passes the exponent by half a step, which overflows it where
        // a step of mx is large (scores of -1e30).
        auto above = [](float mx) {
            mx = fmaxf(mx, -kLowest);
            return mx <= kLowest ? fminf(fmaf(fabsf(mx), 0x1p-23f, mx), kLowest) : mx;
        };
        // Pair of probabilities formed in step x: those of key block 0 from its
        // second step after run A on, those of key block 1 from the second after run
        // C; the last ones (from kLate on) in run A of the next iteration.
        constexpr int kLate = D == 128 ? 12 : 11;
        auto pair_at = [](int x) -> int {
            if (D == 128) return x < 8 ? (x % 2 == 0 ? 12 + x / 2 : -1) : (x >= 9 && x % 2 == 1 ? (x - 9) / 2 : -1);
            return x <= 4 ? 11 + x : x - 5;
        };
        // The tile stored in this iteration is visible to the others from here on.  LDS
        // operations finish in order and kPrefetch operand reads follow the stores, so
        // at most kPrefetch outstanding ones means that the stores are done; the reads
        // themselves stay in flight.
        auto tile_barrier = [&]() {
            __asm__ volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(kPrefetch) : "memory");
        };
        // steps [x0, x1) alone
        auto run = [&](int x0, int x1) {
            bf16x8_t f[2];
            f[0] = read_a(x0, it);
#pragma unroll
            for (int x = x0; x < x1; ++x) {
                if (x + 1 < x1) f[(x + 1 - x0) & 1] = read_a(x + 1, it);
                product(x, f[(x - x0) & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // (m_exp opaque in every iteration: else the compiler takes the exponentials
        // that both ways on from an iteration begin with into its end)
        auto set_m = [&]() {
            m_exp = m_run;
            __asm__ volatile("" : "+v"(m_exp));
        };
        // P formed here, not where the next iteration first needs it
        auto pin_p = [&](int t) { __asm__ volatile("" : "+v"(pb[t])); };
        // the value products of key block 1 of the tile before
        auto finish_tile = [&]() {
            set_m();
#pragma unroll
            for (int p = kLate; p < 16; ++p) {
                exp_pair(p);
                round_pair(p);
                sum_pair(p);
            }
            run(xB, xC);
        };
        // The first tile: its runs in turn, its row maximum (keys past Lk masked) the
        // reference of the exponentials.
#pragma unroll
        for (int x = 0; x < kStores; ++x) store(x, buf(it + 2), kst, vst);
        run(0, xB);
        run(xC, xD);
        if (ragged) {
            const int room = Lk - 1 - ((T - 1) * BN + 4 * hl);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint32_t past = (uint32_t)((room - (kb * 32 + 8 * (i >> 2) + (i & 3))) >> 31);
                    s[kb][i] = __uint_as_float((past & 0xff800000u) | (~past & __float_as_uint(s[kb][i])));
                }
        }
        // A row whose scores here are all -inf takes the lowest finite reference: its
        // keys weigh nothing, and the first other ones overflow its sum.
        m_run = row_max(s[0], s[1]);
        m_run = every ? above(m_run) : fmaxf(m_run, -kLowest);
        set_m();
#pragma unroll
        for (int p = 0; p < kLate; ++p) {
            exp_pair(p);
            round_pair(p);
            sum_pair(p);
        }
        run(xD, NSTEP);
#pragma unroll
        for (int i = 0; i < kPrefetch; ++i) fr[i] = read_a(NSTEP + i, it);
        fetch();
        ++it;
        tile_barrier();
        // The others.  Per step one product, the read of a later step's operand and a
        // share of the tile's other work, pinned in this order.
        while (it < n) {
            if (every) {
                // The running max moves where this tile's exceeds it by more than
                // kRescaleSlack, by whole powers of two (what is scaled stays as it was
                // rounded), or to the tile's own beyond kFarMove, where a sum with the
                // difference would lose it; what the previous tile still has to do takes
                // the new one.
                run(0, xB);
                float mx = row_max(s[0], s[0]);
#pragma unroll
                for (int kk = 0; kk < C::KS; ++kk)
                    s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_a(xC + kk, it), qf[kk],
                                                                   kk == 0 ? f32x16_t{} : s[0], 0, 0, 0);
                mx = above(fmaxf(mx, row_max(s[0], s[0])));
                if (__ballot(mx > m_run + kRescaleSlack)) {
                    const bool move = mx > m_run + kRescaleSlack, far = move && mx - m_run > kFarMove;
                    const float up = far ? mx - m_run : move ? ceilf(mx - m_run) : 0.f;
                    const float alpha = __builtin_amdgcn_exp2f(-up);
                    l_run *= alpha;
                    l2 *= alpha;
#pragma unroll
                    for (int mb = 0; mb < C::MB; ++mb) o[mb] *= alpha;
#pragma unroll
                    for (int p = 8; p < kLate; ++p) {
                        exp_pair(p);
                        e0 *= alpha;
                        e1 *= alpha;
                        round_pair(p);
                    }
                    m_run = far ? mx : m_run + up;
                }
            }
            set_m();
#pragma unroll
            for (int x = 0; x < NSTEP; ++x) {
                product(x, fr[x % kPrefetch]);
                fr[x % kPrefetch] = read_a(x + kPrefetch, it);
                const int p0 = x > 0 ? pair_at(x - 1) : -1, p = pair_at(x);
                if (p0 >= 0) {
                    round_pair(p0);
                    sum_pair(p0);
                }
                if (p >= 0) exp_pair(p);
                if (x == NSTEP - 1 && p >= 0) {
                    round_pair(p);
                    sum_pair(p);
                }
                constexpr int kS = D == 128 ? 2 : 1;
                if (x >= xC && (x - xC) % kS == 0 && (x - xC) / kS < kStores) store((x - xC) / kS, buf(it + 2), kst, vst);
                __builtin_amdgcn_sched_barrier(0);
            }
            pin_p(2);
            fetch();
            ++it;
            tile_barrier();
        }
        // (`it` has moved on: the last tile is "the tile before")
        finish_tile();
        l_run += l2;

        if (every) {
            // (a workgroup whose range goes on stores the next segment's first tiles
            // into buffers that a slower wave may still read here)
            __syncthreads();
            break;
        }
        // redo?
        float z = 0.f;
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) z = fmaf(o[mb][i], 0.f, z);
        if (__ballot(qok && !(l_run <= kSumLimit && z == 0.f)) && lane == 0) *redo = 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane((int)*(volatile uint32_t *)redo) == 0) break;
        __syncthreads();
        if (tid == 0) *redo = 0;
        every = true;
    }

    const float l_tot = l_run + __shfl_xor(l_run, 32);
    float inv = 1.f / l_tot;
    if (slot) {
        if (l_tot == 0.f) inv = 0.f;   // a part whose keys all score -inf: weight 0, not 0 * inf
        // device-scope stores: the workgroup that merges the item may run on
        // another XCD, within this launch
        unsigned long long *op = (unsigned long long *)slot;
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint2 v = pack_bf16x4(o[mb][4 * g] * inv, o[mb][4 * g + 1] * inv, o[mb][4 * g + 2] * inv,
                                            o[mb][4 * g + 3] * inv);
                put_shared(op + ((wave * C::MB + mb) * 4 + g) * 64 + lane, v);
            }
        if (hl == 0) {
            // a sum far above one hands its exponent to the maximum: the weights by
            // which the merge multiplies outputs stay small
            const int e = l_tot > 0x1p24f ? __builtin_amdgcn_frexp_expf(l_tot) : 0;
            put_shared(slot + BM * D / 2 + wave * 32 + l32, m_run + (float)e);
            put_shared(slot + BM * D / 2 + BM + wave * 32 + l32, __builtin_amdgcn_ldexpf(l_tot, -e));
        }
        return;
    }
    if (qok) {
        uint16_t *Oh = (uint16_t *)a.O + ((size_t)h * Lq + qrow) * D;
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g)  // O^T rows d = 32mb + 8g + 4hl + {0..3}
                *(uint2 *)(Oh + mb * 32 + 8 * g + 4 * hl) =
                    pack_bf16x4(o[mb][4 * g] * inv, o[mb][4 * g + 1] * inv, o[mb][4 * g + 2] * inv,
                                o[mb][4 * g + 3] * inv);
        if (a.lse && hl == 0)
            a.lse[(size_t)h * Lq + qrow] = fmaf(m_run, 0.69314718055994530942f, logf(l_tot));
    }
}

// BAL = false: one workgroup per work item (head, query tile), dealt so that
// each XCD (blocks go to the 8 XCDs round-robin) receives a contiguous range
// of items: the query tiles of a head then share that XCD's L2.
// BAL = true: the balanced schedule above, with the same XCD-contiguous
// assignment of ranges (n_blocks is a multiple of 8).
template <int D, bool BAL, bool PAGED>
__global__ __launch_bounds__(kThreads, 2) void attn_bf16_kernel(AttnArgs a) {
    using C = Cfg<D>;
    __shared__ __attribute__((aligned(16))) uint16_t Ks[kBufs * C::TILE];
    __shared__ __attribute__((aligned(16))) uint16_t Vs[kBufs * C::VTILE];
    __shared__ uint32_t flag, redo;
    if (threadIdx.x == 0) redo = 0;   // (barriers follow before its first use)

    if (!BAL) {
        const int item = (blockIdx.x & 7) * a.items_per_xcd + (blockIdx.x >> 3);
        if (item >= a.n_items) return;
        const int li = item / a.n_qtiles;
        attn_segment<D, PAGED>(a, Ks, Vs, &redo, li, item - li * a.n_qtiles, 0, entry_tiles<PAGED>(a, li), 0, nullptr);
        return;
    }
    const WorkList wl = work_list<PAGED>(a);
    const Schedule sc = make_schedule(a, wl);
    const int r = (blockIdx.x & 7) * (a.n_blocks >> 3) + (blockIdx.x >> 3);
    if (sc.total == 0) return;
    // this workgroup's segments: one part of an item, or a range over items
    const int parts = whole_parts(a, wl, sc);
    if (!parts && r >= sc.G) return;
    int64_t cur = parts ? 0 : sc.start(r);
    const int64_t end = parts ? 1 : sc.start(r + 1);
    bool first = true;
    while (cur < end) {
        int li, qt, t0, t1, rot, b0, n_parts, s0;
        if (parts) {
            const int item = r / parts, j = r - item * parts;
            if (item >= a.n_items) return;
            li = item / a.n_qtiles;
            qt = item - li * a.n_qtiles;
            const int T = __builtin_amdgcn_readlane(wl.T, li);
            n_parts = min(parts, T);
            if (j >= n_parts) return;
            t0 = (int)((uint32_t)T * j / n_parts);   // (T < 2^19: cache and chunk are below 2^31 bytes each)
            t1 = (int)((uint32_t)T * (j + 1) / n_parts);
            rot = 0;
            b0 = item * parts;
            s0 = 2 * b0;
            cur = end;
        } else {
            // locate the item holding tile `cur`
            const ItemPos ip = locate(wl, cur);
            const int64_t ibase = ip.ibase;
            li = ip.li;
            qt = ip.qt;
            t0 = (int)(cur - ibase);
            t1 = (int)((end < ibase + ip.T ? end : ibase + ip.T) - ibase);
            b0 = sc.owner(ibase);
            n_parts = sc.owner(ibase + ip.T - 1) - b0 + 1;
            s0 = first_slot(sc, ibase);
            // Rotate the item's key tiles so that its first part, started at time
            // tau0 = ibase - start(b0) of its workgroup, reads key tile tau mod T at
            // time tau: the first parts of all items of a head then sweep its K/V in
            // step (later parts in step among themselves, shifted by a range length),
            // so the XCD's L2 serves the re-reads.
            rot = (int)((ibase - sc.start(b0)) % ip.T);
            cur = ibase + t1;
        }
        float *slot = n_parts == 1 ? nullptr : a.part + (size_t)(2 * r + (first ? 0 : 1)) * slot_floats<D>();
        attn_segment<D, PAGED>(a, Ks, Vs, &redo, li, qt, t0, t1, rot, slot);
        if (slot) {
            // the last of the item's parts to arrive combines them (no wait:
            // every other part is complete when its workgroup arrives)
            uint32_t *cnt = a.item_counters + (size_t)(li * a.n_qtiles + qt) * kItemCounterStride;
            if (arrive_last(cnt, (uint32_t)n_parts, &flag))
                merge_rows<D, 64>(a, b0, b0 + n_parts - 1, s0, li, qt, threadIdx.x >> 6, threadIdx.x & 63);
        }
        first = false;
    }
}

// ------------------------------------------------------------ attention mass
// Offline head profiling (Sec. 4.1, Eq. 1) needs, per head, the attention mass
// each block (bin) of F keys of [Kc[0:kv_len]; K_cur] receives: the sum over
// all query rows of the softmax probabilities exp(scale*q.k - lse_row), with
// lse from fkv_chunk_attention over the same keys.
//
// Work unit = (head, 256-row query tile, bin), 8 waves x 32 rows; the units in
// that order are split evenly over two workgroups per CU (every unit costs the
// same), so a unit is computed by one workgroup and its eight wave sums are
// written once: no read-modify-write, a fixed order, the same bits on every
// run.  A bin's keys are read in tiles of 64 from its first key on (its last
// tile is masked), double buffered in LDS, the next tile's loads in flight
// during the products; a workgroup streams the consecutive bins of a query
// tile without draining.  Per tile the waves compute S^T with the attention
// kernel's score product (the same MFMA sequence, so the same fp32 scores) and
// every lane adds its probabilities in fp32; the lanes are summed (a fixed
// butterfly) once per bin.
//
// Bound: the VALU -- per 64-key tile a wave issues 32 exponentials (quarter
// rate), 32 FMAs and 32 adds against 16 products (512 cycles); four waves per
// SIMD overlap the two.  480P, 12 heads over the whole 21-frame history (37440
// keys): 533 us, 1.01 PFLOP/s of score products; 1350 us with one workgroup
// per query tile, staging and products in turn, and every tile's sum reduced
// and added to its bin in memory.  Finalize 4 us (28 us with one workgroup per
// head walking each bin's sums in series).
//
// Bins are not aligned to tiles: a bin of F keys takes ceil(F / 64) tiles, the
// last one partly empty (F = 65: 51% of the products count).  SHORT, for bins
// of at most half a tile: a unit is the 64 / F whole bins that fit one tile.
// Per tile the rows of each key are summed by a reduce-scatter over the lanes
// (31 exchanges, after which a lane holds one key's sum) and the keys of each
// bin by one lane from LDS, whatever the number of bins.  40 heads of 128, 4096
// query rows, F = 1 / 8 / 16 / 32: 0.38 / 0.37 / 0.50 / 0.56 ms; 12.7 / 2.24 /
// 1.49 / 0.78 with a tile per bin, 7.5 / 1.61 / 1.30 / 0.88 with aligned tiles
// and a masked reduction per bin that a tile touches.
__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// LDS written by other lanes of the wave is read after this (and the reverse): a
// wave's LDS operations finish in order, so it only keeps the compiler's order.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int mass_bins_of(const AttnArgs &a, int h) {
    return (head_kvl(a, h) + a.Lq + a.mass_F - 1) / a.mass_F;
}
constexpr int kShortBin = BN / 2;   // largest bin (keys) of the SHORT kernel

template <int D, bool SHORT>
__global__ __launch_bounds__(kThreads, 4) void attn_mass_kernel(AttnArgs a) {
    using C = Cfg<D>;
    __shared__ __attribute__((aligned(16))) uint16_t Ks[2][C::TILE];
    __shared__ float key_sums[SHORT ? kThreads / 64 : 1][BN];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hl = lane >> 5;
    const int Lq = a.Lq;
    const int per = SHORT ? BN / a.mass_F : 1;   // bins per unit
    const int G = per * a.mass_F;                // keys per unit
    const float c2 = a.scale_log2;
    // staging geometry: all 512 threads, rows r0 + RPP2*i
    constexpr int RPP2 = kThreads / C::CPR;
    constexpr int NV2 = BN / RPP2;
    const int c = tid % C::CPR, r0 = tid / C::CPR;
    const uint32_t voff = (uint32_t)(r0 * D + c * 8) * 2u;
    const int wofs = r0 * C::RSE + c * 8;
    const int kbase = l32 * C::RSE + hl * 8;

    // the units of this workgroup: T = units of the entry's head
    WorkList wl;
    wl.T = lane < a.heads.n ? (head_kvl(a, lane) + Lq + G - 1) / G : 0;   // (every head, in order)
    {
        long long v = (long long)a.n_qtiles * wl.T;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const long long u = __shfl_up(v, d, 64);
            if (lane >= d) v += u;
        }
        wl.incl = (int64_t)v;
    }
    const Schedule sc = make_schedule(a, wl);
    const int r = (blockIdx.x & 7) * (a.n_blocks >> 3) + (blockIdx.x >> 3);
    if (r >= sc.G) return;
    const int64_t end = sc.start(r + 1);
    for (int64_t cur = sc.start(r); cur < end;) {
        const ItemPos ip = locate(wl, cur);
        const int h = ip.li, qt = ip.qt;
        const int b0 = (int)(cur - ip.ibase);
        const int b1 = (int)((end < ip.ibase + ip.T ? end : ip.ibase + ip.T) - ip.ibase);
        cur = ip.ibase + b1;

        const int qrow = qt * BM + wave * 32 + l32;
        const bool qok = qrow < Lq;
        const uint16_t *Qh = (const uint16_t *)a.Q + (size_t)h * Lq * D;
        bf16x8_t qf[C::KS];
#pragma unroll
        for (int kk = 0; kk < C::KS; ++kk) {
            const u32x4 v = qok ? *(const u32x4 *)(Qh + (size_t)qrow * D + kk * 16 + hl * 8) : u32x4{0, 0, 0, 0};
            qf[kk] = __builtin_bit_cast(bf16x8_t, v);
        }
        // rows past Lq contribute nothing: their bias is -inf
        const float bias = qok ? -a.lse[(size_t)h * Lq + qrow] * 1.4426950408889634f : -__builtin_inff();
        const int kvl = head_kvl(a, h);
        const int Lk = kvl + Lq;
        const uint16_t *Kc = (const uint16_t *)a.Kc + (size_t)h * a.slab * D;
        const uint16_t *Kq = (const uint16_t *)a.K_cur + (size_t)h * Lq * D;
        float *bins = a.part + (((size_t)h * a.n_qtiles + qt) * 8 + wave) * a.mass_bins;

        // tile positions: unit b, first key j; past the last unit the position is empty
        struct Pos {
            int b, j, hi;   // hi: end of the unit's keys
        };
        auto bin_at = [&](int b) { return Pos{b, b * G, min((b + 1) * G, Lk)}; };
        auto next = [&](const Pos &p) {
            return p.j + BN < p.hi ? Pos{p.b, p.j + BN, p.hi} : bin_at(p.b + 1);
        };
        u32x4 stage[4];
        auto load = [&](const Pos &p) {
            load_tile<D, NV2>(Kc, Kq, p.j, kvl, Lk, Lq, stage, voff, RPP2 * D * 2);
        };
        auto store = [&](uint16_t *t) {
#pragma unroll
            for (int i = 0; i < NV2; ++i) *(u32x4 *)(t + wofs + i * RPP2 * C::RSE) = stage[i];
        };
        Pos p = bin_at(b0), p1 = next(p);
        load(p);
        store(Ks[0]);                       // (the previous item's last reads are behind its last barrier)
        if (p1.b < b1) load(p1);
        __syncthreads();
        float v0 = 0.f, v1 = 0.f;
        for (int it = 0; p.b < b1; ++it) {
            const Pos p2 = next(p1);
            if (p1.b < b1) {
                store(Ks[(it + 1) & 1]);    // last read before the barrier just passed
                if (p2.b < b1) load(p2);
            }
            f32x16_t s[2];
            score_block<D>(Ks[it & 1], kbase, qf, s);
            // keys of this lane: j + 32kb + 8(i/4) + 4hl + i%4
            if (p.j + BN > p.hi) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (p.j + kb * 32 + 8 * (i >> 2) + 4 * hl + (i & 3) >= p.hi) s[kb][i] = -__builtin_inff();
            }
            if constexpr (SHORT) {
                float x[32];   // entry e: key 32(e/16) + 8(e%16/4) + 4hl + e%4
#pragma unroll
                for (int e = 0; e < 32; ++e) x[e] = __builtin_amdgcn_exp2f(fmaf(s[e >> 4][e & 15], c2, bias));
                // lanes hl * 32 + l, l < 32: the sum of entry l over the half's rows
#pragma unroll
                for (int m = 16; m > 0; m >>= 1) {
                    const bool up = lane & m;
#pragma unroll
                    for (int e = 0; e < m; ++e) {
                        const float give = up ? x[e] : x[e + m];
                        x[e] = (up ? x[e + m] : x[e]) + __shfl_xor(give, m);
                    }
                }
                float *ks = key_sums[wave];
                ks[(l32 >> 4) * 32 + 8 * ((l32 >> 2) & 3) + 4 * hl + (l32 & 3)] = x[0];
                wave_sync();
                float v = 0.f;
                const int b = p.b * per + lane;    // this lane's bin
                if (lane < per && b * a.mass_F < Lk) {
                    for (int k = 0; k < a.mass_F; ++k) v += ks[lane * a.mass_F + k];
                    bins[b] = v;
                }
                wave_sync();
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    v0 += __builtin_amdgcn_exp2f(fmaf(s[0][i], c2, bias));
                    v1 += __builtin_amdgcn_exp2f(fmaf(s[1][i], c2, bias));
                }
            }
            if (!SHORT && p1.b != p.b) {
                const float v = wave_sum_f(v0 + v1);
                if (lane == 0) bins[p.b] = v;
                v0 = v1 = 0.f;
            }
            __syncthreads();
            p = p1;
            p1 = p2;
        }
    }
}

// mass[h][b]: the sum of the bin's n_qtiles * 8 wave sums (0 for a bin past the
// head's keys).  One wave per bin: lane l adds rows l, l + 64, ... in order,
// then a fixed butterfly.
__global__ __launch_bounds__(256) void attn_mass_finalize_kernel(AttnArgs a) {
    const int h = blockIdx.y, lane = threadIdx.x & 63;
    const int n = a.n_qtiles * 8, nb = mass_bins_of(a, h);
    for (int b = blockIdx.x * 4 + (threadIdx.x >> 6); b < a.mass_bins; b += gridDim.x * 4) {
        float v = 0.f;
        if (b < nb)
            for (int k = lane; k < n; k += 64) v += a.part[((size_t)h * n + k) * a.mass_bins + b];
        v = wave_sum_f(v);
        if (lane == 0) {
            float *out = a.mass_out + (size_t)h * a.mass_bins + b;
            *out = a.mass_acc ? *out + v : v;
        }
    }
}

}  // namespace

template <bool PAGED>
hipError_t launch_bf16(const AttnArgs &a, int head_dim, hipStream_t s) {
    if (a.n_blocks > 0) {
        if (head_dim == 128)
            hipLaunchKernelGGL((attn_bf16_kernel<128, true, PAGED>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
        else
            hipLaunchKernelGGL((attn_bf16_kernel<64, true, PAGED>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
        return hipGetLastError();
    }
    const unsigned blocks = (unsigned)a.items_per_xcd * 8u;
    if (head_dim == 128)
        hipLaunchKernelGGL((attn_bf16_kernel<128, false, PAGED>), dim3(blocks), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((attn_bf16_kernel<64, false, PAGED>), dim3(blocks), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_attention_bf16(const AttnArgs &a, int head_dim, hipStream_t s) {
    return a.paged ? launch_bf16<true>(a, head_dim, s) : launch_bf16<false>(a, head_dim, s);
}

hipError_t launch_attention_mass(const AttnArgs &a, int head_dim, hipStream_t s) {
    const bool bins_short = a.mass_F <= kShortBin;
    if (head_dim == 128 && bins_short)
        hipLaunchKernelGGL((attn_mass_kernel<128, true>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else if (head_dim == 128)
        hipLaunchKernelGGL((attn_mass_kernel<128, false>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else if (bins_short)
        hipLaunchKernelGGL((attn_mass_kernel<64, true>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((attn_mass_kernel<64, false>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    const unsigned bx = (unsigned)((a.mass_bins + 3) / 4);
    hipLaunchKernelGGL(attn_mass_finalize_kernel, dim3(bx < 64 ? bx : 64, (unsigned)a.n_heads), dim3(256), 0, s, a);
    return hipGetLastError();
}

size_t attention_part_bytes(int head_dim) { return (size_t)kAttnRowsBf16 * (head_dim / 2 + 2) * 4; }

}  // namespace fkv
