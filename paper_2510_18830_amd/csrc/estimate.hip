// Vertical-slash pattern estimation on one GPU (Algorithm 1; Section 4.1).
//
// For each (batch, query head) the last L <= 64 query rows n attend causally
// to the whole sequence: z = scale q_n . k_m for m <= n, P = softmax over m.
//   v_score[m]     = sum_n P[n, m]            (column / vertical scores)
//   s_score[delta] = sum_n P[n, n - delta]    (diagonal / slash scores)
// followed by an exact top-k of each (ties to the lower index, ascending
// output).  The softmax needs each row's normaliser before any column or
// diagonal sum, so K is streamed twice:
//   pass1    per (up to four heads of a KV group, chunk of 2 to 32 key tiles):
//            S^T = K Q^T on MFMA, per-row running max and sum of exp2 -> chunk
//            partials
//   combine  per head: log2-sum-exp of the chunk partials for the 64 rows
//   pass2    the same workgroups: S = Q K^T on MFMA (lane = key),
//            P = exp2(S - lse); column sums reduce within a lane and its partner
//            lane, the diagonals of each 32x32 block through a skewed LDS scratch
//   select   the k-th largest fp32 bit pattern by its value bins, digit by
//            digit, and an ordered compaction: all entries above it, then the
//            lowest-index ties.  With the top-p budget
//            (score_cover of Algorithm 1) each bin carries its count and its
//            summed mass, the select finds the value t at which the descending
//            cumulative mass reaches p of the list's total, and k follows from
//            the count and mass above t.
// The last 64 query rows form the last 64-row block exactly (N % 64 == 0), so
// tile j (keys 64 j .. 64 j + 63) holds offsets delta = 64 (nb - 1 - j) + r - c
// for in-block row r and key c.
#include "common.h"
#include "kernels.h"
#include "trace.h"
#include "tiles.h"

namespace msparse {

namespace {

constexpr int kChunkTiles = 32;   // most key tiles per workgroup (2048 keys)
constexpr int kCus = 256;
constexpr int kMaxShare = 4;      // query heads per workgroup of the K passes (two waves each)
constexpr float kLog2e = 1.4426950408889634f;

struct EstLayout {
    size_t part_max, part_sum, row_lse, bnd_part, sel_hist, sel_hmass, sel_cand, sel_above, sel_ncand, sel_eq,
        sel_state, bytes;
};

constexpr int kSliceLen = 16384;   // scores per selection slice
constexpr int kSelBins = 2048;     // value bins of a list's histogram (top 11 bits)
constexpr int kSelDigits = 3;      // of 11, 11 and 10 bits
// A list's threshold as far as its first digits decide it: the group of scores
// that share them, and what is left to find inside the group.
struct SelState {
    uint32_t prefix;   // the decided digits (after the last: the threshold score)
    uint32_t above;    // scores above the group
    uint32_t want;     // count select: scores of the group to take
    uint32_t mode;
    uint64_t rem;      // mass select: mass of the group to reach (2^-40 units)
};
// top-p lists start with both: the higher of the two thresholds holds, and the
// digit at which they part says which it is
constexpr uint32_t kModeMass = 1, kModeCount = 2, kModeBoth = 3;

// The query heads of a KV group are dealt evenly to workgroups of at most
// kMaxShare heads.
int32_t head_shares(int32_t G) { return (G + kMaxShare - 1) / kMaxShare; }
// Workgroups of pass 2 with shares of `nh` heads that run at a time: what its LDS
// leaves room for, at most four per CU (more wins nothing: the passes are bound
// by their VALU work then).  Four with one or two heads a share at head dim 64,
// three with one at 128 or three at 64, two otherwise.
int64_t pass_slots(int32_t d, int32_t nh) {
    const int64_t tiles = 2 * 2 * (d == 64 ? DmaTile<64, kRowPad>::kElems : DmaTile<128, kRowPad>::kElems);
    const int64_t lds = tiles + 4 * nh * (2 * 32 * 33 + 2 * 2 * kBlock + 2 * 4 * kBlock);
    return kCus * std::min<int64_t>(4, (160 * 1024) / lds);
}
// Key tiles per workgroup of the passes over K, a power of two from 2: the one
// with the least rounds of workgroups times (tiles + 1.5), what a workgroup
// takes before and after its serial walk being worth about 1.5 tiles, plus what
// the combine takes for the chunks (170 of them cost it as long as a tile costs
// the passes).  Both passes and the combine in us, by tiles, d 64 without GQA: 8
// heads x 32K 39 with 2, 33 with 4 (taken), 40 with 8; 16 x 64K 82, 79, 72 with
// 4, 8, 16 (taken), 103 with 32; 1 x 512K 78, 59, 67 with 4, 8 (taken), 16.
// d 128: 16 x 64K 129, 123, 134 with 4, 8 (taken), 16; 28 over 4 x 512K 829, 776,
// 753 with 8, 16, 32 (taken).  (With two workgroups per CU taken for every share,
// 16 x 64K at d 64 had 32 tiles, slower than 16 tiles for all grids.)
int32_t chunk_tiles_of(int64_t BK, int32_t G, int32_t nb, int32_t d) {
    const int32_t shares = head_shares(G);
    const int64_t slots = pass_slots(d, (G + shares - 1) / shares);
    int32_t best = 2;
    int64_t least = -1;
    for (int32_t t = 2; t <= kChunkTiles; t *= 2) {
        const int64_t chunks = (nb + t - 1) / t, wgs = BK * shares * chunks;
        const int64_t cost = (wgs + slots - 1) / slots * (2 * t + 3) + chunks / 85;   // half tiles
        if (least < 0 || cost < least) {
            least = cost;
            best = t;
        }
    }
    return best;
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

EstLayout est_layout(int64_t BH, int64_t BK, int32_t N, int32_t d) {
    const int64_t nb = N / kBlock;
    const int64_t ct = chunk_tiles_of(BK, int32_t(BH / BK), int32_t(nb), d), nchunk = (nb + ct - 1) / ct;
    EstLayout L{};
    size_t off = 0;
    L.part_max = off;
    off = align256(off + size_t(BH) * nchunk * kBlock * 4);
    L.part_sum = off;
    off = align256(off + size_t(BH) * nchunk * kBlock * 4);
    L.row_lse = off;
    off = align256(off + size_t(BH) * kBlock * 4);
    L.bnd_part = off;
    off = align256(off + size_t(BH) * nchunk * kBlock * 4);
    const int64_t NL = 2 * BH, ns = (N + kSliceLen - 1) / kSliceLen;
    L.sel_hist = off;
    off = align256(off + (ns > 1 ? size_t(NL) * kSelDigits * kSelBins * 4 : 0));
    L.sel_hmass = off;
    off = align256(off + (ns > 1 ? size_t(NL) * kSelDigits * kSelBins * 8 : 0));
    L.sel_cand = off;
    off = align256(off + (ns > 1 ? size_t(NL) * N * 4 : 0));
    L.sel_above = off;
    off = align256(off + size_t(NL) * ns * 4);
    L.sel_ncand = off;
    off = align256(off + size_t(NL) * ns * 4);
    L.sel_eq = off;
    off = align256(off + size_t(NL) * ns * 4);
    L.sel_state = off;
    off = align256(off + size_t(NL) * kSelDigits * sizeof(SelState));
    L.bytes = off;
    return L;
}

// ---------------------------------------------------------------- passes over K
// One workgroup per (batch, KV head, chunk of key tiles, share of at most four
// of the group's query heads) and two waves per head (query rows 0-31 and
// 32-63): each K tile is staged once for the share (direct global->LDS loads,
// double buffer), the shares of a chunk follow one another and find it in L2.
// A wave holds its 32 query rows as one MFMA operand (qreg); a 64-key tile is
// two 32-key halves.  Two workgroups of eight waves then share a CU, where one
// of fourteen or sixteen stood at its barriers alone (LDS and registers of
// pass 2 allow no second): pass 2 at 28 heads x 512K 522 -> 440 us, 32 x 128K
// (groups of four as before) 138 -> 124 us.
// Measured against it: the terms of one tile spread over the MFMAs of the next
// (600-640 us for pass 2 and 310-350 for pass 1, 128 registers and spills),
// two or four tiles per barrier (275-295 us for pass 1, 276 with one).

// (batch x KV head, chunk, share of the group's heads) of workgroup t:
// XCD-chunked, the shares of one chunk and then the chunks of one KV head
// adjacent.
__device__ __forceinline__ void group_chunk_of(int64_t t, int BK, int nchunk, int nshare, int& bk, int& chunk,
                                               int& share) {
    const int64_t u = xcd_chunk(t, int64_t(BK) * nchunk * nshare);
    share = int(u % nshare);
    const int64_t v = u / nshare;
    bk = int(v / nchunk);
    chunk = int(v % nchunk);
}

template <int D>
__device__ __forceinline__ void load_qlast(const EstArgs& a, int bh, int rb, int lane, u32x4* qreg) {
    const int h = lane >> 5, l32 = lane & 31;
    const uint16_t* qp = a.q + (int64_t(bh) * a.N + a.N - kBlock + 32 * rb + l32) * D;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) qreg[s] = *reinterpret_cast<const u32x4*>(qp + 16 * s + 8 * h);
}

// A copy of a lane-dependent value that the compiler can't look through: what
// a rare branch or a per-tile address computes from it stays there instead of
// being kept in registers over the whole loop.
__device__ __forceinline__ int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// pass 1: per-row (max, sum exp2) of the chunk's keys, log2 domain.
// S^T = K Q^T puts one query row per lane (keys in the accumulator).
template <int D, int NH>
__global__ void __launch_bounds__(128 * NH) est_stats_kernel(EstArgs a) {
    constexpr int KD = D / 16;
    constexpr int KE = DmaTile<D, kRowPad>::kElems;
    constexpr int NW = 2 * NH;
    __shared__ uint16_t kt[2][KE];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), rb = w & 1, hw = w >> 1;
    const int nb = a.N / kBlock, G = a.Hq / a.Hkv;
    int bk, chunk, g0;
    group_chunk_of(blockIdx.x, a.B * a.Hkv, a.nchunk, (G + NH - 1) / NH, bk, chunk, g0);
    const bool act = g0 * NH + hw < G;
    const int bh = (bk / a.Hkv) * a.Hq + (bk % a.Hkv) * G + (act ? g0 * NH + hw : 0);
    const uint16_t* __restrict__ kp = a.k + int64_t(bk) * a.N * D;
    const int j0 = chunk * a.chunk_tiles, j1 = min(nb, j0 + a.chunk_tiles);
    const float c2 = a.scale * kLog2e;
    auto load = [&](int buf, int j) {
        dma_rows<D, kRowPad, NW>(kt[buf], kp, ContiguousRows{int64_t(j) * kBlock}, w, opaque(lane));
    };
    u32x4 qreg[KD];
    load_qlast<D>(a, bh, rb, lane, qreg);
    float m = -INFINITY, l = 0.f;
    auto tile = [&](const uint16_t* cur, int j) {
        f32x16 acc[2] = {f32x16{}, f32x16{}};
#pragma unroll
        for (int s = 0; s < KD; ++s)
#pragma unroll
            for (int kh = 0; kh < 2; ++kh)
                acc[kh] = mfma32(dma_read16<D, kRowPad>(cur, 32 * kh + l32, h + 2 * s), qreg[s], acc[kh]);
        if (j == nb - 1) {   // keys after the row are masked (causal), only in the last tile
            keep_branch();
            const int lim = opaque(32 * rb + l32 - 4 * h);
#pragma unroll
            for (int kh = 0; kh < 2; ++kh)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (32 * kh + 8 * (i >> 2) + (i & 3) > lim) acc[kh][i] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[kh][i]);
        const float mn = fmaxf(m, mx * c2);
        if (mn != -INFINITY) {
            float sum = 0.f;
#pragma unroll
            for (int kh = 0; kh < 2; ++kh)
#pragma unroll
                for (int i = 0; i < 16; ++i) sum += fast_exp2(__builtin_fmaf(acc[kh][i], c2, -mn));
            l = (m == -INFINITY ? 0.f : l * fast_exp2(m - mn)) + sum;
            m = mn;
        }
    };
    load(0, j0);
    wait_vmem();
    __syncthreads();
    for (int j = j0, buf = 0; j < j1; ++j, buf ^= 1) {
        if (j + 1 < j1) load(buf ^ 1, j + 1);
        if (act) tile(kt[buf], j);
        wait_vmem();
        __syncthreads();
    }
    if (act) {   // the lane pair l, l ^ 32 holds one row
        const float mo = __shfl_xor(m, 32), lo = __shfl_xor(l, 32);
        const float mm = fmaxf(m, mo);
        const float ll = (m == -INFINITY ? 0.f : l * fast_exp2(m - mm)) + (mo == -INFINITY ? 0.f : lo * fast_exp2(mo - mm));
        if (h == 0) {
            const int64_t o = (int64_t(bh) * a.nchunk + chunk) * kBlock + 32 * rb + l32;
            a.part_max[o] = mm;
            a.part_sum[o] = ll;
        }
    }
}

// One workgroup per (head, 16 rows): 64 threads per row combine the chunk
// partials in a fixed order (per-thread strided runs, then the 64 threads'
// sums one after another).  Neighbouring threads take neighbouring rows, so
// each 64-byte piece of a chunk's partials is one access.  It also clears the
// selection's histograms for this call.
constexpr int kCombineRows = 16, kCombineSplit = 64;
__global__ void __launch_bounds__(kCombineRows * kCombineSplit) est_combine_kernel(EstArgs a) {
    __shared__ float pm_s[kCombineSplit][kCombineRows], ps_s[kCombineSplit][kCombineRows];
    __shared__ float pe_s[kCombineSplit][kCombineRows];
    constexpr int NT = kCombineRows * kCombineSplit;
    if (a.nslice > 1)
        for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < int64_t(2) * a.B * a.Hq * kSelDigits * kSelBins;
             i += int64_t(gridDim.x) * NT) {
            a.sel_hist[i] = 0u;
            if (a.p_v > 0.0) a.sel_hmass[i] = 0u;
        }
    const int bh = blockIdx.x / (kBlock / kCombineRows);
    const int rr = threadIdx.x % kCombineRows, j = threadIdx.x / kCombineRows;
    const int r = (blockIdx.x % (kBlock / kCombineRows)) * kCombineRows + rr;
    float M = -INFINITY;
    for (int c = j; c < a.nchunk; c += kCombineSplit)
        M = fmaxf(M, a.part_max[(int64_t(bh) * a.nchunk + c) * kBlock + r]);
    float S = 0.f;
    for (int c = j; c < a.nchunk; c += kCombineSplit) {
        const int64_t o = (int64_t(bh) * a.nchunk + c) * kBlock + r;
        const float pm = a.part_max[o];
        if (pm != -INFINITY) S += a.part_sum[o] * fast_exp2(pm - M);
    }
    pm_s[j][rr] = M;
    __syncthreads();
    float MM = -INFINITY;
#pragma unroll
    for (int t = 0; t < kCombineSplit; ++t) MM = fmaxf(MM, pm_s[t][rr]);
    ps_s[j][rr] = S;   // 0 without chunks
    pe_s[j][rr] = M != -INFINITY ? fast_exp2(M - MM) : 0.f;
    __syncthreads();
    if (j == 0) {
        float SS = 0.f;
#pragma unroll
        for (int t = 0; t < kCombineSplit; ++t) SS = __builtin_fmaf(ps_s[t][rr], pe_s[t][rr], SS);
        a.row_lse[bh * kBlock + r] = MM + fast_log2(SS);
    }
}

// Orders the LDS accesses of one wave around a wave-private scratch region.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// pass 2: P = exp2(S - lse) per tile (S = Q K^T, one key per lane), the
// vertical scores (column sums over the 64 rows) and the slash scores.
// Diagonal sums: each 32x32 block (rb, kh) of P goes to the wave's LDS
// scratch; lane e (< 63) sums the block's diagonal r - c = e - 31, which is
// diagonal t = 32 (rb - kh) + e + 32 of the tile (t = r - c + 63 over the
// tile's rows r and keys c).  The two waves of a head leave their column and
// diagonal partials in LDS; after a barrier the row-0 wave adds the columns
// and the row-1 wave the diagonals, in a fixed order, and they write the
// scores.  The slash scores are
//   s_score[64 D + e] = T_j[e + 63] + T_{j-1}[e - 1]   (D = nb - 1 - j)
// since the tile j holds offsets delta = 64 (nb - 1 - j) + r - c.  The lower
// part T_{j-1}[e - 1] of a chunk's first tile comes from the previous chunk,
// which leaves it in bnd_part; the selection's first kernel adds it
// (add_bounds).  One barrier per tile: the partials are added after it, from
// two LDS buffers, while other waves are in the next tile.
template <int D, int NH>
__global__ void __launch_bounds__(128 * NH) est_scores_kernel(EstArgs a) {
    constexpr int KD = D / 16;
    constexpr int KE = DmaTile<D, kRowPad>::kElems;
    constexpr int NW = 2 * NH;
    constexpr int SS = 33;   // scratch row stride (floats)
    __shared__ uint16_t kt[2][KE];
    __shared__ float scr[NW][32 * SS];
    // per head and tile (two in turn): column partials [rb][64], diagonal
    // partials A, B0, B1, C [64]
    __shared__ float colp[2][NH][2][kBlock], diagp[2][NH][4][kBlock];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), rb = w & 1, hw = w >> 1;
    const int nb = a.N / kBlock, G = a.Hq / a.Hkv;
    int bk, chunk, g0;
    group_chunk_of(blockIdx.x, a.B * a.Hkv, a.nchunk, (G + NH - 1) / NH, bk, chunk, g0);
    const bool act = g0 * NH + hw < G;
    const int bh = (bk / a.Hkv) * a.Hq + (bk % a.Hkv) * G + (act ? g0 * NH + hw : 0);
    const uint16_t* __restrict__ kp = a.k + int64_t(bk) * a.N * D;
    const int j0 = chunk * a.chunk_tiles, j1 = min(nb, j0 + a.chunk_tiles);
    const float c2 = a.scale * kLog2e;
    auto load = [&](int buf, int j) {
        dma_rows<D, kRowPad, NW>(kt[buf], kp, ContiguousRows{int64_t(j) * kBlock}, w, opaque(lane));
    };
    u32x4 qreg[KD];
    load_qlast<D>(a, bh, rb, lane, qreg);
    // the row lse of this lane's accumulator rows 8 q4 + 4 h + e (log2); rows
    // before the last L contribute nothing
    f32x4 lr[4];
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const int r = 32 * rb + 8 * q4 + 4 * h + e4;
            lr[q4][e4] = r >= kBlock - a.L ? a.row_lse[bh * kBlock + r] : INFINITY;
        }
    float* sc = scr[w];
    float* vs = a.v_score + int64_t(bh) * a.N;
    float* ss = a.s_score + int64_t(bh) * a.N;
    float tlow = 0.f;   // row-1 wave, lane e >= 1: T[e - 1] of the tile before
    // column and diagonal partials of tile j
    auto tile = [&](const uint16_t* cur, int j, int t) {
        const bool last = j == nb - 1;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
            f32x16 acc = f32x16{};
#pragma unroll
            for (int s = 0; s < KD; ++s)
                acc = mfma32(qreg[s], dma_read16<D, kRowPad>(cur, 32 * kh + l32, h + 2 * s), acc);
            // accumulator element i covers row 32 rb + 8 (i/4) + 4 h + i%4, key 32 kh + l32
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = fast_exp2(__builtin_fmaf(acc[i], c2, -lr[i >> 2][i & 3]));
            if (last) {   // causal mask of the last tile: key > row
                keep_branch();
                const int lim = opaque(32 * kh + l32 - 32 * rb - 4 * h);
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (lim > 8 * (i >> 2) + (i & 3)) acc[i] = 0.f;
            }
            // element (r, c) of the 32 x 32 block goes to scratch row r,
            // column (c - r) mod 32: column m then holds diagonal r - c = -m
            // in rows r < 32 - m and diagonal 32 - m in the rows below
            float cs = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int r = 8 * (i >> 2) + 4 * h + (i & 3);
                cs += acc[i];
                sc[r * SS + ((l32 - r) & 31)] = acc[i];
            }
            cs = half_swap_sum(cs);
            if (h == 0) colp[t][hw][rb][32 * kh + l32] = cs;
            wave_lds_sync();
            // lane (h, m) sums rows 16 h .. 16 h + 15 of column m
            float upper = 0.f, lower = 0.f;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int r = 16 * h + k;
                const float v = sc[r * SS + l32];
                const bool up = r < 32 - l32;
                upper += up ? v : 0.f;
                lower += up ? 0.f : v;
            }
            upper = half_swap_sum(upper);
            lower = half_swap_sum(lower);
            // diagonal r - c = e - 31 of the block: e = 31 - m from the upper
            // rows, e = 63 - m from the rest (e = 63 does not exist: 0)
            // block kind: rb < kh -> A (t = e), rb == kh -> B (t = e + 32), rb > kh -> C (t = e + 64)
            float* dpk = diagp[t][hw][rb < kh ? 0 : (rb > kh ? 3 : 1 + rb)];
            if (h == 0) {
                dpk[31 - l32] = upper;
                dpk[63 - l32] = l32 == 0 ? 0.f : lower;
            }
            wave_lds_sync();
        }
    };
    // adds the partials of tile j and writes its scores: the row-0 wave the
    // columns (rows 0-31 + rows 32-63), the row-1 wave the diagonals
    auto finish = [&](int j, int t) {
        const int e = opaque(lane);
        if (rb == 0) {
            vs[int64_t(j) * kBlock + e] = colp[t][hw][0][e] + colp[t][hw][1][e];
            return;
        }
        // the tile's diagonals T[x], x < 64, and T[64 + x], x < 63
        const float* dp = &diagp[t][hw][0][0];
        auto tlo = [&](int x) {
            return dp[x] + (x >= 32 ? dp[kBlock + x - 32] + dp[2 * kBlock + x - 32] : 0.f);
        };
        auto thi = [&](int x) {
            return (x < 32 ? dp[kBlock + x + 32] + dp[2 * kBlock + x + 32] : 0.f) + dp[3 * kBlock + x];
        };
        // s_score of block-diagonal D = nb - 1 - j, offset e: T_j[e + 63] + T_{j-1}[e - 1]
        const float up = e == 0 ? tlo(63) : thi(e - 1);
        ss[int64_t(nb - 1 - j) * kBlock + e] = (e >= 1 && j > j0) ? up + tlow : up;
        tlow = e >= 1 ? tlo(e - 1) : 0.f;
    };
    load(0, j0);
    wait_vmem();
    __syncthreads();
    for (int j = j0, buf = 0; j < j1; ++j, buf ^= 1) {
        if (j + 1 < j1) load(buf ^ 1, j + 1);
        if (act) tile(kt[buf], j, buf);
        wait_vmem();
        __syncthreads();   // tile j + 1's keys are there, tile j's partials complete
        if (act) finish(j, buf);
    }
    // the lower part of the chunk's last tile belongs to the next chunk's first block-diagonal
    if (act && rb == 1 && j1 < nb) a.bnd_part[(int64_t(bh) * a.nchunk + chunk) * kBlock + lane] = tlow;
}

// ---------------------------------------------------------------- top-k / top-p
// Selection over the 2 B Hq score lists (vertical lists first), each cut into
// slices of kSliceLen scores.  Scores are >= 0, so fp32 bit patterns order
// like values.  A list of one slice is decided and written by one workgroup
// (sel_small_kernel); longer lists take five launches over (list, slice):
//   hist     histogram of the top 11 bits (value bins of a quarter octave), added
//            into the list's (integer sums: order-free)
//   split    finds the bin with the threshold from the list's histogram, counts
//            the slice's scores above it, collects those inside it (the
//            candidates) and adds their next 11 bits to the list's second
//            histogram
//   digit    finds the bin there, and adds the last 10 bits of the candidates
//            inside it to the third
//   count    finds the threshold, and counts the slice's scores above and at it
//   write    the selected indices at the offset that the counts of the slices
//            before give, in index order, lowest-index ties first.
// With a top-p fraction every bin also carries its mass, and the bin where the
// descending cumulative mass reaches p of the total takes the place of the
// k-th score's, unless the cap is reached in a higher bin (then the cap-th
// score decides; while both lie in the same bin, the next digit decides).
// How many scores are candidates depends on the scores: a few percent of a list
// with a clear pattern, all of one that is flat (q = 0, padding).  No workgroup
// therefore takes more than a slice.  All launches of the selection, in us, with
// the last two digits and the counts by one workgroup per list -> by the slices:
// a flat list of 512K scores 980 -> 66 (top-p 3600 -> 100), 56 of them 1154 -> 232
// (3865 -> 425); with a pattern 28 x 512K 138 -> 139, top-p 32 x 128K 136 -> 105,
// 16 x 32K 93 -> 52.
constexpr int kSelThreads = 512;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelIters = kSliceLen / (4 * kSelThreads);   // 16-byte loads per thread
constexpr int kSelCopies = 4;    // LDS histogram copies (a list's scores share few bins)

// Masses in fixed point: a score x (0 <= x <= L <= 64) counts floor(x 2^40), so
// every sum of masses is an exact integer (below 2^47) whatever the order of
// the additions, and the budget is deterministic.
__device__ __forceinline__ uint64_t mass_fx(uint32_t bits) {
    const int e = int(bits >> 23) & 255;
    const uint64_t m = (bits & 0x7fffffu) | (e ? 0x800000u : 0u);   // x = m 2^(e - 150) (e = 0 as e = 1)
    if (e == 255) return 0;
    const int sh = (e ? e : 1) - 110;
    return sh >= 0 ? m << min(sh, 40) : (sh > -24 ? m >> -sh : 0);
}

__device__ __forceinline__ uint64_t wave_scan_u64(uint64_t v) {   // inclusive
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(v, o);
        if (lane >= o) v += y;
    }
    return v;
}

// Exclusive prefix over the workgroup's threads and the total (tmp: 17 words).
template <int T>
__device__ __forceinline__ uint64_t block_scan_u64(uint64_t v, uint64_t* tmp, uint64_t& total) {
    const uint64_t x = wave_scan_u64(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();   // tmp may still be read from the call before
    if (lane == 63) tmp[w] = x;
    __syncthreads();
    uint64_t base = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < T / 64; ++i) {
        if (i < w) base += tmp[i];
        total += tmp[i];
    }
    return base + x - v;
}

// The highest bin at which the descending cumulative `val` reaches `want`
// (1 <= want <= total): its number, and the cnt / mass of the bins above it.
// `val` is mass when BY_MASS, else cnt.  All threads get the result.
struct Pick {
    uint32_t bin, above;
    uint64_t mass_above;
};
template <int T, bool MASS, bool BY_MASS>
__device__ __forceinline__ Pick pick_bin(const uint32_t* cnt, const uint64_t* mass, uint64_t want, uint64_t* tmp,
                                         Pick* res) {
    constexpr int PER = kSelBins / T;
    const int top = kSelBins - 1 - int(threadIdx.x) * PER;   // this thread's bins top, top - 1, ...
    uint64_t c = 0, m = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c += cnt[top - i];
        if (MASS) m += mass[top - i];
    }
    uint64_t tc, tm = 0, bc = block_scan_u64<T>(c, tmp, tc), bm = 0;
    if (MASS) bm = block_scan_u64<T>(m, tmp, tm);
    const uint64_t before = BY_MASS ? bm : bc, mine = BY_MASS ? m : c;
    if (before < want && want <= before + mine) {   // exactly one thread
        uint64_t run = before;
        for (int i = 0; i < PER; ++i) {
            const uint64_t x = BY_MASS ? mass[top - i] : uint64_t(cnt[top - i]);
            if (run + x >= want) {
                *res = Pick{uint32_t(top - i), uint32_t(bc), bm};
                break;
            }
            run += x;
            bc += cnt[top - i];
            if (MASS) bm += mass[top - i];
        }
    }
    __syncthreads();
    const Pick r = *res;
    __syncthreads();
    return r;
}

__device__ __forceinline__ void list_of(const EstArgs& a, int list, const u32x4*& sc4, int32_t*& out, int& cap,
                                        double& p) {
    const int BH = a.B * a.Hq;
    const bool is_v = list < BH;
    const int64_t l = is_v ? list : list - BH;
    sc4 = reinterpret_cast<const u32x4*>((is_v ? a.v_score : a.s_score) + l * a.N);
    cap = is_v ? a.k_v : a.k_s;
    p = is_v ? a.p_v : a.p_s;
    out = (is_v ? a.v_idx : a.s_idx) + l * cap;
}

// One slice of a list in registers: wave w owns a run of `per` 256-score
// groups, lane l the scores 4 l .. 4 l + 3 of each.
struct Slice {
    int i0;     // this lane's first score index
    int n;      // groups of this wave
    int hi;     // end of the slice
    u32x4 v[kSelIters];
    __device__ __forceinline__ bool in(int it) const { return it < n && i0 + 256 * it < hi; }
};

__device__ __forceinline__ void load_slice(const EstArgs& a, const u32x4* sc4, int slice, Slice& s) {
    const int lo = slice * kSliceLen;
    s.hi = min(a.N, lo + kSliceLen);
    const int groups = (s.hi - lo + 255) / 256, per = (groups + kSelWaves - 1) / kSelWaves;
    const int w = threadIdx.x >> 6;
    s.i0 = lo + 256 * per * w + 4 * int(threadIdx.x & 63);
    s.n = per;
#pragma unroll
    for (int it = 0; it < kSelIters; ++it) s.v[it] = s.in(it) ? sc4[(s.i0 + 256 * it) >> 2] : u32x4{0u, 0u, 0u, 0u};
}

// The slash scores of the first block-diagonal of every key chunk after the
// first still miss the lower part that the previous chunk left: added (up +
// low, as inside a chunk) and stored by the first kernel that reads them.
__device__ __forceinline__ void add_bounds(const EstArgs& a, int list, Slice& s) {
    const int bh = list - a.B * a.Hq;
    if (bh < 0 || a.nchunk < 2) return;
    const int nb = a.N / kBlock;
#pragma unroll
    for (int it = 0; it < kSelIters; ++it) {
        const int i = s.i0 + 256 * it, j = nb - 1 - (i >> 6);
        if (!s.in(it) || j == 0 || j % a.chunk_tiles != 0) continue;
        const f32x4 low = *reinterpret_cast<const f32x4*>(
            a.bnd_part + (int64_t(bh) * a.nchunk + j / a.chunk_tiles - 1) * kBlock + (i & 63));
        f32x4 x = __builtin_bit_cast(f32x4, s.v[it]);
        x += low;
        s.v[it] = __builtin_bit_cast(u32x4, x);
        *reinterpret_cast<f32x4*>(a.s_score + int64_t(bh) * a.N + i) = x;
    }
}

// One digit of a radix select over the 32 bits (11, 11 and 10 of them).
struct Digit {
    int shift;
    uint32_t width;   // digit mask, unshifted
};
__device__ __forceinline__ Digit digit_of(int d) {
    return d == 0 ? Digit{21, 2047u} : (d == 1 ? Digit{10, 2047u} : Digit{0, 1023u});
}

template <bool MASS>
__device__ __forceinline__ void add_score(uint32_t x, Digit d, uint32_t* hist, uint64_t* mass) {
    const uint32_t b = (x >> d.shift) & d.width;
    atomicAdd(&hist[b], 1u);
    if (MASS) atomicAdd(reinterpret_cast<unsigned long long*>(&mass[b]), (unsigned long long)mass_fx(x));
}

// The same for the lanes with `on` of a whole wave, into one histogram: scores
// that share a bin, as those of a flat list do, are added once.
template <bool MASS>
__device__ __forceinline__ void add_scores(uint32_t x, bool on, Digit d, uint32_t* hist, uint64_t* mass) {
    const uint64_t act = __ballot(on);
    if (act == 0) return;
    const int first = __builtin_ctzll(act);
    const uint32_t b = (x >> d.shift) & d.width, b0 = uint32_t(__shfl(int(b), first));
    if (__ballot(on && b == b0) != act) {
        if (on) add_score<MASS>(x, d, hist, mass);
        return;
    }
    uint64_t m = MASS && on ? mass_fx(x) : 0;
    if (MASS)
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) m += __shfl_xor(m, o);
    if (int(threadIdx.x & 63) == first) {
        atomicAdd(&hist[b0], uint32_t(__popcll(act)));
        if (MASS) atomicAdd(reinterpret_cast<unsigned long long*>(&mass[b0]), (unsigned long long)m);
    }
}

// Histograms in LDS: COPIES of kSelBins counts (and masses), the lanes dealt
// to them so that the few bins which a list's scores share serialise less; the
// pad puts a bin's copies on different banks.
template <bool MASS, int COPIES>
struct Hist {
    static constexpr int kStride = kSelBins + 1;
    uint32_t c[COPIES * kStride];
    uint64_t m[MASS ? COPIES * kStride : 1];
    template <int T>
    __device__ __forceinline__ void clear() {
        for (int i = threadIdx.x; i < COPIES * kStride; i += T) {
            c[i] = 0u;
            if (MASS) m[i] = 0u;
        }
        __syncthreads();
    }
    // sums the copies into the first
    template <int T>
    __device__ __forceinline__ void fold() {
        __syncthreads();
        if (COPIES > 1) {
            for (int b = threadIdx.x; b < kSelBins; b += T) {
#pragma unroll
                for (int i = 1; i < COPIES; ++i) {
                    c[b] += c[i * kStride + b];
                    if (MASS) m[b] += m[i * kStride + b];
                }
            }
            __syncthreads();
        }
    }
    __device__ __forceinline__ void add(uint32_t x, Digit d) {
        const int o = COPIES > 1 ? int(threadIdx.x % COPIES) * kStride : 0;
        add_score<MASS>(x, d, c + o, m + (MASS ? o : 0));
    }
};

template <class F>
__device__ __forceinline__ void for_each_score(const Slice& s, F f) {
#pragma unroll
    for (int it = 0; it < kSelIters; ++it) {
        if (!s.in(it)) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) f(s.v[it][e]);
    }
}

// Writes the slice's selected indices from output slot `off` on: scores above
// `thr`, and the ties from the `eq_before`-th of the list to the `krem`-th.
__device__ __forceinline__ void write_slice(const Slice& s, uint32_t thr, uint32_t krem, int64_t off,
                                            int64_t eq_before, int32_t* out, uint32_t (*sh)[2]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int it = 0; it < kSelIters; ++it)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            gt += __popcll(__ballot(s.in(it) && s.v[it][e] > thr));
            eq += __popcll(__ballot(s.in(it) && s.v[it][e] == thr));
        }
    if (lane == 0) {
        sh[w][0] = gt;
        sh[w][1] = eq;
    }
    __syncthreads();
    for (int i = 0; i < w; ++i) {
        off += sh[i][0] + min<int64_t>(sh[i][1], max<int64_t>(0, int64_t(krem) - eq_before));
        eq_before += sh[i][1];
    }
#pragma unroll
    for (int it = 0; it < kSelIters; ++it) {
        uint64_t bt[4];
        bool take[4];
        uint64_t any_eq = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            take[e] = s.in(it) && s.v[it][e] > thr;
            any_eq |= __ballot(s.in(it) && s.v[it][e] == thr);
        }
        if (any_eq) {   // rare: rank this group's ties in index order
            uint32_t r = 0, n = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t m = __ballot(s.in(it) && s.v[it][e] == thr);
                r += __popcll(m & below);
                n += __popcll(m);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (s.in(it) && s.v[it][e] == thr) {
                    take[e] = eq_before + r < int64_t(krem);
                    ++r;
                }
            eq_before += n;
        }
        uint32_t r = 0, n = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bt[e] = __ballot(take[e]);
            r += __popcll(bt[e] & below);
            n += __popcll(bt[e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (take[e]) out[off + r++] = s.i0 + 256 * it + e;
        off += n;
    }
}

// the budget of a mass select whose threshold score is `t`: `above` entries
// above it, `ties` equal to it, `rem` of mass still to reach
__device__ __forceinline__ uint64_t mass_budget(uint32_t t, uint32_t above, uint32_t ties, uint64_t rem) {
    const uint64_t qt = mass_fx(t);   // every score equal to t adds mass_fx(t)
    const uint64_t need = qt ? (rem + qt - 1) / qt : uint64_t(ties);
    return uint64_t(above) + min<uint64_t>(need, ties);
}

// Radix select over the scores of sel_small_kernel: `scan(f)` calls f(x) for
// this thread's scores.  `want` is a count (or, BY_MASS, a mass) to reach from
// the top; returns the threshold score, what of `want` is left for the scores
// equal to it, their number (ties) and how many are above it.
template <int T, bool MASS, bool BY_MASS, int COPIES, class Scan>
__device__ __forceinline__ uint32_t radix_select(uint64_t& want, uint32_t& above, uint32_t& ties,
                                                 Hist<MASS, COPIES>& h, uint64_t* tmp, Pick* res, Scan scan) {
    uint32_t prefix = 0, mask = 0;
    above = 0;
    for (int d = 0; d < kSelDigits; ++d) {
        const Digit dg = digit_of(d);
        h.template clear<T>();
        scan([&](uint32_t x) {
            if ((x & mask) == prefix) h.add(x, dg);
        });
        h.template fold<T>();
        const Pick p = pick_bin<T, MASS, BY_MASS>(h.c, h.m, want, tmp, res);
        prefix |= p.bin << dg.shift;
        mask |= dg.width << dg.shift;
        above += p.above;
        want -= BY_MASS ? p.mass_above : uint64_t(p.above);
        ties = h.c[p.bin];
        __syncthreads();   // before the next digit clears the bins
    }
    return prefix;
}

// -1 in the unused slots of a top-p list (every `parts`-th run of T from the
// part-th on), and its budget
template <int T>
__device__ __forceinline__ void finish_topp(const EstArgs& a, int list, uint32_t k, int cap, int32_t* out, int part,
                                            int parts) {
    const int BH = a.B * a.Hq;
    for (int i = int(k) + part * T + threadIdx.x; i < cap; i += parts * T) out[i] = -1;
    if (part == 0 && threadIdx.x == 0) (list < BH ? a.v_cnt + list : a.s_cnt + (list - BH))[0] = int32_t(k);
}

// A list of one slice, decided and written by one workgroup.
template <bool MASS>
__global__ void __launch_bounds__(kSelThreads) sel_small_kernel(EstArgs a) {
    __shared__ Hist<MASS, kSelCopies> h;
    __shared__ uint64_t tmp[17];
    __shared__ Pick res;
    __shared__ uint32_t sh[kSelWaves][2];
    const int list = blockIdx.x;
    const u32x4* sc4;
    int32_t* out;
    int cap;
    double p;
    list_of(a, list, sc4, out, cap, p);
    Slice s;
    load_slice(a, sc4, 0, s);
    add_bounds(a, list, s);
    auto scan = [&](auto f) { for_each_score(s, f); };
    uint32_t thr = 0, above = 0, ties = 0, k = uint32_t(cap);
    uint64_t want = uint64_t(cap);
    bool by_count = true;
    if constexpr (MASS) {
        uint64_t m = 0, total;
        scan([&](uint32_t x) { m += mass_fx(x); });
        block_scan_u64<kSelThreads>(m, tmp, total);
        if (total == 0) {   // no mass at all: one entry reaches p of it
            want = 1;
            k = 1;
        } else {
            uint64_t rem = uint64_t(ceil(p * double(total)));
            thr = radix_select<kSelThreads, true, true, kSelCopies>(rem, above, ties, h, tmp, &res, scan);
            const uint64_t kk = mass_budget(thr, above, ties, rem);
            by_count = kk > uint64_t(cap);   // capped: the cap-th largest decides
            if (!by_count) k = uint32_t(kk);
        }
    }
    if (by_count) thr = radix_select<kSelThreads, MASS, false, kSelCopies>(want, above, ties, h, tmp, &res, scan);
    write_slice(s, thr, k - above, 0, 0, out, sh);
    if (MASS) finish_topp<kSelThreads>(a, list, k, cap, out, 0, 1);
}

// The list's histogram of digit `d`.
__device__ __forceinline__ uint32_t* list_hist(const EstArgs& a, int list, int d) {
    return a.sel_hist + (int64_t(list) * kSelDigits + d) * kSelBins;
}
__device__ __forceinline__ uint64_t* list_hmass(const EstArgs& a, int list, int d) {
    return a.sel_hmass + (int64_t(list) * kSelDigits + d) * kSelBins;
}

// Adds a slice's histogram of digit `d` into the list's.
template <bool MASS>
__device__ __forceinline__ void add_to_list(const EstArgs& a, int list, int d, const uint32_t* c, const uint64_t* m) {
    uint32_t* gc = list_hist(a, list, d);
    uint64_t* gm = list_hmass(a, list, d);
    for (int b = threadIdx.x; b < kSelBins; b += kSelThreads) {
        if (c[b] == 0) continue;
        atomicAdd(&gc[b], c[b]);
        if (MASS) atomicAdd(reinterpret_cast<unsigned long long*>(&gm[b]), (unsigned long long)m[b]);
    }
}

// What a list is asked for, before its first digit: `cap` scores, or with a
// top-p fraction the mass p of the total (no mass at all: one score reaches it).
template <bool MASS>
__device__ __forceinline__ SelState select_start(const EstArgs& a, int list, int cap, double p, uint64_t* tmp) {
    SelState st{0u, 0u, uint32_t(cap), kModeCount, 0u};
    if constexpr (MASS) {
        const uint64_t* hm = list_hmass(a, list, 0);
        uint64_t m = 0, total;
        for (int b = threadIdx.x; b < kSelBins; b += kSelThreads) m += hm[b];
        block_scan_u64<kSelThreads>(m, tmp, total);
        if (total == 0) {
            st.want = 1;
        } else {
            st.mode = kModeBoth;
            st.rem = uint64_t(ceil(p * double(total)));
        }
    }
    return st;
}

// The threshold's bin in the list's histogram of digit `d` (every workgroup of
// the list takes the same decision); `ties` receives the scores in the bin.
template <bool MASS>
__device__ __forceinline__ void select_digit(const EstArgs& a, int list, int d, SelState& st, uint32_t& ties,
                                             uint64_t* tmp, Pick* res) {
    const uint32_t* hc = list_hist(a, list, d);
    const uint64_t* hm = list_hmass(a, list, d);
    Pick p{};
    if (!MASS || st.mode == kModeCount) {
        p = pick_bin<kSelThreads, MASS, false>(hc, hm, st.want, tmp, res);
    } else {
        p = pick_bin<kSelThreads, MASS, true>(hc, hm, st.rem, tmp, res);
        if (st.mode == kModeBoth) {
            const Pick pc = pick_bin<kSelThreads, MASS, false>(hc, hm, st.want, tmp, res);
            if (p.bin > pc.bin) st.mode = kModeMass;
            if (p.bin < pc.bin) {
                st.mode = kModeCount;
                p = pc;
            }
        }
    }
    st.prefix |= p.bin << digit_of(d).shift;
    st.above += p.above;
    if (st.mode & kModeCount) st.want -= p.above;
    if (st.mode & kModeMass) st.rem -= p.mass_above;
    ties = hc[p.bin];
}

// The list's state after digit `d` (written by its first slice's workgroup, read
// by the launches after).
__device__ __forceinline__ SelState& list_state(const EstArgs& a, int list, int d) {
    return reinterpret_cast<SelState*>(a.sel_state)[int64_t(list) * kSelDigits + d];
}

template <bool MASS>
__global__ void __launch_bounds__(kSelThreads) sel_hist_kernel(EstArgs a) {
    __shared__ Hist<MASS, kSelCopies> h;
    const int list = blockIdx.x / a.nslice, slice = blockIdx.x % a.nslice;
    const u32x4* sc4;
    int32_t* out;
    int cap;
    double p;
    list_of(a, list, sc4, out, cap, p);
    Slice s;
    load_slice(a, sc4, slice, s);
    add_bounds(a, list, s);
    h.template clear<kSelThreads>();
    for_each_score(s, [&](uint32_t x) { h.add(x, digit_of(0)); });
    h.template fold<kSelThreads>();
    add_to_list<MASS>(a, list, 0, h.c, h.m);
}

template <bool MASS>
__global__ void __launch_bounds__(kSelThreads) sel_split_kernel(EstArgs a) {
    __shared__ Hist<MASS, 1> h;
    __shared__ uint64_t tmp[17];
    __shared__ Pick res;
    __shared__ uint32_t nabove, ncand;
    const int list = blockIdx.x / a.nslice, slice = blockIdx.x % a.nslice;
    const u32x4* sc4;
    int32_t* out;
    int cap;
    double p;
    list_of(a, list, sc4, out, cap, p);
    Slice s;
    load_slice(a, sc4, slice, s);   // in flight while the bin is found
    if (threadIdx.x == 0) nabove = ncand = 0u;
    h.template clear<kSelThreads>();
    SelState st = select_start<MASS>(a, list, cap, p, tmp);
    uint32_t ties;
    select_digit<MASS>(a, list, 0, st, ties, tmp, &res);
    if (slice == 0 && threadIdx.x == 0) list_state(a, list, 0) = st;
    // candidates go to the slice's own part of the buffer, in any order
    uint32_t* cand = a.sel_cand + int64_t(list) * a.N + int64_t(slice) * kSliceLen;
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t bin = st.prefix >> 21;
    uint32_t na = 0;
#pragma unroll
    for (int it = 0; it < kSelIters; ++it) {
        const bool in = s.in(it);
        uint64_t b[4];
        uint32_t n = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t x = s.v[it][e] >> 21;
            na += __popcll(__ballot(in && x > bin));
            b[e] = __ballot(in && x == bin);
            n += __popcll(b[e]);
        }
        if (n == 0) continue;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&ncand, n);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool on = (b[e] >> lane) & 1ull;
            if (on) cand[base + __popcll(b[e] & below)] = s.v[it][e];
            base += __popcll(b[e]);
            add_scores<MASS>(s.v[it][e], on, digit_of(1), h.c, h.m);
        }
    }
    if (lane == 0) atomicAdd(&nabove, na);
    __syncthreads();
    if (threadIdx.x == 0) {
        a.sel_above[int64_t(list) * a.nslice + slice] = nabove;
        a.sel_ncand[int64_t(list) * a.nslice + slice] = ncand;
    }
    add_to_list<MASS>(a, list, 1, h.c, h.m);
}

// f(x, on) for the slice's candidates, by whole waves
template <class F>
__device__ __forceinline__ void for_each_candidate(const EstArgs& a, int list, int slice, F f) {
    const uint32_t* cand = a.sel_cand + int64_t(list) * a.N + int64_t(slice) * kSliceLen;
    const int n = int(a.sel_ncand[int64_t(list) * a.nslice + slice]);
#pragma unroll 4
    for (int i0 = 0; i0 < n; i0 += kSelThreads) {
        const int i = i0 + int(threadIdx.x);
        f(i < n ? cand[i] : 0u, i < n);
    }
}

template <bool MASS>
__global__ void __launch_bounds__(kSelThreads) sel_digit_kernel(EstArgs a) {
    __shared__ Hist<MASS, 1> h;
    __shared__ uint64_t tmp[17];
    __shared__ Pick res;
    const int list = blockIdx.x / a.nslice, slice = blockIdx.x % a.nslice;
    SelState st = list_state(a, list, 0);
    uint32_t ties;
    h.template clear<kSelThreads>();
    select_digit<MASS>(a, list, 1, st, ties, tmp, &res);
    if (slice == 0 && threadIdx.x == 0) list_state(a, list, 1) = st;
    for_each_candidate(a, list, slice, [&](uint32_t x, bool on) {
        add_scores<MASS>(x, on && x >> 10 == st.prefix >> 10, digit_of(2), h.c, h.m);
    });
    __syncthreads();
    add_to_list<MASS>(a, list, 2, h.c, h.m);
}

// Leaves the slice's scores above the threshold (sel_above) and at it (sel_eq).
template <bool MASS>
__global__ void __launch_bounds__(kSelThreads) sel_count_kernel(EstArgs a) {
    __shared__ uint64_t tmp[17];
    __shared__ Pick res;
    const int list = blockIdx.x / a.nslice, slice = blockIdx.x % a.nslice;
    SelState st = list_state(a, list, 1);
    uint32_t ties;
    select_digit<MASS>(a, list, 2, st, ties, tmp, &res);
    const u32x4* sc4;
    int32_t* out;
    int cap;
    double p;
    list_of(a, list, sc4, out, cap, p);
    if (MASS && (st.mode & kModeMass)) {
        const uint64_t k = mass_budget(st.prefix, st.above, ties, st.rem);
        if (st.mode == kModeMass || k <= uint64_t(cap)) st.want = uint32_t(k) - st.above;
    }
    if (slice == 0 && threadIdx.x == 0) list_state(a, list, 2) = st;
    uint64_t n = 0, total;   // above: low half, ties: high half
    for_each_candidate(a, list, slice, [&](uint32_t x, bool on) {
        n += (on && x > st.prefix ? 1ull : 0ull) + (on && x == st.prefix ? 1ull << 32 : 0ull);
    });
    block_scan_u64<kSelThreads>(n, tmp, total);
    if (threadIdx.x == 0) {
        a.sel_above[int64_t(list) * a.nslice + slice] += uint32_t(total);
        a.sel_eq[int64_t(list) * a.nslice + slice] = uint32_t(total >> 32);
    }
    if (MASS) finish_topp<kSelThreads>(a, list, st.above + st.want, cap, out, slice, a.nslice);
}

__global__ void __launch_bounds__(kSelThreads) sel_write_kernel(EstArgs a) {
    __shared__ uint32_t sh[kSelWaves][2];
    const int list = blockIdx.x / a.nslice, slice = blockIdx.x % a.nslice;
    const u32x4* sc4;
    int32_t* out;
    int cap;
    double p;
    list_of(a, list, sc4, out, cap, p);
    Slice s;
    load_slice(a, sc4, slice, s);
    const SelState st = list_state(a, list, 2);
    // scores above the threshold and at it in the slices before (every wave for itself)
    uint64_t gt = 0, eq = 0;
    for (int i = threadIdx.x & 63; i < slice; i += 64) {
        gt += a.sel_above[int64_t(list) * a.nslice + i];
        eq += a.sel_eq[int64_t(list) * a.nslice + i];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        gt += __shfl_xor(gt, o);
        eq += __shfl_xor(eq, o);
    }
    write_slice(s, st.prefix, st.want, int64_t(gt + min<uint64_t>(eq, st.want)), int64_t(eq), out, sh);
}

template <bool MASS>
hipError_t launch_select(const EstArgs& a, hipStream_t s) {
    const int NL = 2 * a.B * a.Hq;
    const dim3 lists(NL), slices(unsigned(NL) * a.nslice);
    if (a.nslice == 1) {
        TraceScope _t("est_select", s);
        hipLaunchKernelGGL(sel_small_kernel<MASS>, lists, dim3(kSelThreads), 0, s, a);
        return hipGetLastError();
    }
    { TraceScope _t("est_select", s); hipLaunchKernelGGL(sel_hist_kernel<MASS>, slices, dim3(kSelThreads), 0, s, a); }
    { TraceScope _t("est_select", s); hipLaunchKernelGGL(sel_split_kernel<MASS>, slices, dim3(kSelThreads), 0, s, a); }
    { TraceScope _t("est_select", s); hipLaunchKernelGGL(sel_digit_kernel<MASS>, slices, dim3(kSelThreads), 0, s, a); }
    { TraceScope _t("est_select", s); hipLaunchKernelGGL(sel_count_kernel<MASS>, slices, dim3(kSelThreads), 0, s, a); }
    { TraceScope _t("est_select", s); hipLaunchKernelGGL(sel_write_kernel, slices, dim3(kSelThreads), 0, s, a); }
    return hipGetLastError();
}

template <int D, int NW>
hipError_t launch_passes(const EstArgs& a, hipStream_t s) {
    const int BH = a.B * a.Hq;
    const int G = a.Hq / a.Hkv;
    const unsigned grid = unsigned(a.B * a.Hkv * a.nchunk * ((G + NW - 1) / NW));
    { TraceScope _t("est_pass1", s); hipLaunchKernelGGL((est_stats_kernel<D, NW>), dim3(grid), dim3(128 * NW), 0, s, a); }
    { TraceScope _t("est_combine", s); hipLaunchKernelGGL(est_combine_kernel, dim3(BH * (kBlock / kCombineRows)), dim3(kCombineRows * kCombineSplit), 0, s, a); }
    { TraceScope _t("est_pass2", s); hipLaunchKernelGGL((est_scores_kernel<D, NW>), dim3(grid), dim3(128 * NW), 0, s, a); }
    return hipGetLastError();
}

template <int D>
hipError_t launch_d(const EstArgs& a, hipStream_t s) {
    hipError_t e;
    const int G = a.Hq / a.Hkv, shares = head_shares(G);
    switch ((G + shares - 1) / shares) {   // two waves per query head of a share
        case 1: e = launch_passes<D, 1>(a, s); break;
        case 2: e = launch_passes<D, 2>(a, s); break;
        case 3: e = launch_passes<D, 3>(a, s); break;
        default: e = launch_passes<D, 4>(a, s); break;
    }
    if (e != hipSuccess) return e;
    return a.p_v > 0.0 ? launch_select<true>(a, s) : launch_select<false>(a, s);
}

}  // namespace

size_t est_workspace_bytes(int32_t B, int32_t Hq, int32_t Hkv, int32_t N, int32_t d) {
    return est_layout(int64_t(B) * Hq, int64_t(B) * Hkv, N, d).bytes;
}

void est_carve(EstArgs& a, char* base) {
    const EstLayout L = est_layout(int64_t(a.B) * a.Hq, int64_t(a.B) * a.Hkv, a.N, a.d);
    a.chunk_tiles = chunk_tiles_of(int64_t(a.B) * a.Hkv, a.Hq / a.Hkv, a.N / kBlock, a.d);
    a.nchunk = (a.N / kBlock + a.chunk_tiles - 1) / a.chunk_tiles;
    a.part_max = reinterpret_cast<float*>(base + L.part_max);
    a.part_sum = reinterpret_cast<float*>(base + L.part_sum);
    a.row_lse = reinterpret_cast<float*>(base + L.row_lse);
    a.bnd_part = reinterpret_cast<float*>(base + L.bnd_part);
    a.nslice = (a.N + kSliceLen - 1) / kSliceLen;
    a.sel_hist = reinterpret_cast<uint32_t*>(base + L.sel_hist);
    a.sel_hmass = reinterpret_cast<uint64_t*>(base + L.sel_hmass);
    a.sel_cand = reinterpret_cast<uint32_t*>(base + L.sel_cand);
    a.sel_above = reinterpret_cast<uint32_t*>(base + L.sel_above);
    a.sel_ncand = reinterpret_cast<uint32_t*>(base + L.sel_ncand);
    a.sel_eq = reinterpret_cast<uint32_t*>(base + L.sel_eq);
    a.sel_state = base + L.sel_state;
}

hipError_t launch_estimate(const EstArgs& a, hipStream_t s) {
    return a.d == 128 ? launch_d<128>(a, s) : launch_d<64>(a, s);
}

}  // namespace msparse
