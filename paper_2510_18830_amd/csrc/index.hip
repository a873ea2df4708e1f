// Sparse index construction on the GPU (Section 4.1 (ii); convert_index of
// Algorithms 1 and 2).
//
// Each selected slash offset delta is executed as the 64 x 64 block-diagonals
// floor(delta/64) and ceil(delta/64) (the set D); query block i gets the key
// blocks i - x (x in D, x <= i) and the verticals v <= 64 i + 63 that lie in a
// block-diagonal outside D.  A ring step keeps only the keys of its KV shard,
// in that shard's local numbering.
//
// Three launches, all deterministic (no atomics decide an output position):
//   prep  one workgroup per head: vertical bitmap -> unique ascending list of
//         the shard's verticals, slash offsets -> D bitset -> ascending list;
//   count one workgroup per chunk of query or key blocks of a head: the blocks'
//         list lengths, prefix-summed inside the chunk;
//   fill  the same chunks: offsets (the chunk totals before it summed again, or
//         by a scan launch in between when there are many) and entries, in
//         order by closed forms or wave ballots.
// The ring workload matrix (msparse_ring_work) reuses prep and counts, per
// (head, worker, chunk of the worker's query blocks), the tiles and columns
// that fall into each worker's KV shard.
#include "common.h"
#include "kernels.h"
#include "trace.h"

namespace msparse {

namespace {

constexpr int kPrepThreads = 1024;
constexpr int kItemThreads = 256, kItemWaves = kItemThreads / 64;
constexpr int kPrepWords = 32768;      // vertical bitmap words held in LDS (1M tokens)

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ uint64_t lanes_below() { return (1ull << lane_id()) - 1ull; }

// inclusive prefix sum over the wavefront
template <class T>
__device__ __forceinline__ T wave_scan(T x) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o);
        if (lane_id() >= o) x += y;
    }
    return x;
}

// Exclusive prefix sum over the NT-thread workgroup and the total; `tmp` holds
// NT / 64 values.
template <int NT, class T>
__device__ __forceinline__ T block_scan(T v, T* tmp, T& total) {
    const T x = wave_scan(v);
    const int wid = threadIdx.x >> 6;
    __syncthreads();   // tmp may still be read from the call before
    if (lane_id() == 63) tmp[wid] = x;
    __syncthreads();
    T base = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        if (w < wid) base += tmp[w];
        total += tmp[w];
    }
    return base + x - v;
}

// Block-diagonals x whose key block can lie in the step's shard: with striped
// shards query block qg = rank and key block qg - x = shard modulo world, so
// only one residue of x (zigzag shards have no such rule).
__device__ __forceinline__ bool diag_in_step(const IndexArgs& a, int32_t x) {
    return a.world == 1 || a.layout != MSPARSE_LAYOUT_STRIPED || (a.rank - a.shard + a.world - x % a.world) % a.world == 0;
}

// One workgroup per head.  Bound by latency: a chain of barriers and scans over
// the head's bitmap, which therefore sits in LDS up to 1M tokens.  Neighbouring
// slashes, which share a block-diagonal, are stored once per wave instead of 64
// times at one address.  28 heads x 512K (k_v 4096, k_s 16384): 135 -> 31 us;
// a step of its 8-worker ring 172 -> 35 us.
template <bool LDSV>
__global__ void __launch_bounds__(kPrepThreads) index_prep_kernel(IndexArgs a) {
    __shared__ int tmp[kPrepThreads / 64], run0;
    __shared__ uint32_t vsh[LDSV ? kPrepWords : 1];
    extern __shared__ uint32_t dsh[];  // D bitset, dwords words
    const int bh = blockIdx.x;
    const int tid = threadIdx.x;
    const Layout L{a.world, a.nb, a.layout};
    const int64_t Ng = int64_t(a.nb) * kBlock;

    // the overflow flag starts at 0 for this build (a kernel store, not a memset,
    // so that the call can be captured in a graph); the fill pass may set it
    if (bh == 0 && tid == 0 && a.overflow) *a.overflow = 0;
    // ---- verticals: bitmap (dedupes and sorts)
    uint32_t* vb = LDSV ? vsh : a.vbits + int64_t(bh) * a.vwords;
    for (int w = tid; w < a.vwords; w += kPrepThreads) vb[w] = 0u;
    for (int w = tid; w < a.dwords; w += kPrepThreads) dsh[w] = 0u;
    if (!LDSV) __threadfence();
    __syncthreads();
    const int32_t* vi = a.v_idx + int64_t(bh) * a.k_v;
    for (int j = tid; j < a.k_v; j += kPrepThreads) {
        int32_t v = vi[j];
        if (v >= 0 && v < Ng) atomicOr(&vb[v >> 5], 1u << (v & 31));
    }
    // ---- slashes: 64 neighbouring offsets share a block-diagonal, so in an
    // ascending list only the lanes that differ from the one before them store
    const int32_t* si = a.s_idx + int64_t(bh) * a.k_s;
    for (int j0 = 0; j0 < a.k_s; j0 += kPrepThreads) {
        const int j = j0 + tid;
        const int32_t dl = j < a.k_s ? si[j] : -1;
        const bool ok = dl >= 0 && dl < Ng;
        const int32_t lo = ok ? dl / kBlock : -1, hi = ok ? (dl + kBlock - 1) / kBlock : -1;
        const int32_t plo = __shfl_up(lo, 1), phi = __shfl_up(hi, 1);
        const bool first = lane_id() == 0;
        if (ok && (first || plo != lo)) atomicOr(&dsh[lo >> 5], 1u << (lo & 31));
        if (ok && hi < a.nb && (first || phi != hi)) atomicOr(&dsh[hi >> 5], 1u << (hi & 31));
    }
    if (!LDSV) __threadfence();
    __syncthreads();

    // ---- the shard's verticals in order, and (whole sequence) the verticals
    // before each block: a block's 64 bits per thread
    {
        auto word = [&](int w) { return LDSV ? vb[w] : __atomic_load_n(&vb[w], __ATOMIC_RELAXED); };
        int32_t* out = a.vlist + int64_t(bh) * a.k_v;
        int32_t* cv = a.cumv + int64_t(bh) * (a.nb + 1);
        int carry = 0;
        for (int j0 = 0; j0 < a.nb; j0 += kPrepThreads) {
            const int j = j0 + tid;
            uint64_t bits = 0;
            if (j < a.nb && L.owner(j) == a.shard) bits = uint64_t(word(2 * j)) | (uint64_t(word(2 * j + 1)) << 32);
            int total;
            int pos = carry + block_scan<kPrepThreads>(int(__popcll(bits)), tmp, total);
            if (j < a.nb && a.world == 1) cv[j] = pos;
            for (; bits; bits &= bits - 1) out[pos++] = j * kBlock + __ffsll((unsigned long long)bits) - 1;
            carry += total;
        }
        if (tid == 0) {
            if (a.world == 1) cv[a.nb] = carry;
            a.vcnt[bh] = carry;
            a.cnt_vcol[bh] = carry;
        }
    }
    // ---- block-diagonals: bitset copy, ascending list of the step's ones,
    // prefix counts per word (dpre) and the run of selected diagonals from 0
    {
        uint32_t* db = a.dbits + int64_t(bh) * a.dwords;
        int32_t* out = a.dlist + int64_t(bh) * a.nb;
        int32_t* dp = a.dpre + int64_t(bh) * (a.dwords + 1);
        if (tid == 0) run0 = a.nb;
        int carry = 0;
        for (int w0 = 0; w0 < a.dwords; w0 += kPrepThreads) {
            const int w = w0 + tid;
            uint32_t bits = w < a.dwords ? dsh[w] : 0u;
            if (w < a.dwords) {
                db[w] = bits;
                if (a.diag_bits_out) a.diag_bits_out[int64_t(bh) * a.dwords + w] = bits;
            }
            const uint32_t all = bits;
            if (a.world > 1)
                for (uint32_t b = all; b; b &= b - 1) {
                    const int x = __ffs(b) - 1;
                    if (!diag_in_step(a, (w << 5) + x)) bits &= ~(1u << x);
                }
            int total;
            int pos = carry + block_scan<kPrepThreads>(int(__popc(bits)), tmp, total);   // (its barriers order run0)
            if (w < a.dwords) {
                dp[w] = pos;
                if (all != 0xffffffffu) atomicMin(&run0, (w << 5) + __ffs(~all) - 1);
            }
            for (; bits; bits &= bits - 1) out[pos++] = (w << 5) + __ffs(bits) - 1;
            carry += total;
        }
        __syncthreads();
        if (tid == 0) {
            dp[a.dwords] = carry;
            a.dcnt[bh] = carry;
            a.drun[bh] = min(run0, a.nb);
        }
    }
    if (bh == 0) {
        if (a.q_blk_global)
            for (int l = tid; l < a.nqb; l += kPrepThreads) a.q_blk_global[l] = L.global(a.rank, l);
        if (a.k_blk_global)
            for (int l = tid; l < a.nkb; l += kPrepThreads) a.k_blk_global[l] = L.global(a.shard, l);
    }
}

__device__ __forceinline__ bool dbit(const uint32_t* db, int32_t x) { return (db[x >> 5] >> (x & 31)) & 1u; }

// Number of selected block-diagonals below x (0 <= x <= nb) from the per-word
// prefix counts.
__device__ __forceinline__ int32_t diag_below(const int32_t* dp, const uint32_t* db, int32_t x) {
    const int w = x >> 5, b = x & 31;
    return dp[w] + (b ? __popc(db[w] & ((1u << b) - 1u)) : 0);
}

// A head's lists, as prep left them.
struct HeadLists {
    const int32_t *dl, *dp, *cv, *vl;
    const uint32_t* db;
    int32_t dc, vc, run;
};
__device__ __forceinline__ HeadLists head_lists(const IndexArgs& a, int bh) {
    return {a.dlist + int64_t(bh) * a.nb,
            a.dpre + int64_t(bh) * (a.dwords + 1),
            a.cumv + int64_t(bh) * (a.nb + 1),
            a.vlist + int64_t(bh) * a.k_v,
            a.dbits + int64_t(bh) * a.dwords,
            a.dcnt[bh],
            a.vcnt[bh],
            a.drun[bh]};
}

// Ring step: one wavefront walks the lists of one item in order and calls
// emit(n, value) on the lanes that hold an entry, n its position; returns the
// number of entries.  Key blocks of query block qg, ascending (x descending):
template <class F>
__device__ __forceinline__ int32_t walk_key_blocks(const IndexArgs& a, const Layout& L, const HeadLists& H, int32_t qg,
                                                   F emit) {
    int32_t n = 0;
    for (int c0 = 0; c0 < H.dc; c0 += 64) {
        const int j = H.dc - 1 - (c0 + lane_id());
        bool pred = false;
        int32_t kg = 0;
        if (j >= 0) {
            const int32_t x = H.dl[j];
            kg = qg - x;
            pred = x <= qg && L.owner(kg) == a.shard;
        }
        const uint64_t m = __ballot(pred);
        if (pred) emit(n + __popcll(m & lanes_below()), L.local(kg));
        n += __popcll(m);
    }
    return n;
}
// columns of query block qg: the shard's verticals v <= 64 qg + 63 outside the
// selected diagonals
template <class F>
__device__ __forceinline__ int32_t walk_columns(const IndexArgs& a, const Layout& L, const HeadLists& H, int32_t qg,
                                                F emit) {
    const int32_t limit = qg * kBlock + kBlock - 1;
    int32_t n = 0;
    for (int c0 = 0; c0 < H.vc; c0 += 64) {
        const int j = c0 + lane_id();
        const int32_t v = j < H.vc ? H.vl[j] : INT32_MAX;
        const bool pred = v <= limit && !dbit(H.db, qg - v / kBlock);
        const uint64_t m = __ballot(pred);
        if (pred) emit(n + __popcll(m & lanes_below()), L.local(v / kBlock) * kBlock + v % kBlock);
        n += __popcll(m);
        if (__ballot(v > limit)) break;   // the list is ascending
    }
    return n;
}
// query blocks of key block kg, ascending
template <class F>
__device__ __forceinline__ int32_t walk_query_blocks(const IndexArgs& a, const Layout& L, const HeadLists& H,
                                                     int32_t kg, F emit) {
    int32_t n = 0;
    for (int c0 = 0; c0 < H.dc; c0 += 64) {
        const int j = c0 + lane_id();
        bool pred = false;
        int32_t qg = 0;
        if (j < H.dc) {
            qg = kg + H.dl[j];
            pred = qg < a.nb && L.owner(qg) == a.rank;
        }
        const uint64_t m = __ballot(pred);
        if (pred) emit(n + __popcll(m & lanes_below()), L.local(qg));
        n += __popcll(m);
    }
    return n;
}

// Count and fill work on chunks of a.chunk (at most 64) consecutive query or
// key blocks of one head, a workgroup per chunk: what a block's list needs (its
// length, and for the whole sequence how many verticals it has to look at) is
// found for all blocks of the chunk at once, a thread each, and the waves then
// take one block after another without a dependent load between them (a wave
// per block, each with its own chain of lookups, was bound by their latency).
// 28 heads x 512K (617 MB of entries): count 76 -> 44 us, fill 307 -> 170 us
// (3.6 TB/s; with 16-byte stores of four gathered entries 268 us); a step of its 8-worker ring: count 73 -> 18 us, fill 84 -> 25 us.
struct Chunk {
    bool key;        // key blocks (transposed lists) or query blocks
    int bh, i0, n;   // head, first local block, blocks
    int64_t id;      // chunk number among its kind
};
__device__ __forceinline__ Chunk chunk_of(const IndexArgs& a, int64_t t) {
    const int64_t nq = int64_t(a.BH) * a.nchq;
    Chunk c;
    c.key = t >= nq;
    c.id = c.key ? t - nq : t;
    const int per = c.key ? a.nchk : a.nchq;
    c.bh = int(c.id / per);
    c.i0 = int(c.id % per) * a.chunk;
    c.n = min(a.chunk, (c.key ? a.nkb : a.nqb) - c.i0);
    return c;
}

// Whole-sequence index (one worker): closed forms from the prefix counts.
// Query block i has the key blocks i - x for the diag_below(i + 1) selected x
// <= i, and as columns the verticals of blocks j <= i - R (blocks i - R + 1 ..
// i lie on the selected diagonals 0 .. R-1) minus those whose diagonal i - j
// is selected; key block k has the query blocks k + x, x < nb - k.
__device__ __forceinline__ int32_t columns_scanned(const HeadLists& H, int32_t i) {
    return H.cv[i - min(H.run, i + 1) + 1];   // verticals of blocks 0 .. i - R
}

// Per chunk: the inclusive prefix sums of its blocks' counts, and their totals.
__global__ void __launch_bounds__(kItemThreads) index_count_kernel(IndexArgs a) {
    __shared__ int32_t nblk[64], ncol[64];
    const Chunk c = chunk_of(a, blockIdx.x);
    const HeadLists H = head_lists(a, c.bh);
    const Layout L{a.world, a.nb, a.layout};
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    if (tid < 64) nblk[tid] = ncol[tid] = 0;
    __syncthreads();
    if (a.world == 1) {
        if (tid < c.n) {
            const int32_t i = c.i0 + tid;
            nblk[tid] = diag_below(H.dp, H.db, c.key ? a.nb - i : i + 1);
            if (!c.key) ncol[tid] = columns_scanned(H, i);
        }
        __syncthreads();
        if (!c.key) {
            // minus the verticals of blocks i - x, x selected, R <= x <= i: the
            // far diagonals dealt to groups of a.chunk threads, a block per
            // thread (neighbours read neighbouring prefix counts).  Their number
            // is known beforehand, so the loads of several are in flight (with
            // a break at the first one beyond the chunk, each waited for its
            // own: 28 heads x 128K with 8192 random slashes 86 -> 33 us)
            const int32_t t = tid & (a.chunk - 1), i = c.i0 + t, groups = kItemThreads / a.chunk;
            const int32_t jend = diag_below(H.dp, H.db, c.i0 + c.n);
            int32_t far = 0;
#pragma unroll 8
            for (int j = H.run + tid / a.chunk; j < jend; j += groups) {
                const int32_t x = H.dl[j];
                const int32_t b = min(max(i - x, 0), a.nb - 1);
                far += i >= x ? H.cv[b + 1] - H.cv[b] : 0;
            }
            if (t < c.n && far > 0) atomicSub(&ncol[t], far);
        }
    } else {
        auto none = [](int32_t, int32_t) {};
        for (int t = w; t < c.n; t += kItemWaves) {
            int32_t nb, nc = 0;
            if (c.key) {
                nb = walk_query_blocks(a, L, H, L.global(a.shard, c.i0 + t), none);
            } else {
                const int32_t qg = L.global(a.rank, c.i0 + t);
                nb = walk_key_blocks(a, L, H, qg, none);
                nc = walk_columns(a, L, H, qg, none);
            }
            if (lane == 0) {
                nblk[t] = nb;
                ncol[t] = nc;
            }
        }
    }
    __syncthreads();
    if (w != 0) return;
    const int64_t b = wave_scan(int64_t(nblk[lane])), k = wave_scan(int64_t(ncol[lane]));
    const int64_t item = int64_t(c.bh) * (c.key ? a.nkb : a.nqb) + c.i0 + lane;
    if (lane < c.n) {
        (c.key ? a.cnt_kblk : a.cnt_blk)[item] = b;
        if (!c.key) a.cnt_col[item] = k;
    }
    if (lane == 63) {
        a.scan_sums[(c.key ? 2 : 0) * a.scan_stride + c.id] = b;
        if (!c.key) a.scan_sums[a.scan_stride + c.id] = k;
    }
}

// Exclusive prefix sums, in place, of the chunks' totals (array blockIdx.x:
// blocks, columns, transposed blocks) and of the heads' verticals (array 3), and
// every list's full length at the end of its offsets.
__global__ void __launch_bounds__(kPrepThreads) index_scan_kernel(IndexArgs a) {
    __shared__ int64_t tmp[kPrepThreads / 64];
    const int which = blockIdx.x;
    const int64_t n = which == 3 ? a.BH : int64_t(a.BH) * (which == 2 ? a.nchk : a.nchq);
    int64_t* v = which == 3 ? a.cnt_vcol : a.scan_sums + which * a.scan_stride;
    int64_t carry = 0;
    for (int64_t i0 = 0; i0 < n; i0 += kPrepThreads) {
        const int64_t i = i0 + threadIdx.x;
        const int64_t x = i < n ? v[i] : 0;
        int64_t total;
        const int64_t pre = carry + block_scan<kPrepThreads>(x, tmp, total);
        if (i < n) v[i] = which == 3 ? pre + x : pre;
        carry += total;
    }
    if (threadIdx.x == 0) {
        if (which == 0) a.blk_ptr[int64_t(a.BH) * a.nqb] = carry;
        else if (which == 1) a.col_ptr[int64_t(a.BH) * a.nqb] = carry;
        else if (which == 2) a.kblk_ptr[int64_t(a.BH) * a.nkb] = carry;
        else a.vcol_ptr[a.BH] = carry;
    }
}

// Sum of v[0 .. n - 1] over the workgroup (all threads get it).
__device__ __forceinline__ int64_t block_sum(const int64_t* v, int64_t n, int64_t* tmp) {
    int64_t x = 0, total;
    for (int64_t i = threadIdx.x; i < n; i += kItemThreads) x += v[i];
    block_scan<kItemThreads>(x, tmp, total);
    return total;
}

// Lookups in flight per lane of the fill pass (a store between two loads would
// make the second wait: 32 heads x 128K with 8192 spread verticals 783 -> 478 us).
constexpr int kFillUnroll = 4;

// The offsets and the entries of a chunk's lists at them; the workgroups after
// the chunks write a head's vertical list each.  A list beyond its capacity is
// left out and sets the overflow flag.
template <bool RING>
__global__ void __launch_bounds__(kItemThreads) index_fill_kernel(IndexArgs a) {
    __shared__ int64_t tmp[kItemWaves], bend[65], cend[65];   // [t + 1]: end of block t's list
    __shared__ int32_t nscan[64];
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int64_t nchunks = int64_t(a.BH) * (a.nchq + a.nchk);
    const Layout L{a.world, a.nb, a.layout};
    if (blockIdx.x >= nchunks) {
        const int bh = int(blockIdx.x - nchunks);
        const int before = a.scanned ? max(bh - 1, 0) : 0;
        const int64_t base = block_sum(a.cnt_vcol + before, bh - before, tmp), n = a.vcnt[bh];
        if (tid == 0) {
            if (bh == 0) a.vcol_ptr[0] = 0;
            a.vcol_ptr[bh + 1] = base + n;
            if (base + n > a.vcol_cap && a.overflow) atomicOr(a.overflow, 1);
        }
        if (base + n > a.vcol_cap) return;
        const int32_t* vl = a.vlist + int64_t(bh) * a.k_v;
        for (int64_t j = tid; j < n; j += kItemThreads)
            a.vcol_idx[base + j] = L.local(vl[j] / kBlock) * kBlock + vl[j] % kBlock;
        return;
    }
    const Chunk c = chunk_of(a, blockIdx.x);
    const HeadLists H = head_lists(a, c.bh);
    // offset of the chunk's first list: the totals of the chunks before it
    const int64_t* sb = a.scan_sums + (c.key ? 2 : 0) * a.scan_stride;
    const int64_t* scol = a.scan_sums + a.scan_stride;
    const int64_t b0 = a.scanned ? sb[c.id] : block_sum(sb, c.id, tmp);
    const int64_t c0 = c.key ? 0 : (a.scanned ? scol[c.id] : block_sum(scol, c.id, tmp));
    const int64_t item0 = int64_t(c.bh) * (c.key ? a.nkb : a.nqb) + c.i0;
    int64_t* bptr = c.key ? a.kblk_ptr : a.blk_ptr;
    if (tid < c.n) {
        const int64_t be = b0 + (c.key ? a.cnt_kblk : a.cnt_blk)[item0 + tid];
        bend[tid + 1] = be;
        bptr[item0 + tid + 1] = be;
        if (!c.key) {
            const int64_t ce = c0 + a.cnt_col[item0 + tid];
            cend[tid + 1] = ce;
            a.col_ptr[item0 + tid + 1] = ce;
            nscan[tid] = !RING ? columns_scanned(H, c.i0 + tid) : 0;
        }
    }
    if (tid == 0) {
        bend[0] = b0;
        cend[0] = c0;
        if (c.id == 0) {
            bptr[0] = 0;
            if (!c.key) a.col_ptr[0] = 0;
        }
    }
    __syncthreads();
    int32_t* bidx = c.key ? a.kblk_idx : a.blk_idx;
    for (int t = w; t < c.n; t += kItemWaves) {
        const int32_t i = c.i0 + t;
        const int64_t base = bend[t];
        const int nblk = int(bend[t + 1] - base);
        if (bend[t + 1] > a.blk_cap) {
            if (lane == 0 && a.overflow) atomicOr(a.overflow, 1);
        } else if constexpr (!RING) {
            // i + dl[0 ..] or i - dl[nblk - 1 .. 0]
            const int32_t* d0 = H.dl + (c.key ? 0 : nblk - 1);
            const int32_t sign = c.key ? 1 : -1;
            int32_t* dst = bidx + base;
            int k = lane;
            for (; k + 64 * (kFillUnroll - 1) < nblk; k += 64 * kFillUnroll) {
                int32_t v[kFillUnroll];
#pragma unroll
                for (int u = 0; u < kFillUnroll; ++u) v[u] = d0[sign * (k + 64 * u)];
#pragma unroll
                for (int u = 0; u < kFillUnroll; ++u) dst[k + 64 * u] = i + sign * v[u];
            }
            for (; k < nblk; k += 64) dst[k] = i + sign * d0[sign * k];
        } else {
            auto emit = [&](int32_t n, int32_t v) { bidx[base + n] = v; };
            if (c.key) walk_query_blocks(a, L, H, L.global(a.shard, i), emit);
            else walk_key_blocks(a, L, H, L.global(a.rank, i), emit);
        }
        if (c.key || cend[t + 1] == cend[t]) continue;
        const int64_t cbase = cend[t];
        if (cend[t + 1] > a.col_cap) {
            if (lane == 0 && a.overflow) atomicOr(a.overflow, 1);
            continue;
        }
        if constexpr (RING) {
            walk_columns(a, L, H, L.global(a.rank, i), [&](int32_t n, int32_t v) { a.col_idx[cbase + n] = v; });
            continue;
        }
        const int32_t scan = nscan[t];
        int32_t n = 0, k0 = 0;
        auto store = [&](int32_t v, bool pred) {
            const uint64_t m = __ballot(pred);
            if (pred) a.col_idx[cbase + n + __popcll(m & lanes_below())] = v;
            n += __popcll(m);
        };
        for (; k0 + 64 * kFillUnroll <= scan; k0 += 64 * kFillUnroll) {
            int32_t v[kFillUnroll];
            bool pred[kFillUnroll];
#pragma unroll
            for (int u = 0; u < kFillUnroll; ++u) v[u] = H.vl[k0 + 64 * u + lane];
#pragma unroll
            for (int u = 0; u < kFillUnroll; ++u) pred[u] = !dbit(H.db, i - v[u] / kBlock);
#pragma unroll
            for (int u = 0; u < kFillUnroll; ++u) store(v[u], pred[u]);
        }
        for (; k0 < scan; k0 += 64) {
            const int32_t j = k0 + lane, v = j < scan ? H.vl[j] : 0;
            store(v, j < scan && !dbit(H.db, i - v / kBlock));
        }
    }
}

// ---------------------------------------------------------------- ring workload
constexpr int kWorkThreads = 256;
constexpr int kWorkChunk = 64;   // query blocks per workgroup

// Adds 1 to bin `bin` for every lane with `on`: lanes sharing the first pending
// lane's bin are counted with a ballot (zigzag shards are runs of neighbouring
// blocks, so most lanes share a bin), up to four rounds, then single adds.
__device__ __forceinline__ void bin_add(uint32_t* h, int32_t bin, bool on) {
    bool pending = on;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const uint64_t pm = __ballot(pending);
        if (pm == 0) return;
        const int first = __builtin_ctzll(pm);
        const int32_t lb = __shfl(bin, first);
        const bool same = pending && bin == lb;
        const uint64_t sm = __ballot(same);
        if (lane_id() == first) atomicAdd(&h[lb], uint32_t(__popcll(sm)));
        pending = pending && !same;
    }
    if (pending) atomicAdd(&h[bin], 1u);
}

__global__ void __launch_bounds__(256) ring_work_zero_kernel(int64_t* tiles, int64_t* cols, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
        tiles[i] = 0;
        cols[i] = 0;
    }
}

__global__ void __launch_bounds__(kWorkThreads) ring_work_kernel(IndexArgs a, int32_t W, int32_t layout,
                                                                 int64_t* tiles, int64_t* cols) {
    __shared__ uint32_t ht[kMaxRingWorld], hc[kMaxRingWorld];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const Layout L{W, a.nb, layout};
    const int per = a.nb / W;                        // query blocks per worker
    const int nchunk = (per + kWorkChunk - 1) / kWorkChunk;
    int item = blockIdx.x;
    const int chunk = item % nchunk;
    item /= nchunk;
    const int r = item % W;
    const int bh = item / W;
    for (int i = tid; i < W; i += kWorkThreads) {
        ht[i] = 0;
        hc[i] = 0;
    }
    __syncthreads();
    const int32_t* dl = a.dlist + int64_t(bh) * a.nb;
    const int dc = a.dcnt[bh];
    const uint32_t* db = a.dbits + int64_t(bh) * a.dwords;
    const int32_t* vl = a.vlist + int64_t(bh) * a.k_v;
    const int vc = a.vcnt[bh];
    const int l1 = min(per, (chunk + 1) * kWorkChunk);
    for (int l = chunk * kWorkChunk + wave; l < l1; l += kWorkThreads / 64) {
        const int32_t i = L.global(r, l);
        // tiles (i, i - x), x in D, x <= i
        for (int c0 = 0; c0 < dc; c0 += 64) {
            const int j = c0 + lane;
            const int32_t x = j < dc ? dl[j] : 0;
            const bool on = j < dc && x <= i;
            bin_add(ht, on ? L.owner(i - x) : 0, on);
        }
        // columns v <= 64 i + 63 whose block-diagonal is not in D
        const int32_t limit = i * kBlock + kBlock - 1;
        for (int c0 = 0; c0 < vc; c0 += 64) {
            if (vl[c0] > limit) break;   // ascending list
            const int j = c0 + lane;
            const int32_t v = j < vc ? vl[j] : 0;
            const bool on = j < vc && v <= limit && !dbit(db, i - v / kBlock);
            bin_add(hc, on ? L.owner(v / kBlock) : 0, on);
        }
    }
    __syncthreads();
    for (int sh = tid; sh < W; sh += kWorkThreads) {
        if (ht[sh]) atomicAdd(reinterpret_cast<unsigned long long*>(tiles + int64_t(r) * W + sh), (unsigned long long)ht[sh]);
        if (hc[sh]) atomicAdd(reinterpret_cast<unsigned long long*>(cols + int64_t(r) * W + sh), (unsigned long long)hc[sh]);
    }
}

}  // namespace

hipError_t launch_ring_work(const IndexArgs& a, int32_t world, int32_t layout, int64_t* tiles, int64_t* cols,
                            hipStream_t s) {
    const int64_t n = int64_t(world) * world;
    {
        TraceScope _t("ring_work_zero", s);
        hipLaunchKernelGGL(ring_work_zero_kernel, dim3(unsigned(std::min<int64_t>((n + 255) / 256, 4096))), dim3(256),
                           0, s, tiles, cols, n);
    }
    const int per = a.nb / world;
    const int64_t grid = int64_t(a.BH) * world * ((per + kWorkChunk - 1) / kWorkChunk);
    {
        TraceScope _t("ring_work", s);
        hipLaunchKernelGGL(ring_work_kernel, dim3(unsigned(grid)), dim3(kWorkThreads), 0, s, a, world, layout, tiles,
                           cols);
    }
    return hipGetLastError();
}

hipError_t launch_index_prep(const IndexArgs& a, hipStream_t s) {
    const size_t shmem = size_t(a.dwords) * sizeof(uint32_t);
    TraceScope _t("index_prep", s);
    if (a.vwords <= kPrepWords)
        hipLaunchKernelGGL(index_prep_kernel<true>, dim3(a.BH), dim3(kPrepThreads), shmem, s, a);
    else
        hipLaunchKernelGGL(index_prep_kernel<false>, dim3(a.BH), dim3(kPrepThreads), shmem, s, a);
    return hipGetLastError();
}

hipError_t launch_index_count(const IndexArgs& a, hipStream_t s) {
    const int64_t grid = int64_t(a.BH) * (a.nchq + a.nchk);
    TraceScope _t("index_count", s);
    hipLaunchKernelGGL(index_count_kernel, dim3(unsigned(grid)), dim3(kItemThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_index_scan(const IndexArgs& a, hipStream_t s) {
    TraceScope _t("index_scan", s);
    hipLaunchKernelGGL(index_scan_kernel, dim3(4), dim3(kPrepThreads), 0, s, a);
    return hipGetLastError();
}

__global__ void index_mark_overflow_kernel(int32_t* flag) {
    if (threadIdx.x == 0) *flag = 1;
}

hipError_t launch_index_mark_overflow(const IndexArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(index_mark_overflow_kernel, dim3(1), dim3(64), 0, s, a.overflow);
    return hipGetLastError();
}

hipError_t launch_index_fill(const IndexArgs& a, hipStream_t s) {
    const int64_t grid = int64_t(a.BH) * (a.nchq + a.nchk) + a.BH;
    TraceScope _t("index_fill", s);
    if (a.world > 1) hipLaunchKernelGGL(index_fill_kernel<true>, dim3(unsigned(grid)), dim3(kItemThreads), 0, s, a);
    else hipLaunchKernelGGL(index_fill_kernel<false>, dim3(unsigned(grid)), dim3(kItemThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace msparse
