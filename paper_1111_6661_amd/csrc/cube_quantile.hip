// cube_quantile.hip -- exact order statistics of the valid voxels: any number
// of ranks refined side by side (selection, the median, quantiles).  The
// median and quantiles are the paper's example of a global, multi-pass task
// (Section 3).
//
// Each wanted rank is found in the 32-bit order key of the voxels (the key
// orders like the value, -0 before +0) a few bits at a time.  Every pass keeps
// one histogram per distinct key prefix still in play, side by side in LDS:
//   pass 0: one 4096-bin histogram of the top 12 key bits;
//   then, when the ranks fall in at most 8 distinct top buckets and number
//   at most 96 ("wide"), 12 and 8 more bits (up to 8 histograms of 4096 bins,
//   then up to 96 of 256);
//   otherwise 8, 6 and 6 more bits (up to 128 histograms of 256 bins, then
//   128 of 64, then 128 of 64).
// A voxel finds its histogram through a chain of direct-mapped LDS byte
// tables, one per level of the prefix.  Entries hold index + 1 (0: none),
// and row 0 of every further table is all zero, so a voxel outside the
// wanted prefixes falls through to 0 with no test: the table of the top 12
// key bits gives its index among the wanted 12-bit prefixes, each further
// table, indexed by that entry and the level's next key bits, its index
// among the longer prefixes.  Only voxels that end at a wanted prefix count, in
// the row of its index.  No search.  (Without a row for entry 0 one prefix has
// room for twice the LDS copies of its 4096 bins: one value in 2^28 voxels,
// three levels, 650 -> 563 us.)
//
// The host queues all the passes at once.  The last block of each adds up that
// pass's histograms, finds the bin of every rank, and lays out the next pass:
// its prefixes, tables and bits (by the functions of cube_quantile_plan.h, which
// also holds the same plan for the host).  The last pass's last block writes
// the ranks' keys to host memory.  When the voxels under the wanted prefixes are few enough, the last
// pass but one also copies them out, and the last reads only the copies.
//
// Measured (call, microseconds; before: the host read every pass's counts
// back, laid out the next pass and uploaded its tables; a fourth full pass
// looked for the upper middle of an even count): median of 2^17 voxels 133 ->
// 42, of 2^24 -> 68 (larger boxes: cube_bracket.h, one read); 64 levels of
// 2^20 302 -> 85, of 2^28 910 -> 737 and, once the last of the four passes
// read copies, 610 (9 levels 703 -> 558).
#include <math.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <mutex>
#include <vector>

#include "cube_quantile_plan.h"
#include "cube_scan.h"

namespace cube {

// Passes of the calling thread's last successful cube_quantiles call.
thread_local int g_quant_reads = 0;
// CUBE_RANK_* of its last successful selection, median or quantiles call.
thread_local int g_rank_route = 0;

namespace {

constexpr int Q_THREADS = 1024;
constexpr int Q_MAX_RANKS = 2 * CUBE_MAX_QUANTILES;   // index + 1 fits a byte
constexpr size_t Q_LDS = QP_LDS;            // dynamic LDS of one block at most
constexpr int Q_ACC = QP_COUNTERS;          // slots << bin width never exceeds this
constexpr size_t Q_TAB = QP_TAB_MAX;        // bytes: T1, T2, T3 at most
static_assert(Q_MAX_RANKS == QP_RANKS, "a table entry is a byte");
// Copied voxels: 2^24 floats (64 MiB) shared out among the blocks.
constexpr unsigned int CAND_TOTAL = 1u << 24;

// The ranks and the next pass's layout, between the passes.
struct RankState {
    unsigned long long rank[Q_MAX_RANKS];  // rank left inside the key prefix found so far
    unsigned int key[Q_MAX_RANKS];         // that prefix, at the top of the word; ascending
    int m;                       // ranks
    int done;                    // the result (or an error) has been written
    int wide;
    int collect;                 // the pass that copies the counted voxels out (0: none)
    unsigned long long nv;       // valid voxels
    unsigned int overflow;       // a block's region of copied voxels was too small
    int shift, width;            // the next pass bins key bits [shift, shift + width)
    int w2, w3;                  // bits of the second and third prefix levels
    int slots;                   // histograms (prefixes) in the next pass
    int t2_bytes, t3_bytes;      // sizes of the second and third tables
};

// What the host reads.
struct RankOut {
    unsigned int done;           // the call's number, written last
    int status;                  // 0, or 1: rank >= n_valid, 2: no valid voxel
    int m, wide;
    int route;                   // CUBE_RANK_COPIES or CUBE_RANK_OVERFLOW
    unsigned long long n_valid;
    unsigned int key[Q_MAX_RANKS];
};

enum { RANK_GIVEN = 0, RANK_MEDIAN = 1, RANK_LEVELS = 2 };
// Status of the single-read search: go on with the passes over the box.
constexpr int RANK_MISSED = 3;

struct RankArgs {
    Geom g;
    Claim claim;                 // the partition (its counter zero on entry)
    RankState *st;
    unsigned char *tab;          // T1 (4096 bytes), T2, T3, back to back
    unsigned long long *acc;     // Q_ACC counters and the valid count, zero between passes
    unsigned int *ticket;
    float *cand;                 // per-block regions of copied voxels, cand_cap each
    unsigned int *cand_n;        // voxels each block copied
    unsigned int cand_cap;
    int32_t max_clog;            // LDS copies of each histogram, at most
    uint32_t lds_bytes;          // dynamic LDS of this launch
    int32_t mode, nq;            // RANK_*; levels (RANK_LEVELS)
    unsigned long long rank;     // RANK_GIVEN
    RankOut *out;                // host memory
    unsigned int gen;
    double q[CUBE_MAX_QUANTILES];
};

// NL: prefix levels of this pass (0 for the first pass).
template <int NL>
struct QuantStep {
    unsigned int *lds;
    const unsigned char *t1, *t2, *t3;
    int shift, w2, w3, clog, cbase;
    unsigned int bmask;
    int wb;
    unsigned int valid;            // first pass: valid voxels seen by this wavefront
    bool collect;                  // second or third pass: copy the counted voxels out
    float *cand;
    unsigned int cand_cap;
    unsigned int *s_cnt;           // voxels this block copied (LDS counter)

    template <int NV>
    __device__ __forceinline__ void operator()(const float (&x)[NV])
    {
        if (NL == 0) {
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const float v = x[j];
                const bool ok = v == v;
                valid += (unsigned int)__popcll(__builtin_amdgcn_ballot_w64(ok));
                // one histogram, blanks skipped (they are rare)
                if (ok) atomicAdd(&lds[((order_key(v) >> 20) << clog) + cbase], 1u);
            }
        } else {
            // Histogram row g of each voxel: 0 (no wanted prefix) counts
            // nothing.  The tables are read level by level for all NV voxels
            // before any count is added: the counts live in the same LDS, so
            // a table read after an add could not be moved ahead of it, and
            // the voxels' lookups would run one after another.  With two or
            // three table levels the key fields are single bit-field extracts
            // (the one-level pass measured slower with them: 2.52 against
            // 2.34 ms on 2^32 voxels).
            unsigned int k[NV], g[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                k[j] = order_key(x[j]);
                g[j] = t1[k[j] >> 20];
            }
            if (NL >= 2) {
#pragma unroll
                for (int j = 0; j < NV; ++j)
                    g[j] = t2[qp_entry(g[j], k[j], 20 - w2, w2)];
            }
            if (NL >= 3) {
#pragma unroll
                for (int j = 0; j < NV; ++j)
                    g[j] = t3[qp_entry(g[j], k[j], 20 - w2 - w3, w3)];
            }
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const unsigned int idx =
                    NL >= 2 ? qp_entry(g[j], k[j], shift, wb)
                            : (g[j] << wb) | ((k[j] >> shift) & bmask);
                if (x[j] == x[j] && g[j] != 0u) atomicAdd(&lds[(idx << clog) + cbase], 1u);
            }
            if ((NL == 1 || NL == 2) && collect) copy_out<NV>(x, g);
        }
    }

    // The counted voxels to the block's region: one LDS atomic per wavefront
    // and step, each voxel at its rank among the step's counted ones.
    template <int NV>
    __device__ __forceinline__ void copy_out(const float (&x)[NV], const unsigned int (&g)[NV])
    {
        unsigned int total = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j)
            total += (unsigned int)__popcll(
                __builtin_amdgcn_ballot_w64(x[j] == x[j] && g[j] != 0u));
        if (!total) return;  // wavefront-uniform
        const int lane = threadIdx.x & 63;
        unsigned int at = 0;
        if (lane == 0) at = atomicAdd(s_cnt, total);
        at = (unsigned int)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const bool in = x[j] == x[j] && g[j] != 0u;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(in);
            if (!m) continue;
            const unsigned int i =
                at + __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32),
                                               __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
            if (in && i < cand_cap) cand[i] = x[j];
            at += (unsigned int)__popcll(m);
        }
    }
};

// ------------------------------------------------- the end of a pass (last block)

struct CountStep {  // inclusive scan, and the total in the last lane
    unsigned long long &v;
    template <class C, class R>
    __device__ __forceinline__ void operator()(C, R)
    {
        v += dpp<C::value, R::value>(0ull, v);
    }
};

// Shared memory of a pass's end.
struct RankShared {
    unsigned long long rank[Q_MAX_RANKS];
    unsigned long long left[Q_MAX_RANKS];  // the rank inside its bin
    unsigned long long count[Q_MAX_RANKS]; // voxels in the rank's bin
    unsigned int key[Q_MAX_RANKS];
    unsigned int bin[Q_MAX_RANKS];
    int slot[Q_MAX_RANKS];                 // index of the rank's key prefix
    int first[Q_MAX_RANKS + 1];            // a slot's first rank
    unsigned long long wave[MAX_WAVES];
    unsigned long long mask[2];
    unsigned long long nv;
    int m, slots, status;
};

// The index of each rank's top `bits` key bits among the distinct ones (the
// keys ascend), for the ranks of threads 0..m-1; returns their number.
// Called by the whole block, with barriers.
__device__ __forceinline__ int prefix_index(RankShared &s, int m, int bits, int *idx)
{
    const int tid = threadIdx.x, wid = tid >> 6;
    const int sh = 32 - bits;
    const bool flag = tid < m && (tid == 0 || (s.key[tid] >> sh) != (s.key[tid - 1] >> sh));
    if (wid < 2) {
        const unsigned long long b = __builtin_amdgcn_ballot_w64(flag);
        if ((tid & 63) == 0) s.mask[wid] = b;
    }
    __syncthreads();
    const unsigned long long m0 = s.mask[0], m1 = s.mask[1];
    __syncthreads();
    const unsigned long long upto = ~0ull >> (63 - (tid & 63));
    *idx = tid < 64 ? __popcll(m0 & upto) - 1 : __popcll(m0) + __popcll(m1 & upto) - 1;
    return __popcll(m0) + __popcll(m1);
}

// The ranks asked for (first pass), ascending and distinct.
__device__ __forceinline__ void wanted_ranks(const RankArgs &a, RankShared &s,
                                             unsigned long long *scratch)
{
    const int tid = threadIdx.x;
    const unsigned long long nv = s.nv;
    if (a.mode != RANK_LEVELS) {
        if (tid == 0) {
            s.status = a.mode == RANK_GIVEN ? (a.rank >= nv ? 1 : 0) : (nv == 0 ? 2 : 0);
            s.rank[0] = a.mode == RANK_GIVEN ? a.rank : (nv - 1) / 2;
            s.rank[1] = s.rank[0] + 1;
            s.m = a.mode == RANK_MEDIAN && nv % 2 == 0 ? 2 : 1;
        }
        __syncthreads();
        return;
    }
    // Level q takes ranks floor(q (n - 1)) and, unless that is whole, the
    // next.  Sorted and made distinct by counting: of B threads, 8 (or 4, 2)
    // share a rank's comparisons.
    const int n = 2 * a.nq, B = blockDim.x;
    unsigned int *dup = reinterpret_cast<unsigned int *>(scratch + Q_MAX_RANKS);
    unsigned int *below = dup + Q_MAX_RANKS;
    if (tid < n) {
        const double h = a.q[tid >> 1] * (double)(nv - 1);
        const double j = floor(h);
        scratch[tid] = (unsigned long long)j + ((tid & 1) && h - j > 0.0 ? 1ull : 0ull);
        dup[tid] = below[tid] = 0u;
    }
    __syncthreads();
    const int share = B / Q_MAX_RANKS, i = tid / share, part = tid % share;
    const unsigned long long mine = i < n ? scratch[i] : 0ull;
    if (i < n) {
        unsigned int same = 0u;
        for (int k = part; k < i; k += share) same |= scratch[k] == mine ? 1u : 0u;
        if (same) atomicOr(&dup[i], 1u);
    }
    __syncthreads();
    if (i < n && !dup[i]) {
        unsigned int less = 0u;
        for (int k = part; k < n; k += share) less += !dup[k] && scratch[k] < mine ? 1u : 0u;
        if (less) atomicAdd(&below[i], less);
    }
    if (tid < 128) {
        const unsigned long long m = __builtin_amdgcn_ballot_w64(tid < n && !dup[tid]);
        if ((tid & 63) == 0) s.mask[tid >> 6] = m;
    }
    __syncthreads();
    if (tid < n && !dup[tid]) s.rank[below[tid]] = scratch[tid];
    if (tid == 0) {
        s.m = __popcll(s.mask[0]) + __popcll(s.mask[1]);
        s.status = nv == 0 ? 2 : 0;
    }
    __syncthreads();
}

// The bin of every rank in its slot's histogram; the counters return to zero.
// `sums`: blockDim.x words of LDS.
__device__ __forceinline__ void find_bins(const RankArgs &a, RankShared &s, int width,
                                          unsigned long long *sums)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, B = blockDim.x;
    const int nw = B >> 6, nbins = 1 << width;
    if (nbins > 64 * 4) {
        // 4096 bins: the whole block on one slot, consecutive bins per thread;
        // the threads' inclusive sums go to LDS, where each rank searches.
        const int per = nbins / B;
        for (int slot = 0; slot < s.slots; ++slot) {
            unsigned long long *h = a.acc + (size_t)slot * nbins;
            unsigned long long sum = 0;
            for (int k = 0; k < per; ++k) sum += h[tid * per + k];
            unsigned long long upto = sum;
            wave_reduce(CountStep{upto});
            if (lane == WAVE_LAST) s.wave[wid] = upto;
            __syncthreads();
            for (int w = 0; w < wid; ++w) upto += s.wave[w];
            sums[tid] = upto;
            __syncthreads();
            const int i = s.first[slot] + tid;
            if (i < s.first[slot + 1]) {
                unsigned long long r = s.rank[i];
                int lo = 0, hi = B - 1;  // the first thread whose sum passes r
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (sums[mid] > r) hi = mid;
                    else lo = mid + 1;
                }
                if (lo > 0) r -= sums[lo - 1];
                const unsigned long long *c = h + lo * per;
                int k = 0;
                while (k < per - 1 && c[k] <= r) r -= c[k++];
                s.left[i] = r;
                s.bin[i] = (unsigned int)(lo * per + k);
                s.count[i] = c[k];
            }
            __syncthreads();
            for (int k = 0; k < per; ++k) h[tid * per + k] = 0ull;
        }
        __syncthreads();
        return;
    }
    // 256 or 64 bins: a wavefront per slot, 4 or 1 consecutive bins per lane.
    const int per = nbins / 64;
    for (int slot = wid; slot < s.slots; slot += nw) {
        unsigned long long *h = a.acc + (size_t)slot * nbins + lane * per;
        unsigned long long c[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[k] = k < per ? h[k] : 0ull;
            sum += c[k];
        }
        unsigned long long upto = sum;
        wave_reduce(CountStep{upto});
        const unsigned long long before = upto - sum;
        for (int i = s.first[slot]; i < s.first[slot + 1]; ++i) {
            unsigned long long r = s.rank[i];
            if (r >= before && r < upto) {  // one lane
                r -= before;
                int k = 0;
                while (k < per - 1 && c[k] <= r) r -= c[k++];
                s.left[i] = r;
                s.bin[i] = (unsigned int)(lane * per + k);
                s.count[i] = c[k];
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < per) h[k] = 0ull;
    }
    __syncthreads();
}

// The last block's part of pass NL: the ranks' bins, then the next pass's
// layout or, after the last bits, the result.  `scratch`: the block's dynamic
// LDS.
template <int NL>
__device__ void rank_end(const RankArgs &a, RankShared &s, unsigned int *scratch, int shift,
                         int width, int slots, int wide, int w2, int w3)
{
    const int tid = threadIdx.x;
    RankState *st = a.st;
    if (tid == 0) {
        s.status = 0;
        s.slots = slots;
        if (NL == 0) {
            s.nv = a.acc[Q_ACC];
            a.acc[Q_ACC] = 0ull;
        } else {
            s.m = st->m;
        }
    }
    __syncthreads();
    if (NL == 0) {
        wanted_ranks(a, s, reinterpret_cast<unsigned long long *>(scratch));
        if (s.status) {  // nothing to find: leave the counters at zero and say so
            for (int b = tid; b < 4096; b += blockDim.x) a.acc[b] = 0ull;
            if (tid == 0) {
                st->done = 1;
                store_result<true>(&a.out->status, s.status);
                store_result<true>(&a.out->n_valid, s.nv);
            }
            tell_host(&a.out->done, a.gen);
            return;
        }
        if (tid < s.m) s.key[tid] = 0u;
        if (tid == 0) {
            s.first[0] = 0;
            s.first[1] = s.m;
        }
        __syncthreads();
    } else {
        if (tid < s.m) {
            s.rank[tid] = st->rank[tid];
            s.key[tid] = st->key[tid];
        }
        __syncthreads();
        int idx = 0;
        const int n = prefix_index(s, s.m, 32 - shift - width, &idx);
        if (tid < s.m && (tid == 0 || (s.key[tid] >> (shift + width)) !=
                                          (s.key[tid - 1] >> (shift + width))))
            s.first[idx] = tid;
        if (tid == 0) s.first[n] = s.m;
        __syncthreads();
    }
    if (tid < s.m) {
        s.bin[tid] = (1u << width) - 1u;
        s.left[tid] = s.count[tid] = 0ull;
    }
    __syncthreads();
    find_bins(a, s, width, reinterpret_cast<unsigned long long *>(scratch));

    const int m = s.m;
    if (tid < m) {
        s.key[tid] |= s.bin[tid] << shift;
        st->key[tid] = s.key[tid];
        st->rank[tid] = s.left[tid];
    }
    __syncthreads();
    if (shift == 0) {  // every key is complete
        if (tid < m) store_result<true>(&a.out->key[tid], s.key[tid]);
        if (tid == 0) {
            st->done = 1;
            store_result<true>(&a.out->m, m);
            store_result<true>(&a.out->wide, wide);
            store_result<true>(&a.out->route, !st->collect     ? 0
                                              : st->overflow ? CUBE_RANK_OVERFLOW
                                                             : CUBE_RANK_COPIES);
            store_result<true>(&a.out->status, 0);
        }
        tell_host(&a.out->done, a.gen);
        return;
    }

    // The next pass: its prefix levels, its tables, its bits.
    int i1 = 0, i2 = 0, i3 = 0;
    const int n1 = prefix_index(s, m, 12, &i1);
    if (NL == 0) wide = qp_wide(n1, m) ? 1 : 0;
    const int next_width = qp_width(wide != 0, NL + 1);
    if (NL == 1) w2 = width;
    if (NL == 2) w3 = width;
    int n2 = 0, n3 = 0, t2_bytes = 0, t3_bytes = 0;
    if (NL >= 1) {
        n2 = prefix_index(s, m, 12 + w2, &i2);
        t2_bytes = qp_table_bytes(n1, w2);
    }
    if (NL >= 2) {
        n3 = prefix_index(s, m, 12 + w2 + w3, &i3);
        t3_bytes = qp_table_bytes(n2, w3);
    }
    const int words = (4096 + t2_bytes + t3_bytes) / 4;
    for (int i = tid; i < words; i += blockDim.x) scratch[i] = 0u;
    __syncthreads();
    unsigned char *t1 = reinterpret_cast<unsigned char *>(scratch);
    if (tid < m) {  // ranks under one prefix write the same byte
        const unsigned int k = s.key[tid];
        t1[k >> 20] = (unsigned char)(i1 + 1);
        if (NL >= 1)
            t1[4096 + qp_entry((unsigned int)i1 + 1u, k, 20 - w2, w2)] = (unsigned char)(i2 + 1);
        if (NL >= 2)
            t1[4096 + t2_bytes + qp_entry((unsigned int)i2 + 1u, k, 20 - w2 - w3, w3)] =
                (unsigned char)(i3 + 1);
    }
    __syncthreads();
    if (NL < 2 && tid < 128) {  // the voxels under the wanted prefixes
        unsigned long long pop =
            tid < m && (tid == 0 || (s.key[tid] >> shift) != (s.key[tid - 1] >> shift))
                ? s.count[tid] : 0ull;
        wave_reduce(CountStep{pop});
        if ((tid & 63) == WAVE_LAST) s.wave[tid >> 6] = pop;
    }
    __syncthreads();
    unsigned int *tab = reinterpret_cast<unsigned int *>(a.tab);
    for (int i = tid; i < words; i += blockDim.x) tab[i] = scratch[i];
    if (tid == 0) {
        if (NL == 0) {
            st->overflow = 0u;
            st->m = m;
            st->wide = wide;
            st->collect = 0;
            st->nv = s.nv;
            st->done = 0;
            store_result<true>(&a.out->n_valid, s.nv);
        }
        // Copy those voxels out in the next pass when that is less than
        // reading the box again and the regions have room: under the top 12
        // bits when three passes are left but one, else under the top 20
        // (64 levels of 2^28 noise voxels: about 0.4 % of them), so that the
        // last pass reads the copies.
        if (NL < 2 && (NL == 0) == (wide != 0)) {
            const unsigned long long pop = s.wave[0] + s.wave[1];
            const unsigned long long nv = NL == 0 ? s.nv : st->nv;
            if (a.cand && pop <= nv / 6 && pop <= (unsigned long long)CAND_TOTAL / 4 * 3)
                st->collect = NL + 1;
        }
        st->shift = shift - next_width;
        st->width = next_width;
        st->w2 = w2;
        st->w3 = w3;
        st->slots = NL == 0 ? n1 : (NL == 1 ? n2 : n3);
        st->t2_bytes = t2_bytes;
        st->t3_bytes = t3_bytes;
    }
}

template <int NL, bool PACKED>
__global__ void __launch_bounds__(Q_THREADS) k_quant(RankArgs a)
{
    extern __shared__ __align__(16) unsigned int lds[];
    __shared__ unsigned int s_valid, s_cnt, s_last;
    __shared__ RankShared s_end;
    const int tid = threadIdx.x, B = blockDim.x;
    const RankState *cs = a.st;
    int shift = 20, width = 12, w2 = 0, w3 = 0, slots = 1, t2_bytes = 0, t3_bytes = 0, wide = 0;
    bool collect = false, from_cand = false;
    if (NL > 0) {
        if (cs->done) return;
        shift = cs->shift;
        width = cs->width;
        w2 = cs->w2;
        w3 = cs->w3;
        slots = cs->slots;
        t2_bytes = cs->t2_bytes;
        t3_bytes = cs->t3_bytes;
        wide = cs->wide;
        collect = NL < 3 && cs->collect == NL;
        from_cand = NL > 1 && cs->collect == NL - 1 && cs->overflow == 0u;
    }
    const int nbins = 1 << width;
    const int tab_words = NL == 0 ? 0 : (4096 + (NL >= 2 ? t2_bytes : 0) +
                                         (NL >= 3 ? t3_bytes : 0)) / 4;
    const int clog = qp_copies_log2(slots, width, tab_words * 4, a.max_clog, a.lds_bytes);
    const int words = (slots * nbins) << clog;
    for (int i = tid; i < words; i += B) lds[i] = 0u;
    // The tables follow the histograms in LDS (all sizes are multiples of 4).
    unsigned int *tw = lds + words;
    const unsigned int *src = (const unsigned int *)a.tab;
    for (int i = tid; i < tab_words; i += B) tw[i] = src[i];
    if (tid == 0) {
        s_valid = 0u;
        s_cnt = 0u;
    }
    __syncthreads();

    QuantStep<NL> st;
    st.lds = lds;
    st.t1 = (const unsigned char *)tw;
    st.t2 = st.t1 + 4096;
    st.t3 = st.t2 + t2_bytes;
    st.shift = shift;
    st.w2 = w2;
    st.w3 = w3;
    st.wb = width;
    st.bmask = (unsigned int)nbins - 1u;
    st.clog = clog;
    // A prefix's row is its table entry less one.
    st.cbase = (tid & 63 & ((1 << clog) - 1)) - (NL == 0 ? 0 : nbins << clog);
    st.valid = 0u;
    st.collect = collect;
    st.cand = a.cand + (size_t)blockIdx.x * a.cand_cap;
    st.cand_cap = a.cand_cap;
    st.s_cnt = &s_cnt;
    if (NL > 1 && from_cand) {
        // The voxels that the pass before copied to this block's region.
        const unsigned int n = a.cand_n[blockIdx.x];
        for (unsigned int i0 = 0; i0 < n; i0 += 4u * (unsigned int)B) {
            float x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned int i = i0 + (unsigned int)(k * B + tid);
                x[k] = i < n ? st.cand[i] : qnan();
            }
            st(x);
        }
    } else {
        scan_box<PACKED>(a.g, st, a.claim);
    }
    // Every lane of a wavefront holds the same count (sums of ballots).
    if (NL == 0 && (tid & 63) == 0 && st.valid) atomicAdd(&s_valid, st.valid);
    __syncthreads();
    // Flush the histograms.
    const int C = 1 << clog;
    for (int b = tid; b < slots * nbins; b += B) {
        unsigned int sum = 0;
        for (int c = 0; c < C; ++c) sum += lds[(b << clog) + ((c + tid) & (C - 1))];
        if (sum) atomicAdd(&a.acc[b], (unsigned long long)sum);
    }
    if (tid == 0) {
        if (NL == 0 && s_valid) atomicAdd(&a.acc[Q_ACC], (unsigned long long)s_valid);
        if (NL > 0 && collect) {
            a.cand_n[blockIdx.x] = min(s_cnt, a.cand_cap);
            if (s_cnt > a.cand_cap) atomicOr(&a.st->overflow, 1u);
        }
    }
    // The last block reads atomics only (what is copied out and the copied
    // counts are the next launch's), so no block writes its L2 back.
    if (!last_to_arrive_wt(a.ticket, gridDim.x, &s_last)) return;
    if (tid == 0) {
        *a.ticket = 0u;
        if (a.claim.nc) *a.claim.ctr = 0u;
    }
    rank_end<NL>(a, s_end, lds, shift, width, slots, wide, w2, w3);
}

}  // namespace
}  // namespace cube

#include "cube_bracket.h"

namespace cube {
namespace {

template <int NL>
const void *quant_kernel(bool packed)
{
    return packed ? reinterpret_cast<const void *>(&k_quant<NL, true>)
                  : reinterpret_cast<const void *>(&k_quant<NL, false>);
}

struct QuantWorkspace {
    unsigned long long *acc = nullptr;  // Q_ACC counters, the valid counter
    unsigned int *ticket = nullptr;     // the ticket and the chunk counter
    unsigned char *tab = nullptr;       // the prefix tables
    RankState *st = nullptr;
    float *cand = nullptr;              // copied voxels (null: none could be allocated)
    unsigned int *cand_n = nullptr;     // voxels in each block's region, or piece
    BracketState *br = nullptr;
    RankOut *h_out = nullptr, *d_out = nullptr;  // pinned; as the device sees it
    unsigned int calls = 0;
};

constexpr int Q_MAX_BLOCKS = 4096;
constexpr unsigned int BR_PIECES = CAND_TOTAL / BR_PIECE;

std::mutex g_qmu;
QuantWorkspace g_qws[64];
bool g_qws_ready[64];

void free_quant(QuantWorkspace &w)
{
    hipFree(w.acc);
    hipFree(w.ticket);
    hipFree(w.tab);
    hipFree(w.st);
    hipFree(w.cand);
    hipFree(w.cand_n);
    hipFree(w.br);
    hipHostFree(w.h_out);
    w = QuantWorkspace();
}

int quant_ws(QuantWorkspace **out)
{
    int dev = 0;
    hipGetDevice(&dev);
    if (dev < 0 || dev >= 64) return fail(CUBE_EINVAL, "device index out of range");
    if (!g_qws_ready[dev]) {
        QuantWorkspace &w = g_qws[dev];
        hipError_t e;
        if ((e = hipMalloc(&w.acc, (Q_ACC + 2) * 8)) != hipSuccess ||
            (e = hipMalloc(&w.ticket, 256)) != hipSuccess ||
            (e = hipMalloc(&w.tab, Q_TAB)) != hipSuccess ||
            (e = hipMalloc(&w.st, sizeof(RankState))) != hipSuccess ||
            (e = hipMalloc(&w.cand_n, std::max<size_t>(Q_MAX_BLOCKS, BR_PIECES) * 4)) !=
                hipSuccess ||
            (e = hipMalloc(&w.br, sizeof(BracketState))) != hipSuccess ||
            (e = hipHostMalloc(&w.h_out, sizeof(RankOut),
                               hipHostMallocMapped | hipHostMallocCoherent)) != hipSuccess ||
            (e = hipHostGetDevicePointer((void **)&w.d_out, w.h_out, 0)) != hipSuccess ||
            (e = hipMemset(w.acc, 0, (Q_ACC + 2) * 8)) != hipSuccess ||
            (e = hipMemset(w.ticket, 0, 256)) != hipSuccess ||
            (e = hipDeviceSynchronize()) != hipSuccess) {
            free_quant(w);
            return hip_fail(e, "quantile workspace");
        }
        if (hipMalloc(&w.cand, (size_t)CAND_TOTAL * 4) != hipSuccess) {
            (void)hipGetLastError();
            w.cand = nullptr;  // the third pass then reads the box
        }
        w.h_out->done = 0u;
        g_qws_ready[dev] = true;
    }
    *out = &g_qws[dev];
    return CUBE_OK;
}

int rank_launch(const void *k, const RankArgs &a, int blocks, size_t lds)
{
    hipError_t e;
    if (lds > 64 * 1024 &&
        (e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
            hipSuccess)
        return hip_fail(e, "quantile LDS");
    RankArgs copy = a;
    copy.lds_bytes = (uint32_t)lds;
    void *args[] = {&copy};
    if ((e = hipLaunchKernel(k, dim3((unsigned)blocks), dim3(Q_THREADS), args, lds, nullptr)) !=
        hipSuccess)
        return hip_fail(e, "quantile launch");
    return CUBE_OK;
}

// The least box for the single-read search: its five passes cost about 65 us
// beside the read (median of 2^24 voxels 81 us against the two reads' 68, of
// 2^25 93 against 92, of 2^26 110 against 134).
constexpr uint64_t BRACKET_MIN_VOXELS = (uint64_t)3 << 24;

// The voxels to sample for the single-read search of box b; 0: read it twice.
// 5 sigma either side of a rank is 5 / sqrt(sample) of the box, and the
// copies have to fit (up to 2^32 voxels they do).  Four times the sample takes
// 20 us more and leaves half the copies: median of 2^28 voxels 252 us against
// 257, of 2^30 769 against 817, of 2^26 133 against 110.
unsigned int sample_of(const Box &b, const QuantWorkspace &w)
{
    if (!w.cand || b.n < BRACKET_MIN_VOXELS) return 0u;
    for (int lg = b.n < ((uint64_t)1 << 29) ? 18 : 20; lg <= 22; lg += 2)
        if (5.0 * (double)b.n / (double)(1u << (lg / 2)) < 0.65 * CAND_TOTAL) return 1u << lg;
    return 0u;
}

// The median, one rank or one level in a single read of the box; status
// RANK_MISSED if the box has to be read again.
int run_bracket(const Box &box, unsigned int n_sample, int mode, uint64_t rank, double level,
                QuantWorkspace *w, std::vector<unsigned int> *keys, uint64_t *n_valid, int *status)
{
    BracketArgs a;
    memset(&a, 0, sizeof a);
    a.st = w->br;
    a.acc = w->acc;
    a.totals = w->acc + Q_ACC;
    a.ticket = w->ticket;
    a.cand = w->cand;
    a.piece_n = w->cand_n;
    a.n_pieces = BR_PIECES;
    a.n_sample = n_sample;
    a.stride = (unsigned int)(box.n / n_sample);
    a.mode = mode;
    a.rank = rank;
    a.level = level;
    a.out = w->d_out;
    if (++w->calls == 0u) w->calls = 1u;
    a.gen = w->calls;
    const int cl = std::max(chunk_override(), 0);
    // One block of 16 wavefronts on each CU: every block adds its totals, its
    // bins and its ticket to the same few words, so with three blocks of 8
    // the read of 2^23 voxels took 29 us against 19.  Static unless the caller
    // asked for chunks: a region of 941 x 937 x 240 took 237 us, with 2^18-voxel
    // chunks 270.
    // Two for rows under four voxels, which are visited one after the other.
    long long blocks = cu_count() * (thin_rows(box) ? 2 : 1);
    long long units = blocks;
    if (cl) {
        units = chunks_of(box.n, cl);
        if (blocks > units) blocks = units;
        a.claim.nc = (int)units;
    }
    a.claim.ctr = w->ticket + CHUNK_CTR_WORD;
    a.waves = (unsigned int)blocks * (BR_READ_THREADS / 64);
    scan_geom(box, units, BR_READ_THREADS, &a.g);
    const void *read = a.g.pack.cb > 0
                           ? reinterpret_cast<const void *>(&k_bracket<BR_BOX, true>)
                           : reinterpret_cast<const void *>(&k_bracket<BR_BOX, false>);
    const struct { const void *k; long long blocks; int threads; } passes[] = {
        {reinterpret_cast<const void *>(&k_bracket<BR_SAMPLE, false>), BR_SAMPLE_BLOCKS, BR_THREADS},
        {reinterpret_cast<const void *>(&k_bracket<BR_SAMPLED, false>), BR_SAMPLE_BLOCKS, BR_THREADS},
        {read, blocks, BR_READ_THREADS},
        {reinterpret_cast<const void *>(&k_bracket<BR_COPIED, false>), cu_count(), BR_THREADS},
        {reinterpret_cast<const void *>(&k_bracket<BR_COPIED, false>), cu_count(), BR_THREADS}};
    void *args[] = {&a};
    hipError_t e;
    for (const auto &p : passes)
        if ((e = hipLaunchKernel(p.k, dim3((unsigned)p.blocks), dim3((unsigned)p.threads), args, 0,
                                 nullptr)) != hipSuccess)
            return hip_fail(e, "rank launch");
    if ((e = poll_host(&w->h_out->done, a.gen)) != hipSuccess) return hip_fail(e, "rank result");
    const RankOut &o = *w->h_out;
    *n_valid = o.n_valid;
    *status = o.status;
    if (!o.status) {
        g_rank_route = CUBE_RANK_BRACKET;
        keys->assign(o.key, o.key + o.m);
    }
    return CUBE_OK;
}

// Queue the passes on the null stream and wait for the result.  `keys`: the
// keys of the ranks, ascending; `missed`: CUBE_RANK_MISSED after a single read.
int run_passes(const Box &box, int mode, uint64_t rank, const double *q, int nq,
               int missed, QuantWorkspace *w, std::vector<unsigned int> *keys, uint64_t *n_valid,
               int *status, int *wide)
{
    RankArgs a;
    memset(&a, 0, sizeof a);
    a.st = w->st;
    a.tab = w->tab;
    a.acc = w->acc;
    a.ticket = w->ticket;
    a.cand = w->cand;
    a.cand_n = w->cand_n;
    a.mode = mode;
    a.rank = rank;
    a.nq = nq;
    for (int i = 0; i < nq; ++i) a.q[i] = q[i];
    a.out = w->d_out;
    if (++w->calls == 0u) w->calls = 1u;
    a.gen = w->calls;
    // One resident wave of blocks, one per CU (the refinement passes take
    // nearly all of a CU's LDS), fewer for small boxes, where clearing and
    // adding up a block's histograms costs more than its share of the scan;
    // for the same reason fewer LDS copies of each.
    // Rows under four voxels are visited one after the other, each at the
    // latency of its loads: two blocks per CU (median of a spectrum of 1000
    // channels of one pixel, by one block 1207 us, by 512 70 us).
    const int cl = scan_chunk_log2(box);
    long long blocks = cu_count();
    if (cl == 0 && thin_rows(box)) {
        blocks = std::min(2 * blocks, thin_rows(box));
    } else if (cl == 0) {
        const long long root = (long long)sqrt((double)box.n) / 16;
        blocks = root < 1 ? 1 : (root < blocks ? root : blocks);
    }
    long long units = blocks;
    if (cl) {
        units = chunks_of(box.n, cl);
        if (blocks > units) blocks = units;
        a.claim.nc = (int)units;
    }
    a.claim.ctr = w->ticket + CHUNK_CTR_WORD;
    a.cand_cap = CAND_TOTAL / (unsigned int)blocks;
    a.max_clog = box.n < ((uint64_t)1 << 22) ? 1 : (box.n < ((uint64_t)1 << 25) ? 2 : 3);
    scan_geom(box, units, Q_THREADS, &a.g);
    const bool packed = a.g.pack.cb > 0;
    const int passes = qp_wide(2 * nq, 2 * nq) ? 3 : 4;  // few ranks are always "wide"
    const size_t lds0 = (size_t)4096 * 4 << a.max_clog;
    int rc;
    if ((rc = rank_launch(quant_kernel<0>(packed), a, (int)blocks, lds0)) ||
        (rc = rank_launch(quant_kernel<1>(packed), a, (int)blocks, Q_LDS)) ||
        (rc = rank_launch(quant_kernel<2>(packed), a, (int)blocks, Q_LDS)) ||
        (passes == 4 && (rc = rank_launch(quant_kernel<3>(packed), a, (int)blocks, Q_LDS))))
        return rc;
    const hipError_t e = poll_host(&w->h_out->done, a.gen);
    if (e != hipSuccess) return hip_fail(e, "quantile result");
    const RankOut &o = *w->h_out;
    *n_valid = o.n_valid;
    *status = o.status;
    if (o.status) return CUBE_OK;
    *wide = o.wide;
    g_rank_route = missed | o.route;
    keys->assign(o.key, o.key + o.m);
    return CUBE_OK;
}

// The ranks' keys by the route that suits the box.
int run_ranks(const Box &box, int mode, uint64_t rank, const double *q, int nq,
              std::vector<unsigned int> *keys, uint64_t *n_valid, int *status, int *wide)
{
    QuantWorkspace *w = nullptr;
    int rc = quant_ws(&w);
    if (rc) return rc;
    const unsigned int n_sample = nq > 1 ? 0u : sample_of(box, *w);
    if (n_sample) {
        *wide = 1;
        rc = run_bracket(box, n_sample, mode, rank, nq ? q[0] : 0.0, w, keys, n_valid, status);
        if (rc || *status != RANK_MISSED) return rc;
    }
    return run_passes(box, mode, rank, q, nq, n_sample ? CUBE_RANK_MISSED : 0, w, keys, n_valid, status, wide);
}

}  // namespace

int box_ranks(const Box &b, int median, uint64_t rank, float *v, int *n_v, uint64_t *n_valid)
{
    std::lock_guard<std::mutex> lk(g_qmu);
    std::vector<unsigned int> keys;
    int status = 0, wide = 0;
    uint64_t n = 0;
    const int rc = run_ranks(b, median ? RANK_MEDIAN : RANK_GIVEN, rank, nullptr, 0, &keys, &n,
                             &status, &wide);
    if (rc) return rc;
    *n_valid = n;
    if (status == 1)
        return fail(CUBE_EINVAL, "rank %llu >= %llu valid voxels", (unsigned long long)rank,
                    (unsigned long long)n);
    if (status) return fail(CUBE_EINVAL, "no valid voxel");
    *n_v = (int)keys.size();
    for (size_t i = 0; i < keys.size(); ++i) v[i] = qp_key_to_float(keys[i]);
    return CUBE_OK;
}

void quant_release()
{
    std::lock_guard<std::mutex> lk(g_qmu);
    int cur = 0;
    hipGetDevice(&cur);
    for (int d = 0; d < 64; ++d) {
        if (!g_qws_ready[d]) continue;
        hipSetDevice(d);
        hipDeviceSynchronize();
        free_quant(g_qws[d]);
        g_qws_ready[d] = false;
    }
    hipSetDevice(cur);
}

}  // namespace cube

using namespace cube;

extern "C" {

int cube_quantiles(const float *ptr, const int64_t *dims, const double *q, int32_t m,
                   double *out, uint64_t *n_valid)
{
    CUBE_GUARD_BEGIN
    if (!q || !out) return fail(CUBE_EINVAL, "q or out is NULL");
    if (m < 1 || m > CUBE_MAX_QUANTILES)
        return fail(CUBE_EINVAL, "m=%d outside [1, %d]", m, CUBE_MAX_QUANTILES);
    for (int i = 0; i < m; ++i)
        if (!(q[i] >= 0.0 && q[i] <= 1.0))
            return fail(CUBE_EINVAL, "level q[%d] outside [0, 1]", i);
    Box b;
    int rc = check_box(ptr, dims, &b);
    if (!rc) rc = check_box_device(&b);
    if (rc) return rc;
    if (b.n == 0) {
        if (n_valid) *n_valid = 0;
        return fail(CUBE_EINVAL, "empty box");
    }
    std::lock_guard<std::mutex> lk(g_qmu);
    std::vector<unsigned int> keys;
    uint64_t n = 0;
    int status = 0, wide = 0;
    if ((rc = run_ranks(b, RANK_LEVELS, 0, q, m, &keys, &n, &status, &wide))) return rc;
    if (n_valid) *n_valid = n;
    if (status) return fail(CUBE_EINVAL, "no valid voxel");
    const std::vector<unsigned long long> ranks = qp_ranks(q, m, n);
    if (ranks.size() != keys.size()) return fail(CUBE_EDEVICE, "quantile ranks disagree");
    for (int i = 0; i < m; ++i) {
        const double h = q[i] * (double)(n - 1);
        const double j = floor(h);
        const double f = h - j;
        const double lo = qp_key_to_float(keys[qp_index(ranks, (unsigned long long)j)]);
        const double hi =
            f > 0.0 ? qp_key_to_float(keys[qp_index(ranks, (unsigned long long)j + 1)]) : lo;
        out[i] = qp_interpolate(lo, hi, f);
    }
    g_quant_reads = wide ? 3 : 4;
    return CUBE_OK;
    CUBE_GUARD_END
}

int cube_last_quantile_reads(void) { return g_quant_reads; }

int cube_last_rank_route(void) { return g_rank_route; }

}  // extern "C"
