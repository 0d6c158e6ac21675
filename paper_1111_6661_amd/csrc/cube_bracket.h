// cube_bracket.h -- one rank, the two middle ranks or those of one quantile
// level of a large box in one read (included by cube_quantile.hip).
//
// A sample of the box (one voxel out of each of 2^18 or more equal strides)
// gives a bracket of keys that holds the wanted ranks unless the sample is
// 5 sigma off: about 1 % of the box.  One read then counts the valid voxels
// and those below the bracket, bins the bracket's into 256 bins of their key,
// and copies them out; two more passes find the remaining key bits in the
// copies.  All of it is exact: the counts of the full read say whether the
// ranks do lie in the bracket, and if they don't, or the copies don't fit, the
// caller goes on with the passes over the box (status RANK_MISSED).  A bracket
// of at most 512 keys (a value held by many voxels) needs no copies.
//
// Five launches, queued at once; each pass's last block finds the bins of the
// ranks and lays out the next pass.
//
// Measured (median, microseconds; before: two reads, by cube_quantile.hip): of
// 2^28 voxels 370 -> 257, of a 941 x 937 x 240 box 362 -> 237; one quantile level
// the same.  About 65 us
// are the five passes' ends and the sample; the read reaches 5.6 TB/s, bound by
// the issue of some 75 instructions for 4 voxels of each lane (loads a tile
// ahead, or more wavefronts, change nothing).
#pragma once

#include "cube_scan.h"

namespace cube {
namespace {

constexpr int BR_SAMPLE_BLOCKS = 128;
constexpr int BR_BINS_LOG2 = 12;   // bits of a pass, but for the read of the box
// Bits the read of the box bins: every block adds its bins to the global ones
// (at about 23 G atomics/s), so few; the copies' passes have 12 bits each for
// the other 24.
constexpr int BR_BOX_LOG2 = 8;
constexpr int BR_BOX_ALL = 9;      // a bracket of at most 2^9 keys is binned whole: both zeros' groups
// The copied voxels' room is handed out in pieces, to a wavefront as it fills
// the one before: a box whose wanted voxels lie together fits as any other
// does (a region for each block would not hold them).  Every wavefront has
// its first piece from the start: claims of 12288 at once of one counter took
// 80 us.
constexpr unsigned int BR_PIECE = 512;       // a multiple of 64
constexpr int BR_THREADS = 1024, BR_READ_THREADS = 1024;
constexpr int BR_WORDS = 2 << BR_BINS_LOG2;  // LDS counters: two prefixes' histograms

enum { BR_SAMPLE = 0, BR_SAMPLED = 1, BR_BOX = 2, BR_COPIED = 3 };

struct BracketState {
    int over;                      // the result (or a miss) has been written
    int m;                         // ranks: 1 or 2, ascending
    unsigned long long rank[2];    // rank left inside the prefix found so far
    unsigned int pre[2];           // that prefix: the bits above the next pass's
    unsigned int base;             // keys are taken relative to this
    int shift, width;              // the next pass bins bits [shift, shift + width)
    int open;                      // bit 0 (1): no lower (upper) bound from the sample
    unsigned long long span;       // sample ranks from the lower to the upper bound
    float lo, hi;                  // the bracket
    int collect;
    unsigned int pieces;           // handed out beyond the first; too many: copies were lost
};

struct BracketArgs {
    Geom g;
    Claim claim;
    BracketState *st;
    unsigned long long *acc;       // BR_WORDS counters; zero between passes
    unsigned long long *totals;    // valid voxels, voxels below; zero between passes
    unsigned int *ticket;
    float *cand;                   // the sample; then the pieces of copied voxels
    unsigned int *piece_n;         // voxels in each
    unsigned int n_pieces;
    unsigned int waves;            // of the read of the box
    unsigned int n_sample, stride;
    int32_t mode;                  // RANK_*: a rank, the median or one level
    unsigned long long rank;       // RANK_GIVEN
    double level;                  // RANK_LEVELS: ranks floor(level (n - 1)) and the next
    RankOut *out;
    unsigned int gen;
};

template <int SRC>
struct BracketStep {
    const BracketArgs &a;
    unsigned int *hist;
    unsigned int base, bmask, pre0, pre1;
    int shift, width, top, clog, cbase;
    float lo, hi;
    unsigned int seen, blank, below;  // voxels, by this wavefront
    bool collect;
    unsigned int piece, used;         // this wavefront's piece (n_pieces: none left), its voxels
    float *buf;                       // LDS: 127 voxels not yet written out
    unsigned int fill;

    // NV (1 or 4) voxels per lane of the box.
    template <int NV>
    __device__ __forceinline__ void read(const float (&x)[NV])
    {
        // Blanks are rare: two voxels are tested by one compare.
        unsigned long long un = 0ull;
#pragma unroll
        for (int j = 0; j < NV; j += 2)
            un |= __builtin_amdgcn_ballot_w64(__builtin_isunordered(x[j], x[NV > 1 ? j + 1 : j]));
        seen += 64u * NV;
        if (un) {
#pragma unroll
            for (int j = 0; j < NV; ++j)
                blank += (unsigned int)__popcll(__builtin_amdgcn_ballot_w64(x[j] != x[j]));
        }
        bool in[NV], any = false;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const bool less = x[j] < lo;
            below += (unsigned int)__popcll(__builtin_amdgcn_ballot_w64(less));
            in[j] = x[j] <= hi && !less;
            any = any || in[j];
        }
        // The wanted voxels, each lane's first, then its second, ...: mostly
        // one step for all four.
        unsigned long long m = __builtin_amdgcn_ballot_w64(any);
        while (m) {
            float v = x[NV - 1];
#pragma unroll
            for (int j = NV - 2; j >= 0; --j) v = in[j] ? x[j] : v;
            if (any)
                atomicAdd(&hist[(((order_key(v) - base) >> shift) << clog) + cbase], 1u);
            if (collect) copy_out(v, any, m);
            bool before = false;
            any = false;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const bool now = in[j];
                in[j] = now && before;
                before = before || now;
                any = any || in[j];
            }
            m = __builtin_amdgcn_ballot_w64(any);
        }
    }

    // The wavefront's copies gather in LDS and leave 64 at a time: written as
    // they came, a few lanes to a store, they took 60 us of 2^28 voxels.
    __device__ __forceinline__ void copy_out(float v, bool in, unsigned long long m)
    {
        const unsigned int i = __builtin_amdgcn_mbcnt_hi(
            (unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
        if (in) buf[fill + i] = v;
        fill += (unsigned int)__popcll(m);
        if (fill >= 64u) {
            write_out(64u);
            const unsigned int lane = threadIdx.x & 63;
            const float rest = buf[64u + lane];  // below 128
            fill -= 64u;
            if (lane < fill) buf[lane] = rest;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    __device__ __forceinline__ void write_out(unsigned int n)
    {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const unsigned int lane = threadIdx.x & 63;
        if (used == BR_PIECE) {
            unsigned int id = 0;
            if (lane == 0) {
                if (piece < a.n_pieces) a.piece_n[piece] = BR_PIECE;
                id = a.waves + atomicAdd(&a.st->pieces, 1u);
            }
            piece = min((unsigned int)__builtin_amdgcn_readfirstlane((int)id), a.n_pieces);
            used = 0u;
        }
        if (lane < n && piece < a.n_pieces)
            a.cand[(size_t)piece * BR_PIECE + used + lane] = buf[lane];
        used += n;
    }

    template <int NV>
    __device__ __forceinline__ void operator()(const float (&x)[NV])
    {
        if constexpr (SRC == BR_BOX) {
            // Four voxels at a time: the masks of sixteen spilled, and a branch
            // for every voxel took 250 us where 2^28 voxels are read in 150.
#pragma unroll
            for (int j = 0; j < NV; j += 4) {
                float part[NV < 4 ? NV : 4];
#pragma unroll
                for (int k = 0; k < (NV < 4 ? NV : 4); ++k) part[k] = x[j + k];
                read(part);
            }
        } else {
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const bool ok = x[j] == x[j];
                if (SRC == BR_SAMPLE)
                    seen += (unsigned int)__popcll(__builtin_amdgcn_ballot_w64(ok));
                const unsigned int d = order_key(x[j]) - base;
                const unsigned int p = (d >> (top - 1)) >> 1;  // top is 1 .. 32
                const unsigned int slot = p == pre0 ? 0u : 1u;
                if (ok && (p == pre0 || p == pre1))
                    atomicAdd(&hist[(((slot << width) | ((d >> shift) & bmask)) << clog) + cbase],
                              1u);
            }
        }
    }
};

struct BracketShared {
    unsigned long long rank[2], left[2], count[2], wave[MAX_WAVES], total;
    unsigned int pre[2], bin[2];
    unsigned long long nv, below;
    int m, over;
};

// The next pass's layout, or the result (thread 0 of the last block).
template <int SRC>
__device__ __forceinline__ void bracket_next(const BracketArgs &a, BracketShared &s, int shift,
                                             int width)
{
    BracketState *st = a.st;
    const int m = s.m;
    if (SRC == BR_BOX && s.rank[m - 1] >= s.total) s.over = RANK_MISSED;
    if (!s.over) {
        for (int i = 0; i < m; ++i) {
            s.pre[i] = (s.pre[i] << width) | s.bin[i];
            st->rank[i] = s.left[i];
        }
        if (m == 1) s.pre[1] = s.pre[0];
        int next = shift > BR_BINS_LOG2 ? shift - BR_BINS_LOG2 : 0, bits = shift - next;
        unsigned int pre0 = s.pre[0], pre1 = s.pre[1];
        if (SRC == BR_SAMPLE) {
            next = 8;
            bits = 12;
            st->base = 0u;
        } else if (SRC == BR_SAMPLED) {
            // The bracket: whole groups of 256 keys, within the infinities.
            // It is tested on the values, where -0 is +0, so it holds both
            // zeros or neither.
            unsigned int klo = pre0 << 8, khi = (pre1 << 8) | 255u;
            if ((st->open & 1) || klo < 0x007fffffu) klo = 0x007fffffu;
            if ((st->open & 2) || khi > 0xff800000u) khi = 0xff800000u;
            if (klo == 0x80000000u) klo = 0x7fffffffu;
            if (khi == 0x7fffffffu) khi = 0x80000000u;
            const unsigned int range = khi - klo;
            const int w = range ? 32 - __builtin_clz(range) : 1;
            st->lo = __uint_as_float(klo & 0x80000000u ? klo ^ 0x80000000u : ~klo);
            st->hi = __uint_as_float(khi & 0x80000000u ? khi ^ 0x80000000u : ~khi);
            st->base = klo;
            bits = w <= BR_BOX_ALL ? w : BR_BOX_LOG2;
            next = w - bits;
            st->collect = next > 0 ? 1 : 0;
            st->pieces = 0u;
            // The voxels to copy, by the sample, and half a piece lost at
            // each wavefront's end; with many in one group of keys they may
            // be too many.
            const double share = (double)(st->span + s.count[0] + s.count[1]) / a.n_sample;
            if (next > 0 && share * (double)a.g.n_total + 0.5 * BR_PIECE * a.waves >
                                0.95 * BR_PIECE * a.n_pieces)
                s.over = RANK_MISSED;
            pre0 = pre1 = 0u;
        } else if (SRC == BR_BOX) {
            store_result<true>(&a.out->n_valid, s.nv);
        }
        if (SRC >= BR_BOX && shift == 0) {
            store_result<true>(&a.out->key[0], st->base + pre0);
            store_result<true>(&a.out->key[1], st->base + pre1);
            store_result<true>(&a.out->m, m);
            store_result<true>(&a.out->wide, 1);
            store_result<true>(&a.out->status, 0);
            s.over = -1;
        }
        st->m = m;
        st->shift = next;
        st->width = bits;
        st->pre[0] = pre0;
        st->pre[1] = pre1;
    }
    if (s.over > 0) store_result<true>(&a.out->status, s.over);
    st->over = s.over;
}

// The last block's part of a pass.
template <int SRC>
__device__ __forceinline__ void bracket_end(const BracketArgs &a, BracketShared &s, int shift,
                                            int width)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, B = blockDim.x;
    BracketState *st = a.st;
    if (tid == 0) {
        s.over = 0;
        s.nv = s.below = 0ull;
        if (SRC == BR_SAMPLE || SRC == BR_BOX) {
            s.nv = a.totals[0];
            s.below = a.totals[1];
            a.totals[0] = a.totals[1] = 0ull;
            s.pre[0] = s.pre[1] = 0u;
        } else {
            s.m = st->m;
            for (int i = 0; i < 2; ++i) {
                s.rank[i] = st->rank[i];
                s.pre[i] = st->pre[i];
            }
        }
        if (SRC == BR_SAMPLE) {
            // The sample ranks 5 standard deviations (of a binomial count)
            // either side of the wanted ones; 16 more for small counts.
            const double v = (double)s.nv;
            const double of = a.mode == RANK_GIVEN ? (double)a.n_sample : v;
            const double c =
                a.mode == RANK_GIVEN
                    ? (double)a.rank * ((double)a.n_sample / (double)a.g.n_total)
                    : (a.mode == RANK_MEDIAN ? 0.5 : a.level) * (v - 1.0);
            const double half = 5.0 * sqrt(fmax(c * (1.0 - c / of), 0.0)) + 16.0;
            const double lo = floor(c - half), hi = ceil(c + half);
            st->open = (lo < 0.0 ? 1 : 0) | (hi >= v ? 2 : 0);
            s.m = 2;
            s.rank[0] = lo < 0.0 ? 0ull : (lo >= v ? s.nv - 1ull : (unsigned long long)lo);
            s.rank[1] = hi >= v ? s.nv - 1ull : (unsigned long long)hi;
            st->span = s.rank[1] - s.rank[0];
            if (s.nv < 1024ull) s.over = RANK_MISSED;
        }
        if (SRC == BR_BOX) {
            unsigned long long r = a.mode == RANK_GIVEN ? a.rank : (s.nv - 1ull) / 2ull;
            s.m = a.mode == RANK_MEDIAN && s.nv % 2 == 0 ? 2 : 1;
            if (a.mode == RANK_LEVELS) {
                const double h = a.level * (double)(s.nv - 1ull), j = floor(h);
                r = (unsigned long long)j;
                s.m = h - j > 0.0 ? 2 : 1;
            }
            s.rank[0] = r - s.below;  // huge if below the bracket
            s.rank[1] = r + 1ull - s.below;
            if (r < s.below || s.nv == 0ull ||
                (st->collect && __hip_atomic_load(&st->pieces, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT) > a.n_pieces - a.waves))
                s.over = RANK_MISSED;
        }
    }
    __syncthreads();
    // The bin of each rank in its prefix's histogram; the counters return to
    // zero.
    const int nbins = 1 << width, per = nbins > B ? nbins / B : 1, m = s.m;
    const int slots = s.pre[0] == s.pre[1] ? 1 : 2;
    for (int slot = 0; slot < slots; ++slot) {
        unsigned long long *h = a.acc + (size_t)slot * nbins, c[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[k] = k < per && tid * per + k < nbins ? h[tid * per + k] : 0ull;
            sum += c[k];
        }
        unsigned long long upto = sum;
        wave_reduce(CountStep{upto});
        if (lane == WAVE_LAST) s.wave[wid] = upto;
        __syncthreads();
        for (int w = 0; w < wid; ++w) upto += s.wave[w];
        const unsigned long long before = upto - sum;
        for (int i = 0; i < m; ++i) {
            unsigned long long r = s.rank[i];
            if ((slots == 1 || i == slot) && r >= before && r < upto) {  // one thread
                r -= before;
                int k = 0;
                while (k < per - 1 && c[k] <= r) r -= c[k++];
                s.left[i] = r;
                s.bin[i] = (unsigned int)(tid * per + k);
                s.count[i] = c[k];
            }
        }
        if (tid == B - 1) s.total = upto;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < per && tid * per + k < nbins) h[tid * per + k] = 0ull;
        __syncthreads();
    }
    if (tid == 0) bracket_next<SRC>(a, s, shift, width);
    __syncthreads();
    if (s.over) tell_host(&a.out->done, a.gen);
}

template <int SRC, bool PACKED>
__global__ void __launch_bounds__(SRC == BR_BOX ? BR_READ_THREADS : BR_THREADS)
    k_bracket(BracketArgs a)
{
    __shared__ unsigned int hist[BR_WORDS];
    __shared__ unsigned int s_valid, s_below, s_last;
    __shared__ BracketShared s_end;
    const int tid = threadIdx.x, B = blockDim.x;
    const BracketState *cs = a.st;
    BracketStep<SRC> st = {a};
    st.base = 0u;
    st.shift = 20;
    st.width = 12;
    st.pre0 = st.pre1 = 0u;
    if (SRC != BR_SAMPLE) {
        if (cs->over) return;
        st.base = cs->base;
        st.shift = cs->shift;
        st.width = cs->width;
        st.pre0 = cs->pre[0];
        st.pre1 = cs->pre[1];
    }
    const int slots = st.pre0 == st.pre1 ? 1 : 2;
    int clog = 0;
    while (clog < 3 && (slots << (st.width + clog + 1)) <= BR_WORDS) ++clog;
    for (int i = tid; i < slots << (st.width + clog); i += B) hist[i] = 0u;
    if (tid == 0) s_valid = s_below = 0u;
    __syncthreads();
    st.hist = hist;
    st.bmask = (1u << st.width) - 1u;
    st.top = st.shift + st.width;
    st.clog = clog;
    st.cbase = tid & ((1 << clog) - 1);
    st.seen = st.blank = st.below = 0u;
    st.lo = st.hi = 0.f;
    st.collect = false;
    st.piece = (unsigned int)__builtin_amdgcn_readfirstlane(blockIdx.x * (B >> 6) + (tid >> 6));
    st.used = st.fill = 0u;
    if constexpr (SRC == BR_BOX) {
        st.lo = cs->lo;
        st.hi = cs->hi;
        st.collect = cs->collect != 0;
        __shared__ float s_buf[BR_READ_THREADS / 64][128];
        st.buf = s_buf[tid >> 6];
        scan_box<PACKED>(a.g, st, a.claim);
        if (st.fill) st.write_out(st.fill);
        if ((tid & 63) == 0 && st.piece < a.n_pieces) a.piece_n[st.piece] = st.used;
    } else if constexpr (SRC == BR_COPIED) {
        // Each half of a block reads its own pieces.
        const unsigned int n = min(a.waves + cs->pieces, a.n_pieces), step = 2u * gridDim.x;
        for (unsigned int p0 = 2u * blockIdx.x; p0 < n; p0 += 4u * step) {
            float x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned int p = p0 + (unsigned int)k * step + (unsigned int)(tid >> 9);
                x[k] = p < n && (unsigned int)(tid & 511) < a.piece_n[p]
                           ? a.cand[(size_t)p * BR_PIECE + (tid & 511)] : qnan();
            }
            st(x);
        }
    } else {
        // The sample: each voxel of it read from the box by the first pass.
        const unsigned int n = a.n_sample / gridDim.x;
        float *mine = a.cand + (size_t)blockIdx.x * n;
        for (unsigned int i0 = 0; i0 < n; i0 += 4u * (unsigned int)B) {
            float x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned int i = i0 + (unsigned int)(k * B + tid);
                x[k] = qnan();
                if (i < n) {
                    if (SRC == BR_SAMPLE) {
                        // Voxel `v` of the box: somewhere in the sample's
                        // stride, so that no period of the box is sampled.
                        const unsigned int j = blockIdx.x * n + i;
                        const unsigned long long v =
                            (unsigned long long)j * a.stride +
                            __umulhi(j * 0x9E3779B1u, a.stride);
                        const unsigned long long row = v / (unsigned long long)a.g.row_len;
                        const unsigned long long z = row / (unsigned long long)a.g.ny;
                        x[k] = a.g.ptr[(long long)(v - row * a.g.row_len) +
                                       (long long)(row - z * a.g.ny) * a.g.sy +
                                       (long long)z * a.g.sz];
                    } else {
                        x[k] = mine[i];
                    }
                }
            }
            st(x);
            if (SRC == BR_SAMPLE) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const unsigned int i = i0 + (unsigned int)(k * B + tid);
                    if (i < n) mine[i] = x[k];
                }
            }
        }
    }
    if ((SRC == BR_SAMPLE || SRC == BR_BOX) && (tid & 63) == 0) {
        if (st.seen != st.blank) atomicAdd(&s_valid, st.seen - st.blank);
        if (st.below) atomicAdd(&s_below, st.below);
    }
    __syncthreads();
    for (int b = tid; b < slots << st.width; b += B) {
        unsigned int sum = 0;
        for (int c = 0; c < 1 << clog; ++c) sum += hist[(b << clog) + ((c + tid) & ((1 << clog) - 1))];
        if (sum) atomicAdd(&a.acc[b], (unsigned long long)sum);
    }
    if (tid == 0 && (SRC == BR_SAMPLE || SRC == BR_BOX)) {
        if (s_valid) atomicAdd(&a.totals[0], (unsigned long long)s_valid);
        if (s_below) atomicAdd(&a.totals[1], (unsigned long long)s_below);
    }
    // The last block reads atomics only; the sample and the copies are the
    // next launch's.
    if (!last_to_arrive_wt(a.ticket, gridDim.x, &s_last)) return;
    if (tid == 0) {
        *a.ticket = 0u;
        if (SRC == BR_BOX && a.claim.nc) *a.claim.ctr = 0u;
    }
    bracket_end<SRC>(a, s_end, st.shift, st.width);
}

}  // namespace
}  // namespace cube
