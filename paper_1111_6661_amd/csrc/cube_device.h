// cube_device.h -- device code shared by the single-box and the batched
// kernels of the cube statistics library: the per-voxel step, the scan of a
// box's work units, the wavefront record (local stage), the LDS histogram
// flush and the FP64 merge of records (global stage).
//
// Per voxel:
//   * blank test (x != x), counted with a wavefront ballot on the scalar unit;
//   * min / max of the quieted value (v_min3/v_max3 order -0 before +0 and
//     skip quiet NaNs; a signalling NaN is quieted first);
//   * moments about a per-wavefront pivot K (the first valid voxel the
//     wavefront meets): (x - K)^2 in FP32 over a chunk of at most two tiles,
//     folded into a TwoSum-compensated lane accumulator (Knuth's TwoSum), and
//     the sum of x in FP64.  An FP64 add issues at the rate of an FP32 add;
//     it makes the mean exact to about 1e-15, where FP32 sums of 32 voxels
//     leave it an error of 5e-7 / sqrt(n) standard deviations (400 boxes of
//     2^17 to 2^26 noise voxels);
//   * the histogram bin min(nbins-1, floor((x - lo) * scale)) in FP32 (two
//     rounded operations, then v_cvt_flr_i32_f32), counted in LDS
//     sub-histograms interleaved per lane; blank and out-of-range voxels go
//     to a dummy slot and are counted with ballots instead.
#pragma once

#include <math.h>

#include <type_traits>

#include "cube_internal.h"

namespace cube {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // any voxel's address

constexpr int MAX_WAVES = 16;   // 1024 threads per block at most

__device__ __forceinline__ int cvt_flr_i32(float u)
{
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(u));
    return r;
}

__device__ __forceinline__ float qnan() { return __int_as_float(0x7fc00000); }

// s + c += x with the rounding error of s + x kept in c (TwoSum).
__device__ __forceinline__ void two_sum_acc(float &s, float &c, float x)
{
    const float t = s + x;
    const float bp = t - s;
    const float e = (s - (t - bp)) + (x - bp);
    s = t;
    c += e;
}

// (ah, al) += (bh, bl), double-float addition.
__device__ __forceinline__ void df_add(float &ah, float &al, float bh, float bl)
{
    const float s = ah + bh;
    const float bp = s - ah;
    float e = (ah - (s - bp)) + (bh - bp);
    e += al + bl;
    ah = s + e;
    al = e - (ah - s);
}

// A value from another lane of the wavefront by a DPP move (lanes without a
// source, or in rows outside RM, get `none`): a reduction step costs a few
// cycles where a shuffle through LDS (ds_bpermute) costs about sixty.
template <int CTRL, int RM>
__device__ __forceinline__ int dpp(int none, int x)
{
    return __builtin_amdgcn_update_dpp(none, x, CTRL, RM, 0xf, false);
}
template <int CTRL, int RM>
__device__ __forceinline__ float dpp(float none, float x)
{
    return __int_as_float(dpp<CTRL, RM>(__float_as_int(none), __float_as_int(x)));
}
template <int CTRL, int RM>
__device__ __forceinline__ unsigned long long dpp(unsigned long long none, unsigned long long x)
{
    const unsigned int lo = (unsigned int)dpp<CTRL, RM>((int)(unsigned int)none, (int)(unsigned int)x);
    const unsigned int hi = (unsigned int)dpp<CTRL, RM>((int)(none >> 32), (int)(x >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
template <int CTRL, int RM>
__device__ __forceinline__ double dpp(double none, double x)
{
    return __longlong_as_double((long long)dpp<CTRL, RM>(
        (unsigned long long)__double_as_longlong(none), (unsigned long long)__double_as_longlong(x)));
}

// Combine the lanes of a row of 16, or of the wavefront, in a fixed order:
// step(ctrl, rows) folds the value a DPP move brings into each lane.  The
// result is in the last lane of each row (ROW_LAST), or in lane 63.
constexpr int ROW_LAST = 15, WAVE_LAST = 63;
template <class Step>
__device__ __forceinline__ void row_reduce(Step step)
{
    step(std::integral_constant<int, 0x111>(), std::integral_constant<int, 0xf>());  // row_shr:1
    step(std::integral_constant<int, 0x112>(), std::integral_constant<int, 0xf>());
    step(std::integral_constant<int, 0x114>(), std::integral_constant<int, 0xf>());
    step(std::integral_constant<int, 0x118>(), std::integral_constant<int, 0xf>());
}
template <class Step>
__device__ __forceinline__ void wave_reduce(Step step)
{
    row_reduce(step);
    step(std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xa>());  // row_bcast:15
    step(std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xc>());  // row_bcast:31
}

__device__ __forceinline__ unsigned long long from_lane(unsigned long long x, int l)
{
    const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)x, l);
    const unsigned int hi = (unsigned int)__builtin_amdgcn_readlane((int)(x >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ double from_lane(double x, int l)
{
    return __longlong_as_double(
        (long long)from_lane((unsigned long long)__double_as_longlong(x), l));
}
__device__ __forceinline__ float from_lane(float x, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// How a pass sums x: CUBE_ACCUM_FP64MERGE in FP64 per voxel; CUBE_ACCUM_NAIVE32
// in FP32; ACC_FP32_SUMS as FP32 deviations from the pivot over a chunk of at
// most two tiles, folded into a TwoSum pair.  The passes with a dynamic
// partition take the last one: their arithmetic is the bound beside HBM, and
// the FP64 sum's one more instruction per voxel costs them 2 % (2^32 voxels,
// 1024 bins: 2.49 against 2.44 ms; the others measure the same with either).
constexpr int ACC_FP32_SUMS = 3;

struct Lane {
    float mn, mx, s2, c2;
    float p2;      // FP32 chunk sum not yet folded into (s2, c2)
    float s1, c1, p1;  // the same of the first moment (ACC_FP32_SUMS; s1 alone: naive)
    double x;      // sum of x (CUBE_ACCUM_FP64MERGE)
};
constexpr Lane LANE_ZERO = {INFINITY, -INFINITY, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.0};

// Fold the pending FP32 chunk sums into the compensated lane accumulators
// (TwoSum).  Called after every second tile and at the end of every unit, so
// a chunk spans at most two tiles (32 voxels per lane) plus head and tail.
template <bool STATS, int ACC>
__device__ __forceinline__ void fold(Lane &L)
{
    if (STATS && ACC == ACC_FP32_SUMS) {
        two_sum_acc(L.s1, L.c1, L.p1);
        L.p1 = 0.f;
    }
    if (STATS && ACC != CUBE_ACCUM_NAIVE32) {
        two_sum_acc(L.s2, L.c2, L.p2);
        L.p2 = 0.f;
    }
}

struct Wave {  // wavefront-uniform
    float K;
    int has_k;
    unsigned long long slots;  // CUBE_ACCUM_FP64MERGE: voxel slots since K was set, valid or not
    unsigned long long valid, ge, le;  // ballot counts: valid, x >= lo, x <= hi
};

// The histogram as one voxel sees it.  LDS layout: slot s of copy c is the
// word s * C + c (C = 1 << copies_log2 copies, interleaved so that lanes of
// one wavefront hitting the same bin hit different banks).  Slot 0 collects
// blank and out-of-range voxels (they are counted with ballots instead);
// slots 1..nbins are bins 0..nbins-1; slot nbins+1 collects the rounding
// case floor(u) == nbins and is added to bin nbins-1 at the flush (this is
// the min(nbins-1, .) of the bin rule).  The byte address of bin b for a
// lane is (b << shift) + base with base = (C + lane % C) * 4, so the dummy
// slot is b = -1, an inline constant.
//
// With a hot bin (HIST_HOT), lanes whose bin is the block's hot bin add
// nothing to LDS; out-of-range and blank lanes are masked off instead of
// going to the dummy slot.
struct Hist {
    float lo, hi, scale;
    int nbins, shift, base;
    int hot;  // HIST_HOT: the block's hot bin (0..nbins), or -2 for none
    unsigned int base_abs;  // HIST_HOT: base plus the LDS byte address of `lds`
    unsigned int *lds;
    unsigned long long *global;
};

// LDS word at byte address `addr` += 1 in the lanes of `m` only: the exec
// mask is narrowed around one ds_add_u32 and restored in the same asm block,
// so the step stays one basic block (a compiler branch per voxel splits the
// loop into small blocks and spills its lane masks).  The compiler does not
// count this LDS operation: whoever reads the histogram waits for it with
// lds_wait() first.
__device__ __forceinline__ void lds_add1_masked(unsigned int addr, unsigned long long m)
{
    unsigned long long saved;
    asm volatile(
        "s_and_saveexec_b64 %0, %1\n\t"
        "ds_add_u32 %2, %3\n\t"
        "s_or_b64 exec, exec, %0"
        : "=&s"(saved)
        : "s"(m), "v"(addr), "v"(1u)
        : "memory", "scc");
}

__device__ __forceinline__ void lds_wait()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// The byte address of an LDS pointer (the LDS aperture keeps the offset in
// the low 32 bits of a generic address).
__device__ __forceinline__ unsigned int lds_offset(const unsigned int *p)
{
    return (unsigned int)(size_t)(__attribute__((address_space(3))) const unsigned int *)p;
}

// m[lane] ? v : 0, m[lane] ? v : k, and m[lane] ? v : -1 -- one v_cndmask_b32 reading a
// ballot mask directly, so a mask a ballot already produced is reused.
__device__ __forceinline__ float keep_where(float v, unsigned long long m)
{
    float r;
    asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(v), "s"(m));
    return r;
}
__device__ __forceinline__ float keep_or(float v, float k, unsigned long long m)
{
    float r;
    asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(k), "v"(v), "s"(m));
    return r;
}
__device__ __forceinline__ int keep_or_minus1(int v, unsigned long long m)
{
    int r;
    asm("v_cndmask_b32_e64 %0, -1, %1, %2" : "=v"(r) : "v"(v), "s"(m));
    return r;
}

// HIST_FINE: every bin is a 16-bit counter, two to a word: at 32768 words a
// block's histogram of up to 65536 bins fits LDS, where 32-bit counters would
// not and every voxel would be one 64-bit global atomic (23 G/s on an MI355X).
// A counter that has reached 0x8000 is seen by whoever adds to it next (the
// add returns the old word), and the wavefront that saw it moves 0x8000 from
// the counter to the global accumulators before its next step.  No counter
// can pass 0xffff meanwhile: a wavefront adds at most 64 * 16 to one counter
// in the step in which it sees the mark, so at most 16 * 1024 = 0x4000 adds
// fall between the mark and its removal.  Lanes without an in-range voxel add
// 0 to a word of their own after the counters (one per lane: no conflicts).
// Measured on 2^28 noise voxels, 65536 bins: 11.0 -> 0.215 ms (2^26: 2.79 ->
// 0.097), against 0.181 ms for 1024 bins: HBM, then the rows' write and sum.
__device__ __forceinline__ unsigned int fine_word(float u, int nbins, unsigned int *half)
{
    const int b = min(cvt_flr_i32(u), nbins - 1);
    *half = (unsigned int)b >> 15;
    return (unsigned int)b & (unsigned int)(FINE_WORDS - 1);
}

template <int NV>
__device__ __forceinline__ void fine_move(const float (&x)[NV], const Hist &H)
{
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        if (!(x[j] >= H.lo && x[j] <= H.hi)) continue;
        unsigned int half;
        const unsigned int w =
            fine_word(__fmul_rn(__fsub_rn(x[j], H.lo), H.scale), H.nbins, &half);
        const unsigned int was = atomicAnd(&H.lds[w], 0x7fff7fffu);
        if (was & 0x8000u) atomicAdd(&H.global[w], 0x8000ull);
        if (was & 0x80000000u) atomicAdd(&H.global[w + FINE_WORDS], 0x8000ull);
    }
}

// One step over NV voxels per lane.  With a histogram, two compares decide
// everything: A = (x >= lo), B = (x <= hi) are both false for a NaN and,
// since lo <= hi, not both false otherwise, so valid = A|B, in-range = A&B,
// and below = valid - |A|, above = valid - |B| (scalar mask algebra and
// popcounts on the ballots).
template <bool STATS, int HIST, int ACC, int NV>
__device__ __forceinline__ void process(const float (&x)[NV], Lane &L, Wave &W,
                                        const Hist &H)
{
    if (STATS && ACC != CUBE_ACCUM_NAIVE32 && !W.has_k) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(x[j] == x[j]);
            if (m) {
                const int l = __builtin_ctzll(m);
                W.K = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[j]), l));
                W.has_k = 1;
                break;
            }
        }
    }
    // Ballot counts of this step in 32-bit scalars (at most 64 * NV each).
    unsigned int cvalid = 0, cge = 0, cle = 0;
    unsigned int fine_seen = 0;  // HIST_FINE: the words added to, as they were
    float t2 = L.p2;
    const float K = W.K;
    float t1 = L.p1;
    if (STATS && ACC == CUBE_ACCUM_FP64MERGE) W.slots += W.has_k ? 64ull * NV : 0ull;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const float v = x[j];
        unsigned long long mvalid, inr = 0;
        const bool ge = v >= H.lo, le = v <= H.hi;
        if (HIST != HIST_NONE) {
            const unsigned long long mge = __builtin_amdgcn_ballot_w64(ge);
            const unsigned long long mle = __builtin_amdgcn_ballot_w64(le);
            mvalid = mge | mle;
            inr = mge & mle;
            cge += __popcll(mge);
            cle += __popcll(mle);
        } else {
            mvalid = __builtin_amdgcn_ballot_w64(v == v);
        }
        cvalid += __popcll(mvalid);
        if (STATS) {
            const float q = __builtin_canonicalizef(v);
            L.mn = fminf(L.mn, q);
            L.mx = fmaxf(L.mx, q);
            if (ACC == CUBE_ACCUM_NAIVE32) {
                const float d = keep_where(v, mvalid);
                L.s1 += d;
                L.s2 = __fmaf_rn(d, d, L.s2);
            } else if (ACC == ACC_FP32_SUMS) {
                const float d = keep_where(__fsub_rn(v, K), mvalid);
                t1 += d;
                t2 = __fmaf_rn(d, d, t2);
            } else {
                // Slots without a valid voxel take K: no deviation, and a
                // known part of the sum.
                const float w = keep_or(v, K, mvalid);
                L.x += (double)w;
                const float d = __fsub_rn(w, K);
                t2 = __fmaf_rn(d, d, t2);
            }
        }
        if (HIST != HIST_NONE) {
            const float u = __fmul_rn(__fsub_rn(v, H.lo), H.scale);
            if (HIST == HIST_LDS) {
                const int b = keep_or_minus1(cvt_flr_i32(u), inr);
                atomicAdd((unsigned int *)((char *)H.lds + ((b << H.shift) + H.base)), 1u);
            } else if (HIST == HIST_HOT) {
                // Only in-range lanes off the hot bin touch LDS.
                const int b = cvt_flr_i32(u);
                const unsigned long long off_hot = __builtin_amdgcn_ballot_w64(b != H.hot);
                lds_add1_masked((unsigned int)((b << H.shift) + H.base_abs), inr & off_hot);
            } else if (HIST == HIST_FINE) {
                unsigned int half;
                int w = (int)fine_word(u, H.nbins, &half);
                const bool in = ge && le;
                w = in ? w : H.base;
                fine_seen |= atomicAdd(&H.lds[w], in ? 1u << (half << 4) : 0u);
            } else {
                const int b = min(cvt_flr_i32(u), H.nbins - 1);
                if ((inr >> (threadIdx.x & 63)) & 1ull) atomicAdd(&H.global[b], 1ull);
            }
        }
    }
    if (HIST == HIST_FINE && __builtin_amdgcn_ballot_w64((fine_seen & 0x80008000u) != 0u))
        fine_move<NV>(x, H);
    // Keep the step counts 32-bit (the compiler would otherwise widen every
    // per-voxel add to 64 bits).
    asm("" : "+s"(cvalid), "+s"(cge), "+s"(cle));
    W.valid += cvalid;
    W.ge += cge;
    W.le += cle;
    if (STATS && ACC != CUBE_ACCUM_NAIVE32) {
        L.p1 = t1;
        L.p2 = t2;
    }
}

// Pairwise merge of (n, mean, m2) summaries (Chan, Golub & LeVeque).
template <typename T>
__device__ __forceinline__ void chan_merge(double &n, T &mean, T &m2, double nb, T mb, T m2b)
{
    if (nb == 0.0) return;
    if (n == 0.0) {
        n = nb;
        mean = mb;
        m2 = m2b;
        return;
    }
    const double nt = n + nb;
    const T d = mb - mean;
    mean = mean + d * (T)(nb / nt);
    m2 = m2 + m2b + d * d * (T)(n * nb / nt);
    n = nt;
}

template <typename T>
struct Summary {
    double n;
    T mean, m2;
    float mn, mx;
    unsigned long long nv, below, above;
};

template <typename T>
__device__ __forceinline__ void summary_merge(Summary<T> &a, const Summary<T> &b)
{
    chan_merge<T>(a.n, a.mean, a.m2, b.n, b.mean, b.m2);
    a.mn = fminf(a.mn, b.mn);
    a.mx = fmaxf(a.mx, b.mx);
    a.nv += b.nv;
    a.below += b.below;
    a.above += b.above;
}

template <typename T>
__device__ __forceinline__ Summary<T> shfl_xor_summary(const Summary<T> &s, int off)
{
    Summary<T> o;
    o.n = __shfl_xor(s.n, off);
    o.mean = __shfl_xor(s.mean, off);
    o.m2 = __shfl_xor(s.m2, off);
    o.mn = __shfl_xor(s.mn, off);
    o.mx = __shfl_xor(s.mx, off);
    o.nv = __shfl_xor(s.nv, off);
    o.below = __shfl_xor(s.below, off);
    o.above = __shfl_xor(s.above, off);
    return o;
}

// The (count, mean, m2) of one wavefront record: S1 = sum(x - K) and
// S2 = sum((x - K)^2) give mean = K + S1/n and m2 = S2 - S1^2/n (clamped at 0).
template <typename T, int ACC>
__device__ __forceinline__ void moments_of(const WaveRec &w, T &mb, T &m2b)
{
    const double nb = (double)w.n_valid;
    if (ACC == CUBE_ACCUM_NAIVE32) {
        const T S1 = (T)w.s1, S2 = (T)w.s2h, n = (T)nb;
        mb = S1 / n;
        m2b = S2 - S1 * S1 / n;
    } else {
        const T S1 = (T)(w.s1 - nb * (double)w.K);
        const T S2 = (T)w.s2h + (T)w.s2l;
        mb = (T)w.K + S1 / (T)nb;
        m2b = S2 - S1 * S1 / (T)nb;
    }
    if (m2b < (T)0) m2b = (T)0;
}

// A chunk record already holds its mean and m2.
template <typename T, int ACC>
__device__ __forceinline__ void moments_of(const ChunkRec &c, T &mb, T &m2b)
{
    mb = (T)c.mean;
    m2b = (T)c.m2;
}

// The global stage: every thread folds a fixed slice of the records (wave
// records, or chunk records in chunk order) in order, then a fixed xor-tree
// inside each wavefront, then the wavefront summaries in order.
// Deterministic for a given record count.
template <typename T, int ACC, typename R = WaveRec>
__device__ Summary<T> merge_records(const R *recs, int n_recs)
{
    const int tid = threadIdx.x, B = blockDim.x;
    const int r0 = (int)(((long long)n_recs * tid) / B);
    const int r1 = (int)(((long long)n_recs * (tid + 1)) / B);
    Summary<T> s = {0.0, (T)0, (T)0, INFINITY, -INFINITY, 0ull, 0ull, 0ull};
    for (int r = r0; r < r1; ++r) {
        const R w = recs[r];
        s.below += w.below;
        s.above += w.above;
        if (w.n_valid == 0) continue;
        s.nv += w.n_valid;
        s.mn = fminf(s.mn, w.mn);
        s.mx = fmaxf(s.mx, w.mx);
        T mb, m2b;
        moments_of<T, ACC>(w, mb, m2b);
        chan_merge<T>(s.n, s.mean, s.m2, (double)w.n_valid, mb, m2b);
    }
    for (int off = 1; off < 64; off <<= 1) {
        Summary<T> o = shfl_xor_summary(s, off);
        // Fixed pairing: the lower lane of each pair is the left operand.
        if ((threadIdx.x & off) == 0) {
            summary_merge(s, o);
        } else {
            summary_merge(o, s);
            s = o;
        }
    }
    __shared__ Summary<T> ws[MAX_WAVES];
    const int lane = tid & 63, wid = tid >> 6, nw = B >> 6;
    if (lane == 0) ws[wid] = s;
    __syncthreads();
    Summary<T> t = ws[0];
    for (int w = 1; w < nw; ++w) summary_merge(t, ws[w]);
    return t;
}

// One double and the counts and extrema that travel with it, combined over
// the lanes of a row, of a wavefront, or of the block, in a fixed order.
struct BlockSums {
    double s;
    unsigned long long nv, below, above;
    float mn, mx;
};

struct SumsStep {
    BlockSums &v;
    template <class C, class R>
    __device__ __forceinline__ void operator()(C, R)
    {
        v.s = dpp<C::value, R::value>(0.0, v.s) + v.s;
        v.nv += dpp<C::value, R::value>(0ull, v.nv);
        v.below += dpp<C::value, R::value>(0ull, v.below);
        v.above += dpp<C::value, R::value>(0ull, v.above);
        v.mn = fminf(v.mn, dpp<C::value, R::value>(INFINITY, v.mn));
        v.mx = fmaxf(v.mx, dpp<C::value, R::value>(-INFINITY, v.mx));
    }
};
struct DoubleStep {
    double &s;
    template <class C, class R>
    __device__ __forceinline__ void operator()(C, R)
    {
        s = dpp<C::value, R::value>(0.0, s) + s;
    }
};

__device__ __forceinline__ BlockSums from_lane(const BlockSums &v, int l)
{
    return {from_lane(v.s, l),     from_lane(v.nv, l), from_lane(v.below, l),
            from_lane(v.above, l), from_lane(v.mn, l), from_lane(v.mx, l)};
}

// Over the block: every thread gets the result.  One barrier; `ws` is not
// used for anything else before the block's next barrier.
__device__ __forceinline__ BlockSums block_sums(BlockSums v, BlockSums *ws)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    wave_reduce(SumsStep{v});
    if (lane == WAVE_LAST) ws[wid] = v;
    __syncthreads();
    BlockSums t = {0.0, 0ull, 0ull, 0ull, INFINITY, -INFINITY};
    if (lane < nw) t = ws[lane];
    row_reduce(SumsStep{t});
    return from_lane(t, ROW_LAST);
}
__device__ __forceinline__ double block_sum(double s, double *ws)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    wave_reduce(DoubleStep{s});
    if (lane == WAVE_LAST) ws[wid] = s;
    __syncthreads();
    double t = lane < nw ? ws[lane] : 0.0;
    row_reduce(DoubleStep{t});
    return from_lane(t, ROW_LAST);
}

// The two terms each record adds to the two sweeps of the FP64 global
// stage below: its sum of x, and its sum of (x - mean)^2 about the global
// mean.  A chunk record holds (n, mean_c, m2_c): n * mean_c and
// m2_c + n * (mean_c - mean)^2.  A wavefront record holds sum(x) itself and
// S2 = sum((x - K)^2): with S1 = sum(x) - n K and d = K - mean,
// sum((x - K) + d)^2 = S2 + 2 d S1 + n d^2.  Both forms are exact identities;
// neither divides.
__device__ __forceinline__ double sweep1_term(const ChunkRec &c)
{
    return (double)c.n_valid * c.mean;
}
__device__ __forceinline__ double sweep2_term(const ChunkRec &c, double mean)
{
    const double d = c.mean - mean;
    return c.m2 + (double)c.n_valid * d * d;
}
__device__ __forceinline__ double sweep1_term(const WaveRec &w)
{
    return w.s1;
}
__device__ __forceinline__ double sweep2_term(const WaveRec &w, double mean)
{
    const double d = (double)w.K - mean;
    const double S1 = w.s1 - (double)w.n_valid * (double)w.K;
    const double S2 = (double)w.s2h + (double)w.s2l;
    return S2 + 2.0 * d * S1 + (double)w.n_valid * d * d;
}

// The FP64 global stage in two sweeps over the records, with no division
// per record: the counts and the records' sums of x give the mean, then the
// records' sums of (x - mean)^2 give M2 -- the exact combination that the
// pairwise update of Chan, Golub & LeVeque applies two at a time.  Thread t
// takes records t, t + B, ... (coalesced loads, four in flight; with at most
// one record per thread it stays in registers between the sweeps), then
// block_sums fixes the rest of the order.  Deterministic for a given record
// count and block size.
template <typename R>
__device__ Summary<double> merge_two_sweep(const R *recs, int n_recs)
{
    __shared__ BlockSums ws1[MAX_WAVES];
    __shared__ double ws2[MAX_WAVES];
    const int tid = threadIdx.x, B = blockDim.x;
    BlockSums a = {0.0, 0ull, 0ull, 0ull, INFINITY, -INFINITY};
    auto take1 = [&](const R &c) {
        a.below += c.below;
        a.above += c.above;
        if (c.n_valid == 0) return;
        a.nv += c.n_valid;
        a.mn = fminf(a.mn, c.mn);
        a.mx = fmaxf(a.mx, c.mx);
        a.s += sweep1_term(c);
    };
    R own;
    own.n_valid = 0;
    const bool one = n_recs <= B;
    if (one) {
        if (tid < n_recs) {
            own = recs[tid];
            take1(own);
        }
    } else {
        int r = tid;
        for (; r + 3 * B < n_recs; r += 4 * B) {
            R c[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = recs[r + k * B];
#pragma unroll
            for (int k = 0; k < 4; ++k) take1(c[k]);
        }
        for (; r < n_recs; r += B) take1(recs[r]);
    }
    const BlockSums t = block_sums(a, ws1);
    const double mean = t.nv ? t.s / (double)t.nv : 0.0;
    double m2 = 0.0;
    auto take2 = [&](const R &c) {
        if (c.n_valid) m2 += sweep2_term(c, mean);
    };
    if (one) {
        take2(own);
    } else {
        int r = tid;
        for (; r + 3 * B < n_recs; r += 4 * B) {
            R c[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = recs[r + k * B];
#pragma unroll
            for (int k = 0; k < 4; ++k) take2(c[k]);
        }
        for (; r < n_recs; r += B) take2(recs[r]);
    }
    Summary<double> S;
    S.n = (double)t.nv;
    S.mean = mean;
    S.m2 = block_sum(m2, ws2);
    S.mn = t.mn;
    S.mx = t.mx;
    S.nv = t.nv;
    S.below = t.below;
    S.above = t.above;
    return S;
}

// The counts of the records alone (passes without statistics).
template <typename R>
__device__ BlockSums merge_counts(const R *recs, int n_recs)
{
    __shared__ BlockSums ws[MAX_WAVES];
    BlockSums a = {0.0, 0ull, 0ull, 0ull, INFINITY, -INFINITY};
    for (int r = threadIdx.x; r < n_recs; r += blockDim.x) {
        a.nv += recs[r].n_valid;
        a.below += recs[r].below;
        a.above += recs[r].above;
    }
    return block_sums(a, ws);
}

// One tile: U float4 loads per lane, lane stride B (a wavefront reads 1 KB
// per load); a uniform base plus fixed per-lane 32-bit byte offsets.
template <int U>
__device__ __forceinline__ void load_tile(f4 (&v)[U], const f4 *q4, long long off, int B, int tid)
{
    const char *base = (const char *)(q4 + off);
#pragma unroll
    for (int k = 0; k < U; ++k)
        v[k] = __builtin_nontemporal_load((const f4 *)(base + (unsigned int)((k * B + tid) * 16)));
}

// The first n (more than 0, under U * B) vectors of a tile; NaN in the others.
template <int U>
__device__ __forceinline__ void load_part(f4 (&v)[U], const f4 *q4, int n, int B, int tid)
{
#pragma unroll
    for (int k = 0; k < U; ++k) {
        v[k] = f4{qnan(), qnan(), qnan(), qnan()};
        if (k * B + tid < n) v[k] = __builtin_nontemporal_load(q4 + (k * B + tid));
    }
}

template <bool STATS, int HIST, int ACC, int U>
__device__ __forceinline__ void process_tile(const f4 (&v)[U], Lane &L, Wave &W, const Hist &H)
{
    float xv[4 * U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        xv[4 * k + 0] = v[k].x;
        xv[4 * k + 1] = v[k].y;
        xv[4 * k + 2] = v[k].z;
        xv[4 * k + 3] = v[k].w;
    }
    process<STATS, HIST, ACC, 4 * U>(xv, L, W, H);
}

// Histogram context of a pass over the valid range r (an invalid range is
// handled by the caller with a pass without histogram).
__device__ __forceinline__ void hist_setup(Hist &H, const HistRange &r, int nbins,
                                           int copies_log2, unsigned int *lds,
                                           unsigned long long *acc)
{
    const int lane = threadIdx.x & 63;
    const int C = 1 << copies_log2;
    H.hot = -2;
    H.nbins = nbins;
    H.shift = copies_log2 + 2;
    H.base = (C + (lane & (C - 1))) * 4;
    H.base_abs = (unsigned int)H.base + lds_offset(lds);
    H.lds = lds;
    H.global = acc;
    H.lo = r.lo;
    H.hi = r.hi;
    H.scale = r.scale;
}

// HIST_FINE: one layout, one copy, a word per lane after the counters.
__device__ __forceinline__ void fine_setup(Hist &H)
{
    H.base = FINE_WORDS + (int)(threadIdx.x & 63);
}

__device__ __forceinline__ void fine_zero(unsigned int *lds)
{
    uint4 *l4 = reinterpret_cast<uint4 *>(lds);
    for (int i = threadIdx.x; i < (FINE_WORDS + 64) / 4; i += blockDim.x)
        l4[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
}

// The block's counters as they are, to its row of the dump.  Starts with a
// barrier.
__device__ __forceinline__ void fine_dump(const unsigned int *lds, unsigned int *row)
{
    __syncthreads();
    const uint4 *l4 = reinterpret_cast<const uint4 *>(lds);
    uint4 *r4 = reinterpret_cast<uint4 *>(row);
    for (int i = threadIdx.x; i < FINE_WORDS / 4; i += blockDim.x) r4[i] = l4[i];
}

// Zero the LDS sub-histograms (nbins + 2 slots per copy); ends with a barrier.
__device__ __forceinline__ void lds_zero(unsigned int *lds, int nbins, int copies_log2)
{
    const int words = (nbins + 2) << copies_log2;
    for (int i = threadIdx.x; i < words; i += blockDim.x) lds[i] = 0u;
    __syncthreads();
}

// The "last block merges" ticket.  Called by every thread of the block after
// its writes; returns the same answer to every thread.  Every write that the
// last block reads is an agent-scope atomic store (written through the XCD's
// L2 to the device's point of coherence) or an agent-scope atomic
// read-modify-write (performed there).  Each wavefront waits for its own such
// writes to complete before the barrier, so all of them are performed at
// device scope before thread 0 takes the ticket; the last block then acquires
// (invalidates its L2) before it reads.  A release fence's buffer_wbl2 would
// only add the write-back of plain stores, of which there are none here; it
// stalls a block for several microseconds per call, which the batched launch
// pays at every tile.
__device__ __forceinline__ bool last_to_arrive_wt(unsigned int *ticket, unsigned int total,
                                                  unsigned int *s_shared)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool last = total == 1u || atomicAdd(ticket, 1u) == total - 1u;
        if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *s_shared = last ? 1u : 0u;
    }
    __syncthreads();
    return *s_shared != 0u;
}

// Scan the work units [u0, u1) of a box (segments of rows, see Geom).
template <bool STATS, int HIST, int ACC, int U>
__device__ __forceinline__ void scan_units(const Geom &g, long long u0, long long u1, Lane &L,
                                           Wave &W, const Hist &H)
{
    if (u0 >= u1) return;
    const int tid = threadIdx.x, B = blockDim.x;
    const int lane = tid & 63, wid = tid >> 6;
    long long row = u0 / g.segs;
    long long s = u0 - row * g.segs;
    long long y = row % g.ny;
    long long z = row / g.ny;
    for (long long u = u0; u < u1; ++u) {
        const float *q = g.ptr + y * g.sy + z * g.sz + s * g.seg_len;
        const long long c0 = s * g.seg_len;
        const long long len = min(g.seg_len, g.row_len - c0);
        const long long mis = (long long)((16 - ((uintptr_t)q & 15)) & 15) >> 2;
        const long long h = min(len, mis);
        const long long n4 = (len - h) >> 2;
        const long long t = len - h - 4 * n4;
        if (wid == 0 && h + t > 0) {
            // Head and tail voxels: lanes [0, h) and [h, h + t).
            long long idx = lane < h ? lane : h + 4 * n4 + (lane - h);
            const bool have = lane < h + t;
            idx = have ? idx : 0;
            float xv[1];
            const float v = q[idx];
            xv[0] = have ? v : qnan();
            process<STATS, HIST, ACC, 1>(xv, L, W, H);
        }
        const f4 *q4 = (const f4 *)(q + h);
        // Full tiles, software-pipelined: the next tile's loads are in
        // flight while the current tile is processed.
        const long long T = (long long)B * U;
        const long long ntiles = n4 / T;
        if (ntiles > 0) {
            f4 va[U], vb[U];
            load_tile<U>(va, q4, 0, B, tid);
            long long k = 0;
            while (true) {
                if (k + 1 < ntiles) load_tile<U>(vb, q4, (k + 1) * T, B, tid);
                process_tile<STATS, HIST, ACC, U>(va, L, W, H);
                if (++k == ntiles) break;
                if (k + 1 < ntiles) load_tile<U>(va, q4, (k + 1) * T, B, tid);
                process_tile<STATS, HIST, ACC, U>(vb, L, W, H);
                fold<STATS, ACC>(L);
                if (++k == ntiles) break;
            }
        }
        // A remainder of more than one vector per lane is one more tile, its
        // missing vectors NaN: one load latency, where a loop over single
        // vectors pays up to U of them.
        const long long rest = n4 - ntiles * T;
        if (rest > B) {
            f4 v[U];
            load_part<U>(v, q4 + ntiles * T, (int)rest, B, tid);
            process_tile<STATS, HIST, ACC, U>(v, L, W, H);
        } else if (rest > 0) {
            const bool have = tid < rest;
            const f4 v = __builtin_nontemporal_load(q4 + (have ? ntiles * T + tid : n4 - 1));
            float xv[4];
            xv[0] = have ? v.x : qnan();
            xv[1] = have ? v.y : qnan();
            xv[2] = have ? v.z : qnan();
            xv[3] = have ? v.w : qnan();
            process<STATS, HIST, ACC, 4>(xv, L, W, H);
        }
        fold<STATS, ACC>(L);
        if (++s == g.segs) {
            s = 0;
            if (++y == g.ny) {
                y = 0;
                ++z;
            }
        }
    }
}

// Visit the rows [u0, u1) of a packed geometry (cube_rows.h): `f` is called
// with 4 * U voxels per lane, lanes without a voxel padded with NaN, and
// f.pair() after every second call and at the end.  Bound by HBM on long
// rows, by the latency of a few tiles on small boxes.  Measured against the
// scan of one row at a time (scan_units), whole calls: a 1187 x 911 x 263
// box in rows of 2048, statistics + 1024 bins 1.71 -> 0.275 ms (4.1 TB/s);
// a 61 x 47 x 200 box, statistics 0.180 -> 0.026 ms; the median of a
// 941 x 937 x 240 box 3.76 -> 0.55 ms.
//
// PIPE: the next tile's loads are issued before a tile is processed (twice the
// load registers); the selection passes, which only count, run faster without.
template <int U, bool PIPE, class F>
__device__ __forceinline__ void scan_rows(const Geom &g, long long u0, long long u1, F &f)
{
    if (u0 >= u1) return;
    const RowPack &pk = g.pack;
    const unsigned int lr = threadIdx.x / (unsigned int)pk.cb;
    const unsigned int lc = threadIdx.x - lr * (unsigned int)pk.cb;
    const unsigned int ny = (unsigned int)g.ny, r0 = (unsigned int)u0, r1 = (unsigned int)u1;
    RowLane ln = row_lane(pk, g.ptr, g.sy, g.sz, ny, r0, r1, lr);
    int s[U], d[U];
    unsigned int edge = 0u;  // bit k: this wavefront masks voxels of its k-th vector
#pragma unroll
    for (int k = 0; k < U; ++k) {
        row_vector(pk, (int)g.row_len, lc, k & (pk.cg - 1), &s[k], &d[k]);
        if (__builtin_amdgcn_ballot_w64(d[k] != 0)) edge |= 1u << k;
    }
    auto load = [&](f4 (&v)[U]) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            v[k] = f4{qnan(), qnan(), qnan(), qnan()};
            if (ln.row < ln.row_end) v[k] = __builtin_nontemporal_load((const f4u *)(ln.p + s[k]));
            if (((k + 1) & (pk.cg - 1)) == 0) row_advance(pk, ny, ln);
        }
    };
    auto take = [&](const f4 (&v)[U]) {
        float x[4 * U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            x[4 * k + 0] = v[k].x;
            x[4 * k + 1] = v[k].y;
            x[4 * k + 2] = v[k].z;
            x[4 * k + 3] = v[k].w;
            if ((edge >> k) & 1u) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    x[4 * k + i] = row_own(i, d[k]) ? x[4 * k + i] : qnan();
            }
        }
        f(x);
    };
    const unsigned int tiles = row_tiles(pk, r0, r1, U);
    f4 va[U];
    if constexpr (!PIPE) {
        for (unsigned int k = 0; k < tiles; ++k) {
            load(va);
            take(va);
            f.pair();
        }
        return;
    }
    f4 vb[U];
    load(va);
    unsigned int k = 0;
    while (true) {
        if (k + 1 < tiles) load(vb);
        take(va);
        if (++k == tiles) break;
        if (k + 1 < tiles) load(va);
        take(vb);
        f.pair();
        if (++k == tiles) break;
    }
    f.pair();
}

// The pass's step for scan_rows.
template <bool STATS, int HIST, int ACC>
struct PassStep {
    Lane &L;
    Wave &W;
    const Hist &H;
    template <int NV>
    __device__ __forceinline__ void operator()(const float (&x)[NV])
    {
        process<STATS, HIST, ACC, NV>(x, L, W, H);
    }
    __device__ __forceinline__ void pair() { fold<STATS, ACC>(L); }
};

// Scan the work units [u0, u1) of a box in the form its geometry asks for.
template <bool STATS, int HIST, int ACC, int U, bool PACKED>
__device__ __forceinline__ void scan(const Geom &g, long long u0, long long u1, Lane &L, Wave &W,
                                     const Hist &H)
{
    if constexpr (PACKED) {
        PassStep<STATS, HIST, ACC> f = {L, W, H};
        scan_rows<U, true>(g, u0, u1, f);
    } else {
        scan_units<STATS, HIST, ACC, U>(g, u0, u1, L, W, H);
    }
}

// A record to global memory; with WT (write-through) as agent-scope atomic
// stores, which gfx950 writes through its XCD's L2 (see last_to_arrive_wt).
template <bool WT, class R>
__device__ __forceinline__ void store_record(const R &r, R *dst)
{
    if (WT) {
        const unsigned long long *w = reinterpret_cast<const unsigned long long *>(&r);
        unsigned long long *d = reinterpret_cast<unsigned long long *>(dst);
#pragma unroll
        for (int i = 0; i < (int)(sizeof(R) / 8); ++i)
            __hip_atomic_store(d + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        *dst = r;
    }
}

template <int ACC>
struct LaneStep {
    Lane &l;
    template <class C, class R>
    __device__ __forceinline__ void operator()(C, R)
    {
        l.mn = fminf(l.mn, dpp<C::value, R::value>(INFINITY, l.mn));
        l.mx = fmaxf(l.mx, dpp<C::value, R::value>(-INFINITY, l.mx));
        const float o2 = dpp<C::value, R::value>(0.f, l.s2);
        if (ACC == CUBE_ACCUM_FP64MERGE)
            l.x = dpp<C::value, R::value>(0.0, l.x) + l.x;
        if (ACC == CUBE_ACCUM_NAIVE32) {
            l.s1 += dpp<C::value, R::value>(0.f, l.s1);
            l.s2 += o2;
        } else {
            df_add(l.s2, l.c2, o2, dpp<C::value, R::value>(0.f, l.c2));
            if (ACC == ACC_FP32_SUMS) {
                const float o1 = dpp<C::value, R::value>(0.f, l.s1);
                df_add(l.s1, l.c1, o1, dpp<C::value, R::value>(0.f, l.c1));
            }
        }
    }
};

// Local stage: reduce the lanes of the calling wavefront into one record
// (written by its last lane).
template <bool STATS, int ACC, bool WT = false>
__device__ __forceinline__ void write_wave_record(const Lane &L, const Wave &W, WaveRec *dst)
{
    Lane l = L;
    if (STATS) wave_reduce(LaneStep<ACC>{l});
    if ((threadIdx.x & 63) == WAVE_LAST) {
        WaveRec r;
        r.n_valid = W.valid;
        r.below = W.valid - W.ge;
        r.above = W.valid - W.le;
        r.K = W.K;
        r.s1 = ACC == CUBE_ACCUM_NAIVE32 ? (double)l.s1
               : ACC == ACC_FP32_SUMS
                   ? (double)W.K * (double)W.valid + ((double)l.s1 + (double)l.c1)
                   : l.x - (double)W.K * (double)(W.slots - W.valid);
        r.s2h = l.s2;
        r.s2l = l.c2;
        r.mn = l.mn;
        r.mx = l.mx;
        r.pad = 0.f;
        r.pad2 = 0ull;
        store_record<WT>(r, dst);
    }
}

// The record of a block's part of the box (its whole range, or one chunk of a
// dynamic partition), formed by the calling wavefront from the block's
// wavefront records (`parts`, in LDS, `nw` <= 16 of them): the two sweeps of
// merge_two_sweep over one row of lanes.  Without STATS only the counts are
// kept.  Fewer records for the last block to merge: 256 blocks of 1024
// threads left 4096 wavefront records, 11.5 us; 256 block records take 3.
template <bool STATS, bool WT>
__device__ __forceinline__ void write_chunk_record(const WaveRec *parts, int nw, ChunkRec *dst)
{
    const int lane = threadIdx.x & 63;
    BlockSums a = {0.0, 0ull, 0ull, 0ull, INFINITY, -INFINITY};
    WaveRec w;
    w.n_valid = 0;
    if (lane < nw) {
        w = parts[lane];
        a.below = w.below;
        a.above = w.above;
        a.nv = w.n_valid;
        if (STATS && w.n_valid) {
            a.mn = w.mn;
            a.mx = w.mx;
            a.s = sweep1_term(w);
        }
    }
    row_reduce(SumsStep{a});
    double mean = 0.0, m2 = 0.0;
    if (STATS) {
        const unsigned long long nv = from_lane(a.nv, ROW_LAST);
        mean = nv ? from_lane(a.s, ROW_LAST) / (double)nv : 0.0;
        m2 = w.n_valid ? sweep2_term(w, mean) : 0.0;
        row_reduce(DoubleStep{m2});
    }
    if (lane == ROW_LAST) {
        ChunkRec c;
        c.mean = mean;
        c.m2 = m2 < 0.0 ? 0.0 : m2;
        c.mn = a.mn;
        c.mx = a.mx;
        c.pad0 = c.pad1 = 0u;
        c.n_valid = a.nv;
        c.below = a.below;
        c.above = a.above;
        c.pad2 = 0ull;
        store_record<WT>(c, dst);
    }
}

// Add the block's LDS sub-histograms into the global accumulators (one
// atomic per non-empty bin), or write them to its row of the dump when there
// is one.  Starts with a barrier.
__device__ __forceinline__ void hist_flush(const unsigned int *lds, int nbins, int copies_log2,
                                           unsigned long long *acc, unsigned int *row = nullptr)
{
    __syncthreads();
    const int C = 1 << copies_log2;
    // Each thread starts at its own copy (c + tid) so that the threads of a
    // wavefront read different banks at every step.
    const int rot = threadIdx.x;
    for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
        unsigned int sum = 0;
        for (int c = 0; c < C; ++c) sum += lds[((b + 1) << copies_log2) + ((c + rot) & (C - 1))];
        if (b == nbins - 1)  // floor(u) == nbins belongs to the last bin
            for (int c = 0; c < C; ++c) sum += lds[((nbins + 1) << copies_log2) + c];
        if (row)
            row[b] = sum;
        else if (sum)
            atomicAdd(&acc[b], (unsigned long long)sum);
    }
}

// The hot bin of a block (HIST_HOT), chosen by its first wavefront before the
// scan: the bin of the first in-range voxel among the first 64 of the block's
// first work unit, computed with the same FP32 operations as every voxel's
// bin (any value is correct; a likely one saves LDS atomics).  -2: none.
__device__ __forceinline__ int hot_bin_pick(const Geom &g, long long u0, long long u1,
                                            const Hist &H)
{
    if (u0 >= u1) return -2;
    const int lane = threadIdx.x & 63;
    const long long row = u0 / g.segs;
    const long long sg = u0 - row * g.segs;
    const long long y = row % g.ny, z = row / g.ny;
    const long long c0 = sg * g.seg_len;
    const long long len = min(g.seg_len, g.row_len - c0);
    const float *q = g.ptr + y * g.sy + z * g.sz + c0;
    const float v = lane < len ? q[lane] : qnan();
    const int b = cvt_flr_i32(__fmul_rn(__fsub_rn(v, H.lo), H.scale));
    const unsigned long long m = __builtin_amdgcn_ballot_w64(v >= H.lo && v <= H.hi);
    if (!m) return -2;
    return __builtin_amdgcn_readlane(b, __builtin_ctzll(m));
}

// The flush of a hot-bin histogram: every other bin as in hist_flush, then
// the hot bin's count, which is the block's in-range count (`s_inr`, summed
// from the wavefronts' ballot counts) minus everything the block added to
// LDS (`s_tot`, zeroed before the scan).  Starts with a barrier.
__device__ __forceinline__ void hist_flush_hot(const unsigned int *lds, int nbins,
                                               int copies_log2, unsigned long long *acc,
                                               int hot, const unsigned int *s_inr,
                                               unsigned int *s_tot)
{
    lds_wait();  // the masked LDS adds of this wavefront
    __syncthreads();
    const int C = 1 << copies_log2;
    const int rot = threadIdx.x;
    unsigned int mine = 0;
    for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
        unsigned int sum = 0;
        for (int c = 0; c < C; ++c) sum += lds[((b + 1) << copies_log2) + ((c + rot) & (C - 1))];
        if (b == nbins - 1)  // floor(u) == nbins belongs to the last bin
            for (int c = 0; c < C; ++c) sum += lds[((nbins + 1) << copies_log2) + c];
        mine += sum;
        if (sum) atomicAdd(&acc[b], (unsigned long long)sum);
    }
    if (mine) atomicAdd(s_tot, mine);
    __syncthreads();
    if (threadIdx.x == 0 && hot >= 0) {
        const unsigned int n_hot = *s_inr - *s_tot;
        if (n_hot) atomicAdd(&acc[hot < nbins ? hot : nbins - 1], (unsigned long long)n_hot);
    }
}

// The in-range count of the calling wavefront (ballots: x >= lo, x <= hi and
// valid = either), added to the block's LDS counter by lane 0.
__device__ __forceinline__ void add_in_range(const Wave &W, unsigned int *s_inr)
{
    if ((threadIdx.x & 63) == 0)
        atomicAdd(s_inr, (unsigned int)(W.ge + W.le - W.valid));
}

// The [min, max] histogram range with its FP32 scale, formed from the data
// extrema exactly as the host forms a given range: ok = 1 valid, 0 invalid
// (infinite extrema, or a width or scale that overflows), 2 no valid voxel.
__device__ __forceinline__ HistRange range_of_extrema(float fmn, float fmx, unsigned long long nv,
                                                      int nbins)
{
    HistRange r = {qnan(), qnan(), 0.f, 2};
    if (nv == 0) return r;
    r.ok = 0;
    if (isfinite(fmn) && isfinite(fmx)) {
        const float w = __fsub_rn(fmx, fmn);
        if (isfinite(w)) {
            const float sc = w == 0.f ? 0.f : __fdiv_rn((float)nbins, w);
            if (isfinite(sc)) {
                r.lo = fmn;
                r.hi = fmx;
                r.scale = sc;
                r.ok = 1;
            }
        }
    }
    return r;
}

// A result word to memory; with HOST to host memory, as a system-scope atomic
// store (written through; a plain store may stay in the L2 until the kernel
// ends, or longer: a poll that sees a later kernel's word says nothing of it).
template <bool HOST, class T>
__device__ __forceinline__ void store_result(T *dst, T v)
{
    if (HOST)
        __hip_atomic_store(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    else
        *dst = v;
}

// The statistics that an earlier pass left in device memory, to the host with
// this pass's own results (called by every thread of the block).
__device__ __forceinline__ void forward_stats(const cube_stats_t *from, cube_stats_t *to)
{
    constexpr int words = (int)(sizeof(cube_stats_t) / 8);
    if ((int)threadIdx.x < words)
        store_result<true>(reinterpret_cast<unsigned long long *>(to) + threadIdx.x,
                           reinterpret_cast<const unsigned long long *>(from)[threadIdx.x]);
}

// Tell the polling CPU that the block's results are in host memory: every
// thread has waited for its own write-through stores before the barrier.
__device__ __forceinline__ void tell_host(unsigned int *done, unsigned int gen)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(done, gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Moments over the extended reals.  An infinite voxel is a valid value and
// always one of the extrema, so the exact min and max show whether any are
// present, at no cost per voxel: +Inf alone makes the mean +Inf, -Inf alone
// -Inf, both NaN (Inf - Inf); and since the deviation of an infinite voxel
// from such a mean is not finite, m2 and std are NaN.  Without infinities
// the merged finite moments stand.
__device__ __forceinline__ void extended_real_moments(cube_stats_t &o)
{
    const bool pinf = o.max == INFINITY, ninf = o.min == -INFINITY;
    if (!pinf && !ninf) return;
    o.mean = (pinf && ninf) ? (double)qnan() : (pinf ? (double)INFINITY : -(double)INFINITY);
    o.m2 = o.std = (double)qnan();
}

// The global stage of a stats pass: merge `n_recs` records (all threads of
// the block call it), then thread 0 writes the result and, when `range_out`
// is given, the [min, max] histogram range with its FP32 scale.  Returns the
// total valid / below / above counts to every thread.
template <int ACC, typename R = WaveRec>
__device__ void finish_stats(const R *recs, int n_recs, int accum_mode,
                             unsigned long long n_total, cube_stats_t *out,
                             HistRange *range_out, int nbins, unsigned long long &nv,
                             unsigned long long &below, unsigned long long &above,
                             bool host = false)
{
    float fmn, fmx;
    double mean, m2;
    if (accum_mode == CUBE_ACCUM_FP64MERGE) {
        // Pivoted wavefront records (FP64MERGE partials) and chunk records
        // take the two-sweep merge; the naive partials keep the pairwise one.
        Summary<double> S;
        if constexpr (std::is_same<R, ChunkRec>::value || ACC == CUBE_ACCUM_FP64MERGE)
            S = merge_two_sweep<R>(recs, n_recs);
        else
            S = merge_records<double, ACC, R>(recs, n_recs);
        nv = S.nv; below = S.below; above = S.above;
        fmn = S.mn; fmx = S.mx; mean = S.mean; m2 = S.m2;
    } else {
        const Summary<float> S = merge_records<float, ACC, R>(recs, n_recs);
        nv = S.nv; below = S.below; above = S.above;
        fmn = S.mn; fmx = S.mx; mean = (double)S.mean; m2 = (double)S.m2;
    }
    if (threadIdx.x != 0) return;
    cube_stats_t o;
    o.n_total = n_total;
    o.n_valid = nv;
    o.n_nan = n_total - nv;
    o.flags = 0u;
    o.reserved = 0u;
    if (nv == 0) {
        o.min = o.max = qnan();
        o.mean = o.m2 = o.std = (double)qnan();
        o.flags |= CUBE_NO_VALID;
    } else {
        o.min = fmn;
        o.max = fmx;
        o.mean = mean;
        o.m2 = m2 < 0.0 ? 0.0 : m2;
        o.std = accum_mode == CUBE_ACCUM_FP64MERGE ? sqrt(o.m2 / (double)nv)
                                                   : (double)sqrtf((float)o.m2 / (float)nv);
        extended_real_moments(o);
    }
    if (range_out) {
        const HistRange r = range_of_extrema(fmn, fmx, nv, nbins);
        if (r.ok == 0) o.flags |= CUBE_HIST_BAD_RANGE;
        *range_out = r;
    }
    if (host) {
        const unsigned long long *w = reinterpret_cast<const unsigned long long *>(&o);
        for (int i = 0; i < (int)(sizeof o / 8); ++i)
            store_result<true>(reinterpret_cast<unsigned long long *>(out) + i, w[i]);
    } else {
        *out = o;
    }
}

// Copy the global accumulators to the caller's counts (or, with `add`, add
// them to the counts already there) and return them to zero; thread 0 writes
// below / above / NaN.  `deferred`: the bins are left to launch_hist_sum.
// `host`: the counts are host memory (store_result).
__device__ __forceinline__ void finish_hist(unsigned long long *acc, unsigned long long *counts,
                                            int nbins, bool on, unsigned long long below,
                                            unsigned long long above, unsigned long long n_nan,
                                            bool add = false, bool deferred = false,
                                            bool host = false)
{
    if (host) {
        for (int b = threadIdx.x; b < nbins && !deferred; b += blockDim.x) {
            store_result<true>(&counts[b], acc[b]);
            acc[b] = 0ull;
        }
    } else {
        for (int b = threadIdx.x; b < nbins && !deferred; b += blockDim.x) {
            counts[b] = (add ? counts[b] : 0ull) + acc[b];
            acc[b] = 0ull;
        }
    }
    if (threadIdx.x == 0) {
        const unsigned long long last[3] = {on ? below : 0ull, on ? above : 0ull, n_nan};
        for (int i = 0; i < 3; ++i) {
            if (host)
                store_result<true>(&counts[nbins + i], last[i]);
            else
                counts[nbins + i] = (add ? counts[nbins + i] : 0ull) + last[i];
        }
    }
}

}  // namespace cube
