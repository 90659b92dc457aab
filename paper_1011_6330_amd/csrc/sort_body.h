// sort_body.h -- bodies of the scan and scatter passes of the cell sort, shared by
// the single-tube kernels and the batched sort.
//
// A tile is SORT_TILE consecutive source slots, taken by a block of
// SORT_BLOCK threads as SORT_PPT columns of SORT_BLOCK consecutive slots
// (thread t holds slot tile0 + k SORT_BLOCK + t of column k).  For each
// column, the lanes of a run of equal keys take consecutive destination slots
// with one atomic per run on the key's running offset.  The columns' atomics
// are issued together, in source order, so their latencies overlap and the
// particles of a key keep roughly their source order.  That order carries no
// result (every step is per particle or an integer reduction), but between
// sorts it keeps particles with similar histories, and hence similar
// velocities, in the same wave.
#pragma once

#include <limits.h>
#include <math.h>

#include "pcpic_internal.h"
#include "wave.h"

namespace pcpic {

// The two FP32-bulk particle streams of one buffer parity.
struct Streams {
    int *CL;
    float *OL;
    float *UL;
    unsigned *HP;   // high stream: position words, cells of wide groups, group headers
    int *HW;
    int *HG;
    double *UH;
};

// Cell (-1 for a removed slot) and offset of high-stream slot p.
__device__ __forceinline__ int hi_slot(const Streams &s, int64_t p, float &off)
{
    const unsigned w = s.HP[p];
    off = hi_offset(w);
    if (w == HI_DEAD) return -1;
    const int hdr = s.HG[p >> HI_GROUP_LOG2];
    return hdr >= 0 ? hi_cell(w, hdr, 0) : s.HW[p];
}

// Writes a live particle (cell, frac in units of 2^-24) at high-stream slot q
// of a stream being filled in the wide form (the sort, the appends); the first
// slot of each group sets the group's header.
__device__ __forceinline__ void hi_put_wide(const Streams &s, int64_t q, int cell, unsigned frac, double u)
{
    s.HW[q] = cell;
    s.HP[q] = frac;
    s.UH[q] = u;
    if ((q & (HI_GROUP - 1)) == 0) s.HG[q >> HI_GROUP_LOG2] = HI_WIDE;
}

// Adds to *jumps the jumps (step_route.h) among the loaded particles of this block of 256,
// one per thread, cell < 0 for none, waves of the push taking `wave` of them; a block
// stands for `stride` of them, and the others return at once.  Called by every thread.
__device__ __forceinline__ void count_jumps(int cell, int wave, int stride, int64_t *jumps)
{
    if (blockIdx.x % (unsigned)stride != 0) return;
    __shared__ int s_lo[4], s_n;
    const int w = threadIdx.x >> 6;
    const int lo1 = wave_min_i32(cell >= 0 ? cell : INT_MAX);
    if (threadIdx.x == 0) s_n = 0;
    if (__lane_id() == 0) s_lo[w] = lo1;
    __syncthreads();
    const int lo2 = min(s_lo[w], s_lo[w ^ 1]), lo = wave == 256 ? min(lo2, min(s_lo[w ^ 2], s_lo[w ^ 3])) : lo2;
    const int before = __shfl_up(cell, 1);
    const unsigned long long m = __ballot(cell >= 0 && cell - lo > 62 && (cell >> 3) != (before >> 3));
    if (__lane_id() == 0 && m) atomicAdd(&s_n, __popcll(m));
    __syncthreads();
    if (threadIdx.x == 0 && s_n) atomicAdd((unsigned long long *)jumps, (unsigned long long)s_n * (unsigned)stride);
}

// Destination stream of a particle: the high stream from |u| >= u_hi on.
__device__ __forceinline__ bool goes_high(double u, double u_hi) { return fabs(u) >= u_hi; }

// Exclusive scan of the key counts, one block of SORT_BLOCK threads per
// SORT_SCAN_TILE keys.  What comes before a block's keys is summed by the block itself:
// from the counts up to SCAN_DIRECT blocks (no other kernel), from block totals
// (scan_totals) up to SCAN_SUMS blocks, and past that it is read from a scan of those
// totals (scan_blocks).
// Small sorts are bound by their launches: a round of two steps and a sort of an empty
// tube took, with totals and their scan / totals / counts only, 24.6 / 23.0 / 21.1 us at
// 2 blocks, 25.0 / 23.7 / 23.3 at 8, 25.4 / 24.1 / 25.7 at 16.  The sums of totals grow
// with the square of the blocks: 247 (scanned) / 242 us at 2048, 956 / 940 at 8192.
constexpr int64_t SCAN_DIRECT = 8;
constexpr int64_t SCAN_SUMS = 8192;

struct ScanTube {
    int64_t n_keys;
    const long long *count;
    long long *off, *blk;
    DevCounters *ctr;
    StepScratch *sc;
    int64_t klo;            // first key of the high stream (-1: one stream)
    long long *total_lo;    // its offset
};
__host__ __device__ inline int64_t scan_blocks_of(int64_t n_keys) { return (n_keys + SORT_SCAN_TILE - 1) / SORT_SCAN_TILE; }

__device__ __forceinline__ void scan_load(const long long *count, int64_t n, int64_t base, long long (&v)[4],
                                          long long &s)
{
    static_assert(SORT_SCAN_TILE == 4 * SORT_BLOCK, "four keys per thread");
    s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = base + k < n ? count[base + k] : 0;
        s += v[k];
    }
}

__device__ __forceinline__ void scan_totals(const ScanTube &t, int64_t lb)
{
    __shared__ long long s_wave[SORT_BLOCK / 64];
    long long v[4], s;
    scan_load(t.count, t.n_keys, lb * SORT_SCAN_TILE + (int64_t)threadIdx.x * 4, v, s);
    const long long inc = block_scan_incl(s, s_wave);
    if (threadIdx.x == SORT_BLOCK - 1) t.blk[lb] = inc;
}

// Exclusive scan of the block totals (one block, sequential chunks).
__device__ __forceinline__ void scan_blocks(const ScanTube &t, int64_t nblk)
{
    __shared__ long long s_wave[SORT_BLOCK / 64];
    __shared__ long long s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < nblk; b0 += SORT_BLOCK) {
        const int64_t i = b0 + threadIdx.x;
        const long long v = i < nblk ? t.blk[i] : 0;
        const long long inc = block_scan_incl(v, s_wave);
        const long long carry = s_carry;
        if (i < nblk) t.blk[i] = carry + inc - v;
        __syncthreads();
        if (threadIdx.x == SORT_BLOCK - 1) s_carry = carry + inc;
        __syncthreads();
    }
}

// Offsets of the keys of block lb of nblk; the last block sets the live count, the
// first keeps the source slot counts for the scatter.
__device__ __forceinline__ void scan_apply(const ScanTube &t, int64_t lb, int64_t nblk)
{
    __shared__ long long s_wave[SORT_BLOCK / 64];
    const int64_t base = lb * SORT_SCAN_TILE + (int64_t)threadIdx.x * 4;
    long long v[4], s;
    scan_load(t.count, t.n_keys, base, v, s);
    long long run = 0;
    if (nblk > SCAN_SUMS) {
        run = t.blk[lb];
    } else if (lb > 0) {
        const bool direct = nblk <= SCAN_DIRECT;
        const long long *p = direct ? t.count : t.blk;
        const int64_t n = direct ? lb * SORT_SCAN_TILE : lb;
        long long q = 0;
#pragma unroll 4
        for (int64_t i = threadIdx.x; i < n; i += SORT_BLOCK) q += p[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
        if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = q;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SORT_BLOCK / 64; ++k) run += s_wave[k];
        __syncthreads();
    }
    run += block_scan_incl(s, s_wave) - s;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (base + k < t.n_keys) {
            t.off[base + k] = run;
            if (base + k == t.klo) *t.total_lo = run;
        }
        run += v[k];
    }
    if (lb == nblk - 1 && threadIdx.x == SORT_BLOCK - 1) t.ctr->n_alive = run;
    if (lb == 0 && threadIdx.x == 0) {
        t.sc->sort_n[0] = t.ctr->n_slots;
        t.sc->sort_n[1] = t.ctr->n_slots_hi;
    }
}

// The scatter's blocks also clear the key counts, for the next step that accumulates
// them, and its first sets the slot counts of the sorted streams.
__device__ __forceinline__ void sort_finish(long long *count, int64_t n_keys, DevCounters *ctr,
                                            const long long *total_lo, int64_t blk, int64_t nblk)
{
    for (int64_t i = blk * SORT_BLOCK + threadIdx.x; i < n_keys; i += nblk * SORT_BLOCK) count[i] = 0;
    if (blk == 0 && threadIdx.x == 0) {
        const int64_t n = ctr->n_alive, lo = total_lo ? *total_lo : n;
        ctr->n_slots = lo;
        ctr->n_slots_hi = n - lo;
        ctr->n_removed = 0;
    }
}

// Item k of a pass over a tube's slots in tiles of SORT_TILE: FP64 has one
// stream; in FP32-bulk mode the low stream's tiles come first, then the high
// stream's.  Returns false for an item past the slots (so ceil(capacity /
// SORT_TILE) items, plus one in FP32-bulk mode, cover any split).
__device__ __forceinline__ bool sort_item(int64_t k, bool f32, const StepScratch *sc, bool &hi, int64_t &tile0,
                                          int64_t &n)
{
    const int64_t n_lo = sc->sort_n[0];
    const int64_t items_lo = (n_lo + SORT_TILE - 1) / SORT_TILE;
    hi = f32 && k >= items_lo;
    tile0 = (hi ? k - items_lo : k) * SORT_TILE;
    n = hi ? sc->sort_n[1] : n_lo;
    return tile0 < n;
}

// Scatter of the FP64 slots [tile0, tile0 + SORT_TILE) of (X, U), tile0 < n,
// into (Xo, Uo) at the running offsets off[key]; removed slots (x < 0) are
// dropped.  Called by every thread of a block of SORT_BLOCK threads.
__device__ __forceinline__ void scatter_tile_f64(const Consts &c, const double *X, const double *U, double *Xo,
                                                 double *Uo, unsigned long long *off, int64_t n, int64_t tile0)
{
    const int lane = (int)__lane_id();
    double x[SORT_PPT], u[SORT_PPT];
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        const int64_t p = tile0 + (int64_t)k * SORT_BLOCK + threadIdx.x;
        x[k] = p < n ? __builtin_nontemporal_load(X + p) : -1.0;
        u[k] = p < n ? __builtin_nontemporal_load(U + p) : 0.0;
    }
    int64_t key[SORT_PPT];
    bool want[SORT_PPT];
    WaveRun r[SORT_PPT];
    unsigned long long f[SORT_PPT];
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        want[k] = x[k] >= 0.0;
        key[k] = want[k] ? sort_key_f64(c, x[k]) : 0;
        r[k] = wave_runs(key[k], want[k]);
    }
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        f[k] = 0;
        if (want[k] && r[k].is_head) f[k] = atomicAdd(off + key[k], (unsigned long long)(r[k].end - lane));
    }
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        f[k] = __shfl(f[k], r[k].head);
        if (want[k]) {
            const int64_t d = (int64_t)f[k] + r[k].rank;
            Xo[d] = x[k];
            Uo[d] = u[k];
        }
    }
}

// Scatter of the FP32-bulk slots [tile0, tile0 + SORT_TILE) of one source
// stream (HI: the high stream), tile0 < n.  The key (sort_key_f32) names the
// destination stream from the particle's momentum, so particles migrate
// between the streams here; tlo is the number of slots of the destination low
// stream (the high stream's keys start there).
template <bool HI>
__device__ __forceinline__ void scatter_tile_f32(const Consts &c, const Streams &src, const Streams &dst,
                                                 double u_hi, int64_t tlo, unsigned long long *off, int64_t n,
                                                 int64_t tile0)
{
    const int lane = (int)__lane_id();
    int cl[SORT_PPT];
    float o[SORT_PPT];
    double u[SORT_PPT];
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        const int64_t p = tile0 + (int64_t)k * SORT_BLOCK + threadIdx.x;
        const bool in = p < n;
        if (HI) {
            o[k] = 0.0f;
            cl[k] = in ? hi_slot(src, p, o[k]) : -1;
            u[k] = in ? __builtin_nontemporal_load(src.UH + p) : 0.0;
        } else {
            cl[k] = in ? __builtin_nontemporal_load(src.CL + p) : -1;
            o[k] = in ? __builtin_nontemporal_load(src.OL + p) : 0.0f;
            u[k] = in ? (double)__builtin_nontemporal_load(src.UL + p) : 0.0;
        }
    }
    const int64_t klo = sort_low_keys(c);
    int64_t key[SORT_PPT];
    bool want[SORT_PPT];
    WaveRun r[SORT_PPT];
    unsigned long long f[SORT_PPT];
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        want[k] = cl[k] >= 0;
        key[k] = want[k] ? sort_key_f32(c, cl[k], o[k], goes_high(u[k], u_hi)) : 0;
        r[k] = wave_runs(key[k], want[k]);
    }
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        f[k] = 0;
        if (want[k] && r[k].is_head) f[k] = atomicAdd(off + key[k], (unsigned long long)(r[k].end - lane));
    }
#pragma unroll
    for (int k = 0; k < SORT_PPT; ++k) {
        f[k] = __shfl(f[k], r[k].head);
        if (want[k]) {
            const int64_t d = (int64_t)f[k] + r[k].rank;
            if (key[k] >= klo) {
                // a low particle reaching the threshold was put on the 2^-24 grid by its push
                int cell = cl[k];
                unsigned frac;
                hi_snap((double)o[k], cell, frac);
                if (cell >= (int)c.N) { cell = (int)c.N - 1; frac = HI_FRAC_MASK; }
                hi_put_wide(dst, d - tlo, cell, frac, u[k]);
            } else {
                dst.CL[d] = cl[k];
                dst.OL[d] = o[k];
                dst.UL[d] = (float)u[k];
            }
        }
    }
}

}  // namespace pcpic
