// diag_body.h -- per-block accumulators of the particle passes of the
// diagnostics and of the Poisson start: the signed-gamma profile and the CIC
// node weights.
//
// A block walks one contiguous range of slots (block_range), so between sorts
// its particles sit in a few profile bins and cells.  Each wave keeps a current
// bin and a current cell: lanes whose particle belongs to them add to registers
// of their own, without any exchange between lanes.  When the current one
// changes, the lanes add their partial sums to the block's LDS window; a
// particle of yet another bin or cell goes there by itself, and one outside the
// window straight to memory.  The block adds its window to memory once, at its
// end.  Every sum is an integer sum, a minimum or a maximum, so the result does
// not depend on the order.
//
// (A form that reduced the partial sums over the wave and added them to memory
// from every wave took 19 us for a tube of 2e5 particles, all of it atomics of
// 3,000 waves on 64 bins, and 222 us for 4e7 particles, whose 640 MB take 97 us
// at the copy rate.)
#pragma once

#include "pcpic_internal.h"
#include "short_math.h"
#include "wave.h"

namespace pcpic {

constexpr int MOM_BLOCK = 256;             // threads per block
constexpr int MOM_TILE = 4 * MOM_BLOCK;    // slots per block and iteration: 256 per wave, two pairs per lane
constexpr int MOM_MIN = MOM_TILE;          // fewest slots per block
constexpr int MOM_BINS = 256;              // profile bins in the LDS window
constexpr int MOM_NODES = 1024;            // grid nodes in the LDS window

// Slots [lo, hi) of block b of nblocks over n slots: contiguous ranges of
// whole tiles, at least MOM_MIN slots long.
__device__ __forceinline__ void block_range(int64_t n, int64_t nblocks, int64_t b, int64_t &lo, int64_t &hi)
{
    int64_t per = (((n + nblocks - 1) / nblocks) + MOM_TILE - 1) & ~(int64_t)(MOM_TILE - 1);
    if (per < MOM_MIN) per = MOM_MIN;
    lo = b * per < n ? b * per : n;
    hi = lo + per < n ? lo + per : n;
}

// Signed-gamma profile: per bin the count, the 128-bit fixed-point sum in units
// of 2^-32, min and max of the ordered bit images.
struct ProfOut {
    long long *cnt;
    unsigned long long *lo;
    long long *hi;
    long long *mn, *mx;
};

// The block's LDS windows; b0 and n0 are the first bin and the first node.
struct MomWindow {
    long long cnt[MOM_BINS];
    unsigned long long lo[MOM_BINS];   // low 32 bits of the addends
    long long hi[MOM_BINS];            // the rest
    long long mn[MOM_BINS], mx[MOM_BINS];
    int b0;
};
struct NodeWindow {
    unsigned long long w[MOM_NODES];
    int n0;
};

__device__ __forceinline__ void emit_bin(const ProfOut &o, int64_t b, long long c, __int128 sum, long long mn,
                                         long long mx)
{
    atomicAdd((unsigned long long *)&o.cnt[b], (unsigned long long)c);
    atomic_add_i128(&o.lo[b], &o.hi[b], sum);
    atomicMin(&o.mn[b], mn);
    atomicMax(&o.mx[b], mx);
}

// A lane's partial sums (c particles, integer parts si and 2^-32 fractions sf of
// their signed gammas) into bin b.
__device__ __forceinline__ void add_bin(MomWindow &s, const ProfOut &o, int b, int c, long long si, long long sf,
                                        double mn, double mx)
{
    const long long omn = ordered_bits(mn), omx = ordered_bits(mx);
    const int k = b - s.b0;
    if (k >= 0 && k < MOM_BINS) {
        atomicAdd((unsigned long long *)&s.cnt[k], (unsigned long long)c);
        atomicAdd(&s.lo[k], (unsigned long long)sf & 0xffffffffull);
        atomicAdd((unsigned long long *)&s.hi[k], (unsigned long long)(si + (sf >> 32)));
        atomicMin(&s.mn[k], omn);
        atomicMax(&s.mx[k], omx);
    } else {
        emit_bin(o, b, c, ((__int128)si << 32) + (__int128)sf, omn, omx);
    }
}

// w0 to node `node`, w1 to the next.
__device__ __forceinline__ void add_nodes(NodeWindow &s, unsigned long long *w, int node, int64_t w0, int64_t w1)
{
    const int k = node - s.n0;
    if (k >= 0 && k + 1 < MOM_NODES) {
        atomicAdd(&s.w[k], (unsigned long long)w0);
        atomicAdd(&s.w[k + 1], (unsigned long long)w1);
    } else {
        atomicAdd(w + node, (unsigned long long)w0);
        atomicAdd(w + node + 1, (unsigned long long)w1);
    }
}

// A wave's profile accumulator.  The partial sums are whole numbers in doubles:
// a lane adds at most 2^21 gammas below 2^31 and their fractions of at most 2^32
// units between two flushes, so every sum is exact; larger gammas go to the window
// one by one.
struct ProfAcc {
    int bin = -1;                 // current bin (wave-uniform), -1: none
    int c = 0;
    double si = 0.0, sf = 0.0, mn = INFINITY, mx = -INFINITY;

    __device__ __forceinline__ void flush(MomWindow &s, const ProfOut &o)
    {
        if (c > 0) add_bin(s, o, bin, c, (long long)si, (long long)sf, mn, mx);
        c = 0;
        si = sf = 0.0;
        mn = INFINITY;
        mx = -INFINITY;
    }

    // One particle per lane (want: the lane has one); called by every lane.
    __device__ __forceinline__ void add(MomWindow &s, const ProfOut &o, bool want, int b, double sg)
    {
        const double fl = floor(sg);
        const double f = rint((sg - fl) * 4294967296.0);
        bool rest = want;
        bool fit = want && fabs(sg) < 0x1p31 && c < (1 << 21);
#pragma unroll
        for (int turn = 0; turn < 2; ++turn) {
            if (fit && b == bin) {
                c += 1;
                si += fl;
                sf += f;
                mn = fmin(mn, sg);
                mx = fmax(mx, sg);
                fit = rest = false;
            }
            if (turn == 1) break;
            const unsigned long long m = __ballot(fit);
            if (!m) break;
            flush(s, o);                                    // the wave moves on to its last particle's bin
            bin = __shfl(b, 63 - __clzll(m));
        }
        if (rest) add_bin(s, o, b, 1, (long long)fl, (long long)f, sg, sg);
    }
};

// A wave's node weights: 2^P - F to node `cell`, F to node cell + 1, as a count
// and the sum of F (whole numbers below 2^53: at most 2^16 of F <= 2^36).
struct WeightAcc {
    int cell = -1;                // current cell (wave-uniform), -1: none
    int c = 0;
    double f = 0.0;

    __device__ __forceinline__ void flush(NodeWindow &s, unsigned long long *w, int64_t oneP)
    {
        if (c > 0) add_nodes(s, w, cell, (int64_t)c * oneP - (int64_t)f, (int64_t)f);
        c = 0;
        f = 0.0;
    }

    // One particle per lane; called by every lane.
    __device__ __forceinline__ void add(NodeWindow &s, unsigned long long *w, bool live, int cl, int64_t oneP, double F)
    {
        bool rest = live, fit = live && c < (1 << 16);
#pragma unroll
        for (int turn = 0; turn < 2; ++turn) {
            if (fit && cl == cell) {
                c += 1;
                f += F;
                fit = rest = false;
            }
            if (turn == 1) break;
            const unsigned long long m = __ballot(fit);
            if (!m) break;
            flush(s, w, oneP);
            cell = __shfl(cl, 63 - __clzll(m));
        }
        if (rest) add_nodes(s, w, cl, oneP - (int64_t)F, (int64_t)F);
    }
};

// sign(u) gamma(u) (sqrt(1 + u^2) correctly rounded: its short form where that is the same).
__device__ __forceinline__ double signed_gamma(double u)
{
    double t = u * u;
    t = 1.0 + t;
    double gam = gs_sqrt(t);
    if (!(fabs(u) <= 0x1p+400)) gam = sqrt(t);
    return u < 0.0 ? -gam : gam;
}

// Profile bin of x (cell units): floor(x nb / N), clamped; rN = nr_recip(N).
// The short division gives the division's bits for a dividend in its range; a
// smaller one has quotient 0 either way.
__device__ __forceinline__ int profile_bin(double x, double nbd, double Nd, double rN, int nb)
{
    const int b = (int)floor(nr_div(x * nbd, Nd, rN));
    return b < 0 ? 0 : (b > nb - 1 ? nb - 1 : b);
}

}  // namespace pcpic
