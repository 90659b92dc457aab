// k_diag.hip -- diagnostics: discrete Gauss residual (divergence equation of
// eq. 2 with d/dr -> 1/R) and the signed-gamma profile of sec. 3 (returning
// electrons counted with negative gamma).  All reductions are integer or
// max/min on ordered bit images, so every result is independent of the
// order in which particles are visited.
#include <limits.h>
#include <math.h>

#include "pcpic_internal.h"
#include "diag_body.h"
#include "sort_body.h"
#include "wave.h"

namespace pcpic {

// G_i = (E_z,i+1/2 - E_z,i-1/2)/dz + E_r,i/R - 4 pi (rho_i - rho_GJ,i), nodes 1..N-1
// (PIC_GR_ALPHA: the first and the rho term times alpha_i).
__global__ __launch_bounds__(256) void k_gauss(Consts c, const double *ez, const double *er,
                                               const int64_t *w, const double *rho_gj, double *g,
                                               DevCounters *ctr)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double a = 0.0;
    if (i <= c.N) {
        double gi = 0.0;
        if (i >= 1 && i < c.N) {
            double rho = (c.qmP * (double)w[i]) / c.dz;
            double dez = (ez[i] - ez[i - 1]) / c.dz;
            if (c.flags & PIC_GR_ALPHA) {
                // alpha_i dE_z/dz + E_r/R = 4 pi (alpha_i lambda_i - rho_GJ,i)
                const double an = gr_alpha_node(c, i);
                dez = an * dez;
                rho = an * rho;
            }
            const double d = dez + er[i] / c.R;
            gi = d - c.fourpi * (rho - rho_gj[i]);
        }
        g[i] = gi;
        a = fabs(gi);
    }
    block_max_abs(&ctr->gauss_max_bits, a);
}

// Clears nb profile bins, nw node weights and, with ctr, the Gauss maximum of the diagnostics.
__global__ __launch_bounds__(256) void k_moments_clear(int nb, ProfPtrs p, int64_t nw, unsigned long long *w,
                                                       DevCounters *ctr)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < nb) {
        p.cnt[i] = 0;
        p.lo[i] = 0;
        p.hi[i] = 0;
        p.mn[i] = ordered_bits(INFINITY);
        p.mx[i] = ordered_bits(-INFINITY);
    }
    if (i < nw) w[i] = 0;
    if (i == 0 && ctr) ctr->gauss_max_bits = 0;
}

// The accumulated bins in the caller's layout: counts and the 128-bit sums as
// they are, min and max back from their ordered bit images to doubles (an empty
// bin gives +inf and -inf).  Any output may be null.
__global__ __launch_bounds__(256) void k_profile_finish(int nb, ProfPtrs p, int64_t *count, uint64_t *sum_lo,
                                                        int64_t *sum_hi, double *vmin, double *vmax)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nb) return;
    if (count) count[i] = p.cnt[i];
    if (sum_lo) sum_lo[i] = p.lo[i];
    if (sum_hi) sum_hi[i] = p.hi[i];
    if (vmin) vmin[i] = from_ordered_bits(p.mn[i]);
    if (vmax) vmax[i] = from_ordered_bits(p.mx[i]);
}

// The particle pass of the diagnostics and of the Poisson start: the signed-gamma
// profile (PROF) and the CIC node weights (WTS) of the live particles, both from
// one read of x and u.  Block b takes a contiguous range of each stream's slots
// in tiles of 1024, each wave 256 consecutive slots of a tile as two pairs per
// lane (16-byte accesses, in FP32-bulk mode the group of the high stream that
// one wave of the push takes).
template <int F32, int PROF, int WTS>
__global__ __launch_bounds__(MOM_BLOCK) void k_moments(Consts c, int nb, const double *__restrict__ X,
                                                       const double *__restrict__ U, Streams s,
                                                       const DevCounters *ctr, ProfOut o, unsigned long long *w)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef int i2 __attribute__((ext_vector_type(2)));
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __shared__ MomWindow sb;
    __shared__ NodeWindow sw;
    const int tid = (int)threadIdx.x, wv = tid >> 6, lane = (int)__lane_id();
    const int64_t n_lo = ctr->n_slots, n_hi = F32 ? ctr->n_slots_hi : 0;
    const double nbd = (double)nb, Nd = (double)c.N, rN = nr_recip(Nd);
#pragma unroll 1
    for (int high = 0; high < 1 + F32; ++high) {
        const int64_t n = high ? n_hi : n_lo;
        int64_t lo, hi;
        block_range(n, gridDim.x, blockIdx.x, lo, hi);
        if (lo >= hi) continue;                              // uniform over the block
        if (PROF) {
            sb.cnt[tid] = 0;
            sb.lo[tid] = 0;
            sb.hi[tid] = 0;
            sb.mn[tid] = ordered_bits(INFINITY);
            sb.mx[tid] = ordered_bits(-INFINITY);
            if (tid == 0) sb.b0 = nb <= MOM_BINS ? 0 : INT_MAX;
        }
        if (WTS) {
#pragma unroll
            for (int k = 0; k < MOM_NODES / MOM_BLOCK; ++k) sw.w[k * MOM_BLOCK + tid] = 0;
            if (tid == 0) sw.n0 = INT_MAX;
        }
        __syncthreads();
        ProfAcc pa;
        WeightAcc wa;
        bool first = true;
#pragma unroll 1
        for (int64_t base = lo; base < hi; base += MOM_TILE) {
            const int64_t g0 = base + wv * 256, q0 = g0 + 2 * lane, q1 = q0 + 128;
            double x[4], u[4];       // FP32-bulk: x holds the offset in the cell until it is used
            int cell[4];
            if (!F32) {
                if (g0 + 256 <= hi) {
                    const d2 xa = *(const d2 *)(X + q0), xb = *(const d2 *)(X + q1);
                    x[0] = xa.x; x[1] = xa.y; x[2] = xb.x; x[3] = xb.y;
                    if (PROF) {
                        const d2 ua = *(const d2 *)(U + q0), ub = *(const d2 *)(U + q1);
                        u[0] = ua.x; u[1] = ua.y; u[2] = ub.x; u[3] = ub.y;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int64_t p = (k < 2 ? q0 : q1) + (k & 1);
                        x[k] = p < hi ? X[p] : -1.0;
                        u[k] = PROF && p < hi ? U[p] : 0.0;
                    }
                }
            } else if (!high) {
                if (g0 + 256 <= hi) {
                    const i2 ca = *(const i2 *)(s.CL + q0), cb = *(const i2 *)(s.CL + q1);
                    const f2 oa = *(const f2 *)(s.OL + q0), ob = *(const f2 *)(s.OL + q1);
                    cell[0] = ca.x; cell[1] = ca.y; cell[2] = cb.x; cell[3] = cb.y;
                    x[0] = oa.x; x[1] = oa.y; x[2] = ob.x; x[3] = ob.y;
                    if (PROF) {
                        const f2 ua = *(const f2 *)(s.UL + q0), ub = *(const f2 *)(s.UL + q1);
                        u[0] = ua.x; u[1] = ua.y; u[2] = ub.x; u[3] = ub.y;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int64_t p = (k < 2 ? q0 : q1) + (k & 1);
                        cell[k] = p < hi ? s.CL[p] : -1;
                        x[k] = p < hi ? s.OL[p] : 0.0f;
                        u[k] = PROF && p < hi ? s.UL[p] : 0.0f;
                    }
                }
            } else {
                const int hdr = g0 < hi ? s.HG[g0 >> HI_GROUP_LOG2] : 0;   // one group per wave
                unsigned v[4];
                int wc[4] = {0, 0, 0, 0};
                if (g0 + 256 <= hi) {
                    const u2 pa2 = *(const u2 *)(s.HP + q0), pb2 = *(const u2 *)(s.HP + q1);
                    v[0] = pa2.x; v[1] = pa2.y; v[2] = pb2.x; v[3] = pb2.y;
                    if (PROF) {
                        const d2 ua = *(const d2 *)(s.UH + q0), ub = *(const d2 *)(s.UH + q1);
                        u[0] = ua.x; u[1] = ua.y; u[2] = ub.x; u[3] = ub.y;
                    }
                    if (hdr < 0) {
                        const i2 ca = *(const i2 *)(s.HW + q0), cb = *(const i2 *)(s.HW + q1);
                        wc[0] = ca.x; wc[1] = ca.y; wc[2] = cb.x; wc[3] = cb.y;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int64_t p = (k < 2 ? q0 : q1) + (k & 1);
                        v[k] = p < hi ? s.HP[p] : HI_DEAD;
                        u[k] = PROF && p < hi ? s.UH[p] : 0.0;
                        if (hdr < 0 && p < hi) wc[k] = s.HW[p];
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    cell[k] = v[k] != HI_DEAD ? hi_cell(v[k], hdr, wc[k]) : -1;
                    x[k] = (double)hi_offset(v[k]);
                }
            }
            if (first) {
                // the windows start at the lowest bin and cell of the range's first tile
                first = false;
                int m = INT_MAX;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int cl = F32 ? cell[k] : (x[k] >= 0.0 && x[k] < Nd ? (int)x[k] : -1);
                    m = cl >= 0 && cl < m ? cl : m;
                }
                m = wave_min_i32(m);
                if (m != INT_MAX && lane == 0) {
                    if (WTS) atomicMin(&sw.n0, m);
                    if (PROF && nb > MOM_BINS) atomicMin(&sb.b0, profile_bin((double)m, nbd, Nd, rN, nb));
                }
                __syncthreads();
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double cd = F32 ? (double)cell[k] : floor(x[k]);
                const double off = F32 ? x[k] : x[k] - cd;
                const bool live = F32 ? cell[k] >= 0 : x[k] >= 0.0 && x[k] < Nd;
                if (WTS) wa.add(sw, w, live, F32 ? cell[k] : (int)cd, c.oneP, rint(off * c.twoP));
                if (PROF) pa.add(sb, o, live, profile_bin(F32 ? cd + off : x[k], nbd, Nd, rN, nb), signed_gamma(u[k]));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (WTS) wa.flush(sw, w, c.oneP);
        if (PROF) pa.flush(sb, o);
        __syncthreads();
        if (PROF && sb.cnt[tid] != 0)
            emit_bin(o, (int64_t)sb.b0 + tid, sb.cnt[tid],
                     ((__int128)sb.hi[tid] << 32) + (__int128)sb.lo[tid], sb.mn[tid], sb.mx[tid]);
        if (WTS) {
#pragma unroll
            for (int k = 0; k < MOM_NODES / MOM_BLOCK; ++k) {
                const unsigned long long v = sw.w[k * MOM_BLOCK + tid];
                if (v != 0) atomicAdd(w + sw.n0 + k * MOM_BLOCK + tid, v);
            }
        }
        __syncthreads();
    }
}

hipError_t launch_clear_bins(pic_handle *h, int n, const ProfPtrs &p)
{
    hipLaunchKernelGGL(k_moments_clear, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, h->stream, n, p, (int64_t)0,
                       nullptr, nullptr);
    return hipGetLastError();
}

// Clears (the bins unless bins_clear) and accumulates the profile (nb > 0) into p and
// the node weights (w_out non-null); clear_gauss also clears the Gauss maximum.
hipError_t launch_moments(pic_handle *h, int nb, const ProfPtrs &p, int64_t *w_out, bool clear_gauss, bool bins_clear)
{
    const Consts &c = h->c;
    const Workspace &w = h->ws;
    const int64_t nw = w_out ? c.N + 1 : 0, nc = bins_clear ? 0 : nb, m = nw > nc ? nw : (nc > 0 ? nc : 1);
    unsigned long long *wo = (unsigned long long *)w_out;
    if (nc > 0 || nw > 0 || clear_gauss)
        hipLaunchKernelGGL(k_moments_clear, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, h->stream, (int)nc, p, nw,
                           wo, clear_gauss ? w.ctr : nullptr);
    if (nb <= 0 && !w_out) return hipGetLastError();
    // eight blocks per CU, fewer when the capacity does not give each MOM_MIN slots
    const int64_t most = (int64_t)h->n_cu * 8, fit = (c.cap + MOM_MIN - 1) / MOM_MIN;
    const dim3 g((unsigned)(fit < most ? fit : most)), bl(MOM_BLOCK);
    const int b = h->pbuf;
    const ProfOut o{p.cnt, p.lo, p.hi, p.mn, p.mx};
    const Streams s{w.cl[b], w.ol[b], w.ul[b], w.hp[b], w.hw[b], w.hg[b], w.uh[b]};
#define MOMENTS(F32, PROF, WTS) \
    hipLaunchKernelGGL((k_moments<F32, PROF, WTS>), g, bl, 0, h->stream, c, nb, w.x[b], w.u[b], s, w.ctr, o, wo)
    if (h->p.precision == PIC_FP32_BULK) {
        if (nb > 0 && w_out) MOMENTS(1, 1, 1);
        else if (nb > 0) MOMENTS(1, 1, 0);
        else MOMENTS(1, 0, 1);
    } else {
        if (nb > 0 && w_out) MOMENTS(0, 1, 1);
        else if (nb > 0) MOMENTS(0, 1, 0);
        else MOMENTS(0, 0, 1);
    }
#undef MOMENTS
    return hipGetLastError();
}

// The Gauss residual from the node weights in w.w (launch_moments).
hipError_t launch_gauss(pic_handle *h)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    const int f = h->fbuf;
    hipLaunchKernelGGL(k_gauss, dim3((unsigned)((c.N + 1 + 255) / 256)), dim3(256), 0, h->stream, c,
                       w.ez[f], w.er[f], w.w, w.rho_gj, w.gauss, w.ctr);
    return hipGetLastError();
}

// Results of a read-out gathered into page-locked host memory (the GPU writes it
// directly): segment y copies its 8-byte words, two per thread.  One kernel and
// one wait take the place of a copy per array: 3 KB arrive in 11.4 us, where five
// copies into pageable memory took 74.
__global__ __launch_bounds__(256) void k_pack(PackArgs a, unsigned long long *dst)
{
    typedef unsigned long long l2 __attribute__((ext_vector_type(2)));
    const PackSeg g = a.seg[blockIdx.y];
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 2; i < g.words; i += (int64_t)gridDim.x * 512) {
        if (i + 2 <= g.words) *(l2 *)(dst + g.at + i) = *(const l2 *)(g.src + i);
        else dst[g.at + i] = g.src[i];
        if (g.reset) {
            g.src[i] = g.value;
            if (i + 2 <= g.words) g.src[i + 1] = g.value;
        }
    }
}

hipError_t launch_pack(pic_handle *h, const PackArgs &a, void *dst)
{
    int64_t most = 0;
    for (int k = 0; k < a.n; ++k) most = a.seg[k].words > most ? a.seg[k].words : most;
    if (most == 0) return hipSuccess;
    const int64_t blocks = (most + 511) / 512;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)(blocks < 1024 ? blocks : 1024), (unsigned)a.n), dim3(256), 0, h->stream, a,
                       (unsigned long long *)dst);
    return hipGetLastError();
}

hipError_t launch_profile_finish(pic_handle *h, int nb, const ProfPtrs &p, int64_t *count, uint64_t *sum_lo,
                                 int64_t *sum_hi, double *vmin, double *vmax)
{
    if (nb > 0)
        hipLaunchKernelGGL(k_profile_finish, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, h->stream, nb, p,
                           count, sum_lo, sum_hi, vmin, vmax);
    return hipGetLastError();
}

}  // namespace pcpic
