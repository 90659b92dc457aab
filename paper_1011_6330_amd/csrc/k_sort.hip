// k_sort.hip -- counting sort of the particles by cell, dropping removed slots.
//
// key counts (taken by the push of the step before) -> exclusive scan over the
// keys -> scatter into the other particle buffer, lanes of a wave that share a
// key taking consecutive slots.  Every step of the method is per
// particle or an integer reduction, so the order this produces (which varies
// from run to run between waves of the same cell) never changes a result.
//
// Two kernels up to 8192 keys, three up to 8.4 million (sort_body.h); the scatter
// also clears the counts and sets the slot counts.  A small sort is bound by its
// launches (a tube of 1024 cells, 205 steps with a sort every 16: 1210 us with six
// kernels per sort, 1138 with two), a large one by its scattered writes (2.5e8
// particles 1.56 ms, 1.2 at the copy rate).
#include <math.h>

#include "pcpic_internal.h"
#include "sort_body.h"
#include "wave.h"

namespace pcpic {

__global__ __launch_bounds__(256) void k_fill_ll(long long *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ __launch_bounds__(SORT_BLOCK) void k_scan_totals(ScanTube t) { scan_totals(t, blockIdx.x); }
__global__ __launch_bounds__(SORT_BLOCK) void k_scan_blocks(ScanTube t, int64_t nblk) { scan_blocks(t, nblk); }
__global__ __launch_bounds__(SORT_BLOCK) void k_scan_apply(ScanTube t) { scan_apply(t, blockIdx.x, gridDim.x); }

// Scatter into the other buffer, one block per tile of SORT_TILE slots.
__global__ __launch_bounds__(SORT_BLOCK) void k_scatter(Consts c, const double *__restrict__ X,
                                                        const double *__restrict__ U, double *__restrict__ Xo,
                                                        double *__restrict__ Uo, DevCounters *ctr,
                                                        const StepScratch *sc, unsigned long long *off,
                                                        long long *count, int64_t n_keys)
{
    sort_finish(count, n_keys, ctr, nullptr, blockIdx.x, gridDim.x);
    const int64_t n = sc->sort_n[0];
    const int64_t tile0 = (int64_t)blockIdx.x * SORT_TILE;
    if (tile0 >= n) return;
    scatter_tile_f64(c, X, U, Xo, Uo, off, n, tile0);
}

static hipError_t launch_scan(pic_handle *h, int64_t n)
{
    Workspace &w = h->ws;
    const bool f32 = h->p.precision == PIC_FP32_BULK;
    const ScanTube t{n, w.cell_count, w.cell_off, w.blk_sum, w.ctr, w.sc, f32 ? sort_low_keys(h->c) : -1, w.total_lo};
    const int64_t nblk = scan_blocks_of(n);
    if (nblk > SCAN_DIRECT)
        hipLaunchKernelGGL(k_scan_totals, dim3((unsigned)nblk), dim3(SORT_BLOCK), 0, h->stream, t);
    if (nblk > SCAN_SUMS) hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(SORT_BLOCK), 0, h->stream, t, nblk);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nblk), dim3(SORT_BLOCK), 0, h->stream, t);
    return hipGetLastError();
}

// Zero the key counts, if a sort has not left them so, before the step that
// accumulates them (the step before a sort).
hipError_t launch_clear_hist(pic_handle *h)
{
    if (h->counts_clear) return hipSuccess;
    const int64_t nkeys = sort_key_count(h->c, h->p.precision == PIC_FP32_BULK);
    hipLaunchKernelGGL(k_fill_ll, dim3((unsigned)((nkeys + 255) / 256)), dim3(256), 0, h->stream, h->ws.cell_count,
                       nkeys);
    const hipError_t e = hipGetLastError();
    h->counts_clear = e == hipSuccess;
    return e;
}

// Counting sort by cell into the other particle buffer, dropping removed slots;
// in FP32-bulk mode the destination stream follows the particle's gamma.
hipError_t launch_sort(pic_handle *h)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    const bool f32 = h->p.precision == PIC_FP32_BULK;
    const int64_t nkeys = sort_key_count(c, f32);
    const int src = h->pbuf, dst = 1 - h->pbuf;
    hipError_t e = launch_scan(h, nkeys);
    if (e != hipSuccess) return e;
    if (f32) {
        e = launch_sort32_scatter(h, nkeys);
    } else {
        const unsigned blocks = (unsigned)scatter_blocks((c.cap + SORT_TILE - 1) / SORT_TILE, nkeys);
        hipLaunchKernelGGL(k_scatter, dim3(blocks), dim3(SORT_BLOCK), 0, h->stream, c, w.x[src], w.u[src], w.x[dst],
                           w.u[dst], w.ctr, w.sc, (unsigned long long *)w.cell_off, w.cell_count, nkeys);
        e = hipGetLastError();
    }
    h->pbuf = dst;
    h->counts_clear = e == hipSuccess;
    return e;
}

}  // namespace pcpic
