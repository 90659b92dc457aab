// k_field.hip -- grid kernels: rho_GJ, Poisson initialisation (eq. 4), the
// leap-frog update of the reduced Maxwell system (eq. 3) fused with the
// space-charge-limited injection at the base (sec. 2).
//
// Every floating-point expression is written with the operand order of the
// step's definition and compiled with -ffp-contract=off, so the results are
// bit-identical to an IEEE double evaluation of the same formulas.
#include <math.h>

#include "pcpic_internal.h"
#include "wave.h"
#include "field_body.h"
#include "sort_body.h"
#include "thomas_body.h"

namespace pcpic {

__global__ __launch_bounds__(256) void k_rho_gj(Consts c, const double *knots, double *rho,
                                                DevCounters *ctr)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double a = 0.0;
    if (i <= c.N) {
        const double r = rho_node(c, knots, i);
        rho[i] = r;
        a = fabs(r);
    }
    block_max_abs(&ctr->rho_max_bits, a);   // max |rho_GJ| for the Gauss normalisation
}

// Right-hand side of eq. (4) times dz^2 on nodes 1..N; node N carries the
// mirror-doubled particle weight (phi' = 0 at the tube end: phi, rho even about N).
// PIC_GR_ALPHA: rho_GJ / alpha at the node.
__global__ __launch_bounds__(256) void k_poisson_rhs(Consts c, const int64_t *w, const double *rho_gj,
                                                     double *rhs)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x + 1;
    if (i > c.N) return;
    const int64_t wi = (i == c.N) ? 2 * w[i] : w[i];
    const double rho = (c.qmP * (double)wi) / c.dz;
    const double rg = (c.flags & PIC_GR_ALPHA) ? rho_gj[i] / gr_alpha_node(c, i) : rho_gj[i];
    const double t = rho - rg;
    rhs[i] = -(c.cpois * t);
}

// phi of eq. (4) from the right-hand side (thomas_body.h); one block.
__global__ __launch_bounds__(256) void k_thomas(Consts c, const double *rhs, double *cp, double *dp,
                                                double *phi)
{
    thomas_block<false>(c, rhs, cp, dp, phi, 1.0);
}

// The same solve for many tubes of a batch at once, one block per listed tube.
__global__ __launch_bounds__(256) void k_thomas_batch(const TubeDev *tubes, const int32_t *list)
{
    const TubeDev &T = tubes[list[blockIdx.x]];
    const Consts c = T.c;
    thomas_block<false>(c, generic(T.rhs), generic(T.cp), generic(T.dp), generic(T.phi), 1.0);
}

// Current of one drift step of the loaded beam, no kick (steady start,
// PIC_B_STEADY_INIT): J_{i+1/2} += S_i(x) - S_i(x + (dt/dz) v), v = u / sqrt(1 + u^2),
// in the push's fixed point.  One atomic per touched face (once per run).
__device__ __forceinline__ void drift_current(const Consts &c, double x, double u, unsigned long long *J)
{
    const int64_t N = c.N;
    double t = u * u;
    t = 1.0 + t;
    const double gam = sqrt(t);
    const double v = u / gam;
    const double x1 = (c.flags & PIC_GR_ALPHA) ? x + c.dtdz * (gr_alpha2(c, x * c.dz) * v) : x + c.dtdz * v;
    const double c0d = floor(x), c1d = floor(x1);
    const int64_t c0 = (int64_t)c0d, c1 = (int64_t)c1d;
    const double F0 = rint((x - c0d) * c.twoP), F1 = rint((x1 - c1d) * c.twoP);
    double va, vb = 0.0;
    bool hb = false;
    if (c1 == c0) {
        va = F1 - F0;
    } else if (c1 > c0) {
        va = c.twoP - F0;
        if (c1 < N) { vb = F1; hb = true; }
    } else {
        va = -F0;
        if (c1 >= 0) { vb = F1 - c.twoP; hb = true; }
    }
    if (va != 0.0) atomicAdd(J + c0, (unsigned long long)(long long)va);
    if (hb && vb != 0.0) atomicAdd(J + c1, (unsigned long long)(long long)vb);
}

__global__ __launch_bounds__(256) void k_drift_current_f64(Consts c, const double *X, const double *U,
                                                           const DevCounters *ctr, unsigned long long *J)
{
    const int64_t n = ctr->n_slots;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
        const double x = X[p];
        if (x >= 0.0) drift_current(c, x, U[p], J);
    }
}

__global__ __launch_bounds__(256) void k_drift_current_f32(Consts c, Streams s, const DevCounters *ctr,
                                                           unsigned long long *J)
{
    const int64_t nl = ctr->n_slots, nh = ctr->n_slots_hi;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < nl + nh; p += (int64_t)gridDim.x * 256) {
        const bool hi = p >= nl;
        const int64_t q = hi ? p - nl : p;
        float off = 0.0f;
        int cell;
        if (hi) cell = hi_slot(s, q, off);
        else { cell = s.CL[q]; off = s.OL[q]; }
        if (cell < 0) continue;
        const double x = (double)cell + (double)off;
        drift_current(c, x, hi ? s.UH[q] : (double)s.UL[q], J);
    }
}

// B_phi = 4 pi R j: (dt/R) B = 4 pi q_m 2^-P J (PIC_GR_ALPHA: divided by alpha at
// the face, from alpha B/R = 4 pi alpha j), then J is cleared.
__global__ __launch_bounds__(256) void k_b_from_current(Consts c, int64_t *J, double *b)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < c.N) {
        const double bi = (c.c4 * (double)J[i]) / c.dtR;
        b[i] = (c.flags & PIC_GR_ALPHA) ? bi / gr_alpha_face(c, i) : bi;
        J[i] = 0;
    }
}

// E_z = -dphi/dz at faces, E_r = phi/R at nodes (PIC_GR_ALPHA: phi/(alpha R)),
// B_phi = 0, J = 0, f32 kick array.
__global__ __launch_bounds__(256) void k_fields_from_phi(Consts c, const double *phi, double *ez,
                                                         double *er, double *b, float *k32, int64_t *j0,
                                                         int64_t *j1, int64_t *j2)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i > c.N) return;
    er[i] = ((c.flags & PIC_GR_ALPHA) ? phi[i] / gr_alpha_node(c, i) : phi[i]) / c.R;
    if (i < c.N) {
        const double e = -((phi[i + 1] - phi[i]) / c.dz);
        ez[i] = e;
        b[i] = 0.0;
        if (k32) k32[i] = (float)(c.qmdt * e);
        j0[i] = 0;
        j1[i] = 0;
        j2[i] = 0;
    }
}

__global__ __launch_bounds__(256) void k_fill_i64(int64_t *p, int64_t n, int64_t v)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

template <int GR>
__global__ __launch_bounds__(256) void k_field_inject(Consts c, FieldArgs a)
{
    field_tile<GR>(c, a, blockIdx.x, 256);
}

// FP32-bulk: the f32 kick array from E_z (after the caller overwrote the fields).
__global__ __launch_bounds__(256) void k_kick(Consts c, const double *ez, float *k32)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < c.N) k32[i] = (float)(c.qmdt * ez[i]);
}

// Check appended particles in slots [base, base + n): 0 <= x < N and u finite.
__global__ __launch_bounds__(256) void k_check_append(Consts c, const double *X, const double *U, int64_t base,
                                                      int64_t n, DevCounters *ctr, int64_t *jumps, int stride)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool bad = false;
    int cell = -1;
    if (i < n) {
        const double x = X[base + i], u = U[base + i];
        bad = !(x >= 0.0 && x < (double)c.N) || !isfinite(u);
        if (!bad) cell = (int)x;
    }
    count_jumps(cell, 128, stride, jumps);
    const int64_t nb = wave_sum_i64(bad ? 1 : 0);
    if (__lane_id() == 0 && nb) atomicAdd((unsigned long long *)&ctr->bad_inputs, (unsigned long long)nb);
}

// Commit n appended particles (slots [n_slots, n_slots + n)) unless any failed the check.
__global__ void k_commit_append(DevCounters *ctr, int64_t n)
{
    if (threadIdx.x == 0 && blockIdx.x == 0 && ctr->bad_inputs == 0) {
        ctr->n_slots += n;
        ctr->n_alive += n;
    }
}

static inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

hipError_t launch_rho_gj(pic_handle *h)
{
    const Consts &c = h->c;
    hipLaunchKernelGGL(k_rho_gj, dim3(grid_for(c.N + 1, 256)), dim3(256), 0, h->stream, c, h->ws.knots,
                       h->ws.rho_gj, h->ws.ctr);
    return hipGetLastError();
}

// Right-hand side of eq. (4) from the loaded charge (before the solve).
hipError_t launch_poisson_rhs(pic_handle *h)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    hipError_t e = launch_moments(h, 0, ProfPtrs{}, w.w, false);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_poisson_rhs, dim3(grid_for(c.N, 256)), dim3(256), 0, h->stream, c, w.w,
                       w.rho_gj, w.rhs);
    return hipGetLastError();
}

// E_z, E_r, B_phi = 0, cleared J and the kick arrays from the solved phi.
hipError_t launch_fields_from_phi(pic_handle *h)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    const int f = h->fbuf;
    hipLaunchKernelGGL(k_fields_from_phi, dim3(grid_for(c.N + 1, 256)), dim3(256), 0, h->stream, c,
                       w.phi, w.ez[f], w.er[f], w.b[f], h->p.precision == PIC_FP32_BULK ? w.k32 : nullptr,
                       w.j[0], w.j[1], w.j[2]);
    if (c.flags & PIC_B_STEADY_INIT) {
        // steady start: B_phi from the current the loaded beam carries (J is clear here)
        unsigned long long *J = (unsigned long long *)w.j[h->jbuf];
        const unsigned g = (unsigned)(h->n_cu * 8);
        const int b = h->pbuf;
        if (h->p.precision == PIC_FP32_BULK)
            hipLaunchKernelGGL(k_drift_current_f32, dim3(g), dim3(256), 0, h->stream, c,
                               Streams{w.cl[b], w.ol[b], w.ul[b], w.hp[b], w.hw[b], w.hg[b], w.uh[b]}, w.ctr, J);
        else
            hipLaunchKernelGGL(k_drift_current_f64, dim3(g), dim3(256), 0, h->stream, c, w.x[b], w.u[b], w.ctr, J);
        hipLaunchKernelGGL(k_b_from_current, dim3(grid_for(c.N, 256)), dim3(256), 0, h->stream, c, w.j[h->jbuf],
                           w.b[f]);
    }
    return hipGetLastError();
}

hipError_t launch_poisson(pic_handle *h)
{
    hipError_t e = launch_poisson_rhs(h);
    if (e != hipSuccess) return e;
    Workspace &w = h->ws;
    hipLaunchKernelGGL(k_thomas, dim3(1), dim3(256), 0, h->stream, h->c, w.rhs, w.cp, w.dp, w.phi);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_fields_from_phi(h);
}

// Solve eq. (4) for the listed tubes of a batch together (one Thomas block per tube).
hipError_t launch_thomas_batch(pic_handle *b, const int32_t *d_list, int n)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_thomas_batch, dim3((unsigned)n), dim3(256), 0, b->stream, b->d_tubes, d_list);
    return hipGetLastError();
}

hipError_t launch_field_inject(pic_handle *h)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    const int f = h->fbuf, g = 1 - h->fbuf;
    const bool f32 = h->p.precision == PIC_FP32_BULK;
    const int b = h->pbuf;
    FieldArgs a{w.ez[f], w.er[f], w.b[f], w.ez[g], w.er[g], w.b[g], w.j[h->jbuf], w.j[1 - h->jbuf],
                f32 ? w.k32 : nullptr, f32 ? nullptr : w.x[b], f32 ? nullptr : w.u[b],
                f32 ? w.cl[b] : nullptr, f32 ? w.ol[b] : nullptr, f32 ? w.ul[b] : nullptr, w.ctr,
                h->d_sched, h->sched_first, h->sched_n,
                h->hist_on ? (unsigned long long *)w.cell_count : nullptr,
                f32 && 0.0 >= h->u_hi ? sort_low_keys(c) : 0};
    if (c.flags & PIC_GR_ALPHA)
        hipLaunchKernelGGL((k_field_inject<1>), dim3(grid_for(c.N, 256)), dim3(256), 0, h->stream, c, a);
    else
        hipLaunchKernelGGL((k_field_inject<0>), dim3(grid_for(c.N, 256 * FIELD_CPT)), dim3(256), 0, h->stream, c, a);
    return hipGetLastError();
}

hipError_t launch_check_append(pic_handle *h, int64_t base, int64_t n)
{
    if (n > 0)
        hipLaunchKernelGGL(k_check_append, dim3(grid_for(n, 256)), dim3(256), 0, h->stream, h->c,
                           h->ws.x[h->pbuf], h->ws.u[h->pbuf], base, n, h->ws.ctr, &h->ws.sc->jumps, (int)jump_stride(n));
    return hipGetLastError();
}

hipError_t launch_commit_append(pic_handle *h, int64_t n)
{
    hipLaunchKernelGGL(k_commit_append, dim3(1), dim3(64), 0, h->stream, h->ws.ctr, n);
    return hipGetLastError();
}


hipError_t launch_zero_i64(pic_handle *h, int64_t *p, int64_t n)
{
    if (n > 0)
        hipLaunchKernelGGL(k_fill_i64, dim3(grid_for(n, 256)), dim3(256), 0, h->stream, p, n, (int64_t)0);
    return hipGetLastError();
}

// The f32 kick array of the FP32-bulk low stream from the current E_z (the
// FP64 path and the high stream form the kick from E_z itself: nothing to do).
hipError_t launch_kick(pic_handle *h)
{
    if (h->p.precision != PIC_FP32_BULK) return hipSuccess;
    hipLaunchKernelGGL(k_kick, dim3(grid_for(h->c.N, 256)), dim3(256), 0, h->stream, h->c, h->ws.ez[h->fbuf],
                       h->ws.k32);
    return hipGetLastError();
}

}  // namespace pcpic
