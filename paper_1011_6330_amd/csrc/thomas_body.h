// thomas_body.h -- the tridiagonal solve of eq. (4) and of its transpose, in the
// operation order of the plain Thomas recurrence, bit for bit.
//
// Rows i = 1..N of phi_{i-1} + b_i phi_i + phi_{i+1} = rhs_i (row N: 2 phi_{N-1}
// in place of phi_{N-1}; transposed: the 2 sits in row N-1's upper entry):
//   m_i = b_i - c'_{i-1}, c'_i = 1/m_i, d'_i = (rhs_i - d'_{i-1})/m_i   (row N with the 2),
//   phi_N = d'_N, phi_i = d'_i - c'_i phi_{i+1}.
// The recurrences are sequential, and what bounds them is the latency of one
// wave's dependent instructions (about 6.5 cycles each).  So one block splits them
// over its waves, in chunks of TH_T rows that move through a pipeline:
//   wave 0   c' of chunk a;
//   wave 2   chunk a-1: m, the operands of the next stage, and a check of every c'
//            against the division 1/m itself, all rows at once;
//   wave 1   d' of the chunk before: quotient from c' (the reciprocal of m) and a
//            residual correction, four dependent operations a row;
//   wave 3   a check of every d' against the division.
// Without the lapse c' has a closed form, -sinh(i t)/sinh((i+1) t) with
// 2 cosh t = -b: wave 2 forms it ahead, and the recurrence is left with m and one
// Newton step from it (three operations).  With the lapse the step starts from the
// line through the two values before (past the first rows, where their difference is
// too large: the hardware estimate there) and is followed by a residual correction.
// A lane holds TH_R consecutive rows, and the value before its first row comes from
// the lane below (DPP): all lanes repeat their rows until the values have passed
// through, which keeps the operands in registers.  (The same chains on one lane,
// operands read from LDS row by row, took 85 cycles a row for d' and 56 for the back
// substitution, most of them in the LDS accesses.)
// A row whose check fails (operands near the ends of the exponent range, where the
// short forms round differently, or a reciprocal within 2^-27 ulp of a rounding
// midpoint) sends its chunk back to be computed with plain divisions, which is then
// taken as it is; so the result is the plain recurrence's in every case, and each
// chunk is computed at most twice.  Without the lapse every row has the same
// diagonal, and once c' repeats it stays fixed.
// 16,384 rows take 0.34 ms (0.42 with the lapse); one lane that ran both recurrences
// with inline range checks took 1.44 ms (3.5), the transposed solve with plain
// divisions 185 ns a row.
#pragma once

#include "pcpic_internal.h"
#include "short_math.h"
#include "wave.h"

namespace pcpic {

constexpr int TH_T = 512;      // rows per chunk
constexpr int TH_R = TH_T / 64;  // consecutive rows per lane of a chain
constexpr int TH_BUF = 4;      // chunks in the pipeline
constexpr int TH_BLOCK = 256;  // threads

struct ThShared {
    double s[TH_BUF][TH_T], c[TH_BUF][TH_T], m[TH_BUF][TH_T], d[TH_BUF][TH_T];
    double b[TH_BUF][TH_T];    // the diagonal with the lapse, else the closed form of c'
    int bad_a, bad_b;
};

// Diagonal of row i (PIC_GR_ALPHA: -(2 + (dz/R)^2 / alpha_i^2)).
__device__ __forceinline__ double th_diag(const Consts &c, int64_t i)
{
    return (c.flags & PIC_GR_ALPHA) ? -(2.0 + c.h2 / gr_alpha2(c, (double)i * c.dz)) : c.bdiag;
}

// Barrier of the block that orders its LDS accesses only: the stores to memory of
// the checked rows need not arrive before the next chunk starts.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ bool th_same(double a, double b)
{
    return __builtin_bit_cast(long long, a) == __builtin_bit_cast(long long, b) || (a != a && b != b);
}

// The value of the lane below (lane 0: `first`), of the lane above (lane 63: `last`).
__device__ __forceinline__ double th_below(double v, double first)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(first), __double2loint(v), 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(first), __double2hiint(v), 0x138, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double th_above(double v, double last)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(last), __double2loint(v), 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(last), __double2hiint(v), 0x130, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Orders a wave's own LDS accesses.
__device__ __forceinline__ void th_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// t of the closed form: 2 cosh t = -b, from w = (-b - 2)/2 (exact).
__device__ __forceinline__ double th_angle(const Consts &c)
{
    const double w = 0.5 * (-c.bdiag - 2.0);
    return log1p(w + sqrt(w * (w + 2.0)));
}
// c'_i = -sinh(i t)/sinh((i+1) t) = -e^-t (1 - e^-2it)/(1 - e^-2(i+1)t), et = e^-t.
__device__ __forceinline__ double th_closed(double i, double t, double et)
{
    return -et * (expm1(-2.0 * i * t) / expm1(-2.0 * (i + 1.0) * t));
}

// Wave 0: c' of the rows of chunk k (cnt of them, the last one row N if last).
__device__ __forceinline__ void th_chunk_c(const Consts &c, ThShared &S, int64_t k, int cnt, bool last, bool plain)
{
    const int q = (int)(k & (TH_BUF - 1)), qp = (int)((k - 1) & (TH_BUF - 1)), lane = (int)__lane_id();
    const bool gr = (c.flags & PIC_GR_ALPHA) != 0;
    const double first = k > 0 ? S.c[qp][TH_T - 1] : 0.0;
    const int nf = last ? cnt - 1 : cnt;         // rows below N
    int t = 0;
    if (!gr && k > 0 && first == S.c[qp][TH_T - 2]) {   // c' has reached its fixed point
        for (int j = lane; j < nf; j += 64) S.c[q][j] = first;
        t = nf;
    } else if (!plain) {
        double b[TH_R], r[TH_R];
#pragma unroll
        for (int j = 0; j < TH_R; ++j) {
            b[j] = S.b[q][lane * TH_R + j];
            r[j] = 0.0;
        }
        const int turns = (nf + TH_R - 1) / TH_R;
        if (gr && k >= 2) {
            const double second = S.c[qp][TH_T - 2];
#pragma unroll 1
            for (int n = 0; n < turns; ++n) {
                double p = th_below(r[TH_R - 1], first), p2 = th_below(r[TH_R - 2], second);
#pragma unroll
                for (int j = 0; j < TH_R; ++j) {
                    const double m = b[j] - p, y0 = fma(2.0, p, -p2);
                    const double y = fma(y0, fma(-m, y0, 1.0), y0);
                    p2 = p;
                    r[j] = p = fma(fma(-m, y, 1.0), y, y);
                }
            }
        } else if (gr) {
#pragma unroll 1
            for (int n = 0; n < turns; ++n) {
                double p = th_below(r[TH_R - 1], first);
#pragma unroll
                for (int j = 0; j < TH_R; ++j) {
                    const double m = b[j] - p, y = nr_recip(m);
                    r[j] = p = fma(fma(-m, y, 1.0), y, y);
                }
            }
        } else {
#pragma unroll 1
            for (int n = 0; n < turns; ++n) {
                double p = th_below(r[TH_R - 1], first);
#pragma unroll
                for (int j = 0; j < TH_R; ++j) {
                    const double m = c.bdiag - p;
                    r[j] = p = fma(fma(-m, b[j], 1.0), b[j], b[j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < TH_R; ++j) S.c[q][lane * TH_R + j] = r[j];
        t = nf;
    }
    th_wave_sync();
    if (lane != 0 || t == cnt) return;
    double p = t > 0 ? S.c[q][t - 1] : first;
    for (; t < cnt; ++t) {
        const double a = last && t == cnt - 1 ? 2.0 : 1.0;
        const double m = (gr ? S.b[q][t] : c.bdiag) - a * p;
        p = 1.0 / m;
        S.c[q][t] = p;
    }
}

// Wave 1: d' of the rows of chunk k.
template <bool TRANS>
__device__ __forceinline__ void th_chunk_d(ThShared &S, int64_t k, int cnt, bool last, bool plain)
{
    const int q = (int)(k & (TH_BUF - 1)), qp = (int)((k - 1) & (TH_BUF - 1)), lane = (int)__lane_id();
    const double first = k > 0 ? S.d[qp][TH_T - 1] : 0.0;
    const int nf = last ? cnt - 1 : cnt;
    int t = 0;
    // a chain that has left the middle of the exponent range would fail its checks
    if (!plain && fabs(first) <= 0x1p+400 && (first == 0.0 || fabs(first) >= 0x1p-500)) {
        double s[TH_R], r[TH_R], m[TH_R], d[TH_R];
#pragma unroll
        for (int j = 0; j < TH_R; ++j) {
            s[j] = S.s[q][lane * TH_R + j];
            r[j] = S.c[q][lane * TH_R + j];
            m[j] = S.m[q][lane * TH_R + j];
            d[j] = 0.0;
        }
        const int turns = (nf + TH_R - 1) / TH_R;
#pragma unroll 1
        for (int n = 0; n < turns; ++n) {
            double p = th_below(d[TH_R - 1], first);
#pragma unroll
            for (int j = 0; j < TH_R; ++j) d[j] = p = nr_div(s[j] - p, m[j], r[j]);
        }
#pragma unroll
        for (int j = 0; j < TH_R; ++j) S.d[q][lane * TH_R + j] = d[j];
        t = nf;
    }
    th_wave_sync();
    if (lane != 0 || t == cnt) return;
    double p = t > 0 ? S.d[q][t - 1] : first;
    for (; t < cnt; ++t) {
        const double a = !TRANS && last && t == cnt - 1 ? 2.0 : 1.0;
        p = (S.s[q][t] - a * p) / S.m[q][t];
        S.d[q][t] = p;
    }
}

// Wave 0: phi of the rows of a chunk (cnt of them, TOP: the last one row N) from its
// d', c' and phi of the row above the chunk.
template <bool TOP>
__device__ __forceinline__ void th_chunk_phi(const double *D, const double *C, double *F, int cnt, double above)
{
    const int lane = (int)__lane_id();
    double d[TH_R], c[TH_R], f[TH_R];
#pragma unroll
    for (int j = 0; j < TH_R; ++j) {
        d[j] = D[lane * TH_R + j];
        c[j] = C[lane * TH_R + j];
        f[j] = 0.0;
    }
    const int turns = (cnt + TH_R - 1) / TH_R;
#pragma unroll 1
    for (int n = 0; n < turns; ++n) {
        double p = th_above(f[0], above);
#pragma unroll
        for (int j = TH_R - 1; j >= 0; --j) {
            p = d[j] - c[j] * p;
            if (TOP) p = lane * TH_R + j >= cnt - 1 ? d[j] : p;   // phi_N = d'_N
            f[j] = p;
        }
    }
#pragma unroll
    for (int j = 0; j < TH_R; ++j) F[lane * TH_R + j] = f[j];
}

// The solve by one block of TH_BLOCK threads: phi[1..N] = scale times the solution
// (scale = 1: the solution itself), phi[0] = 0; cp, dp: scratch of N + 1 doubles.
template <bool TRANS>
__device__ __forceinline__ void thomas_block(const Consts &c, const double *rhs, double *cp, double *dp, double *phi,
                                             double scale)
{
    __shared__ ThShared S;
    const int64_t N = c.N;
    const int tid = (int)threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool gr = (c.flags & PIC_GR_ALPHA) != 0;
    const int64_t K = (N + TH_T - 1) / TH_T;
    auto rows = [&](int64_t k) { return (int)(N - k * TH_T < TH_T ? N - k * TH_T : TH_T); };
    const int h = tid & 63;
    // chunks started by a stage (ia, ib) and checked (va, vb); pa, pb: computed plainly
    int64_t ia = 0, va = 0, ib = 0, vb = 0;
    bool pa = false, pb = false;
    const double ang = th_angle(c), eang = exp(-ang);
    auto before_c = [&](int64_t k, int from, int step) {     // S.b of chunk k
        const int q = (int)(k & (TH_BUF - 1));
        for (int t = from; t < rows(k); t += step) {
            const int64_t i = 1 + k * TH_T + t;
            S.b[q][t] = gr ? th_diag(c, i) : th_closed((double)i, ang, eang);
        }
    };
    before_c(0, tid, TH_BLOCK);
    if (tid == 0) S.bad_a = S.bad_b = 0;
    __syncthreads();
    while (vb < K) {
        const bool do_a = ia < K && ia < vb + TH_BUF && ia - va <= 1;
        const bool do_va = va < ia;
        const bool do_b = ib < va && ib - vb <= 1;
        const bool do_vb = vb < ib;
        if (wv == 0) {
            if (do_a) th_chunk_c(c, S, ia, rows(ia), ia == K - 1, pa);
        } else if (wv == 1) {
            if (do_b) th_chunk_d<TRANS>(S, ib, rows(ib), ib == K - 1, pb);
        } else if (wv == 2) {
            if (ia + 1 < K) before_c(ia + 1, h, 64);
            if (do_va) {
                const int q = (int)(va & (TH_BUF - 1)), qp = (int)((va - 1) & (TH_BUF - 1));
                const int64_t i0 = 1 + va * TH_T;
                bool bad = false;
                for (int t = h; t < rows(va); t += 64) {
                    const int64_t i = i0 + t;
                    const double sv = rhs[i];
                    const double prev = t > 0 ? S.c[q][t - 1] : (va > 0 ? S.c[qp][TH_T - 1] : 0.0);
                    const double m = (gr ? S.b[q][t] : c.bdiag) - (i == N ? 2.0 : 1.0) * prev;
                    const double cc = S.c[q][t];
                    bad = bad || !th_same(cc, 1.0 / m);
                    S.m[q][t] = m;
                    S.s[q][t] = sv;
                    cp[i] = TRANS && i == N - 1 ? 2.0 * cc : cc;
                }
                if (bad) S.bad_a = 1;
            }
        } else {
            if (do_vb) {
                const int q = (int)(vb & (TH_BUF - 1)), qp = (int)((vb - 1) & (TH_BUF - 1));
                const int64_t i0 = 1 + vb * TH_T;
                bool bad = false;
                for (int t = h; t < rows(vb); t += 64) {
                    const int64_t i = i0 + t;
                    const double prev = t > 0 ? S.d[q][t - 1] : (vb > 0 ? S.d[qp][TH_T - 1] : 0.0);
                    const double n = S.s[q][t] - (!TRANS && i == N ? 2.0 : 1.0) * prev;
                    const double dd = S.d[q][t];
                    bad = bad || !th_same(dd, n / S.m[q][t]);
                    dp[i] = dd;
                }
                if (bad) S.bad_b = 1;
            }
        }
        lds_barrier();
        const bool again_a = do_va && S.bad_a != 0, again_b = do_vb && S.bad_b != 0;
        // a chunk computed plainly is taken as it is: the flag pa (pb) belongs to the
        // chunk at va (vb) once its stage has run it
        const bool plain_a = pa && do_va, plain_b = pb && do_vb;
        lds_barrier();
        if (tid == 0) S.bad_a = S.bad_b = 0;
        if (again_a && !plain_a) {
            ia = va;
            pa = true;
        } else {
            if (do_va) ++va;
            if (do_a) ++ia;
            if (plain_a) pa = false;
        }
        if (again_b && !plain_b) {
            ib = vb;
            pb = true;
        } else {
            if (do_vb) ++vb;
            if (do_b) ++ib;
            if (plain_b) pb = false;
        }
        lds_barrier();
    }
    __syncthreads();
    // back substitution, chunks downwards: wave 0 runs the chain on one while the
    // others bring the operands of the next and store the one before
    auto bring = [&](int64_t k, int from, int step) {
        const int q = (int)(k & 1);
        for (int t = from; t < rows(k); t += step) {
            S.d[q][t] = dp[1 + k * TH_T + t];
            S.c[q][t] = cp[1 + k * TH_T + t];
        }
    };
    auto store = [&](int64_t k, int from, int step) {
        const int q = (int)(k & 1);
        for (int t = from; t < rows(k); t += step) {
            const double v = S.s[q][t];
            phi[1 + k * TH_T + t] = scale == 1.0 ? v : scale * v;
        }
    };
    bring(K - 1, tid, TH_BLOCK);
    __syncthreads();
    for (int64_t k = K - 1; k >= 0; --k) {
        if (wv == 0) {
            const int q = (int)(k & 1);
            if (k == K - 1) th_chunk_phi<true>(S.d[q], S.c[q], S.s[q], rows(k), 0.0);
            else th_chunk_phi<false>(S.d[q], S.c[q], S.s[q], TH_T, S.s[q ^ 1][0]);
        } else {
            if (k < K - 1) store(k + 1, tid - 64, TH_BLOCK - 64);
            if (k > 0) bring(k - 1, tid - 64, TH_BLOCK - 64);
        }
        lds_barrier();
    }
    store(0, tid, TH_BLOCK);
    if (tid == 0) phi[0] = 0.0;
}

}  // namespace pcpic
