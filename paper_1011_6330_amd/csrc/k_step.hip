// k_step.hip -- fused steps: one kernel per step in place of a push and a field
// kernel, for tubes and batches small enough that a step's time is its kernels'
// latency.
//
// A run of m steps is m + 1 kernels.  The first pushes in the fields as they are;
// each further one takes the field update of the step before and the push of its
// own step together: the push blocks form the E_z values they gather from the
// fields before the update and that step's current (updated_ez, the expressions of
// the field update, so the same bits), while the field blocks write the updated
// fields into the other buffers; the last kernel is the field update of the last
// step.  Nothing a kernel reads is written by it:
//   * three current buffers take turns (run_j): step s reads J of s-1, adds to J of s,
//     and its field blocks clear the third, J of s+1 (likewise the node-0 tallies);
//   * the slot count the pushes take has two words in turn (StepScratch);
//   * the particles injected at the end of step s-1 all start from x = 0, u = 0, so
//     the block that injects them also pushes them (push_injected), and the push
//     blocks take the slots before the injection only.
// What bounds a small step: the push and the field kernel of the 1,024-cell tube
// (4e3 particles) take 4.4 and 3.0 us, a chain of dependent memory latencies each,
// where an empty kernel of a graph takes 1.7.  Per step with its share of the sort
// (every 64 steps), push and field kernels against fused: 2e5 particles 10.7 -> 6.6
// us, 7e5 11.9 -> 9.5.  step_route.h says which tubes and batches take them, by the
// slots that they are expected to hold, not by their capacity: eight cold tubes of
// 11,036 cells, 1e4 of whose 5.4e5 slots each are taken, 16.1 -> 11.1 us.
#include <math.h>

#include "field_body.h"
#include "pcpic_internal.h"
#include "push_body.h"

namespace pcpic {

// Nontemporal accesses in ascending order, as the separate pushes of the same sizes take
// (push_nontemporal; a fused FP64 tube has 24 MiB of slots at most).
constexpr int STEP_BLOCK = 128;
constexpr int STEP_TILE_F64 = STEP_BLOCK * 2;
constexpr int STEP_TILE_F32 = STEP_BLOCK * F32_PPT_HI;
constexpr int STEP_FACES = STEP_BLOCK * FIELD_CPT;    // faces per field block
static_assert(F32_PPT_LO == F32_PPT_HI, "one item size for both streams");

// The field block `tile` of a run's first kernel: clears the current buffer of the
// second step and notes the slot count.
__device__ __forceinline__ void step_first_fields(const Consts &c, int64_t *jclear, const DevCounters *ctr,
                                                  StepScratch *sc, int64_t *rec, int64_t tile)
{
    const int64_t i = tile * STEP_FACES + threadIdx.x;
#pragma unroll
    for (int k = 0; k < FIELD_CPT; ++k)
        if (i + k * STEP_BLOCK < c.N) jclear[i + k * STEP_BLOCK] = 0;
    if (tile == 0 && threadIdx.x == 0) {
        sc->n[0] = ctr->n_slots;
        if (rec) *rec = ctr->n_slots;
    }
}

// One tube: field blocks first, then the push blocks (at capacity; those past the
// slots return).  UPD 0: the first kernel of a run.
template <int UPD>
__global__ __launch_bounds__(STEP_BLOCK) void k_step_f64(Consts c, FieldArgs f, PushArgs a, int field_blocks)
{
    const int b = (int)blockIdx.x;
    if (b < field_blocks) {
        if (UPD) field_tile(c, f, b, STEP_BLOCK);
        else step_first_fields(c, f.jnext, f.ctr, f.sc, f.rec, b);
        return;
    }
    const int64_t n = UPD ? f.sc->n[f.n_in] : f.ctr->n_slots;
    const int64_t tile0 = (int64_t)(b - field_blocks) * STEP_TILE_F64;
    if (tile0 < n) push_tile_f64<STEP_BLOCK, 2, 1, 0, UPD>(c, a, n, tile0);
}

template <int UPD>
__global__ __launch_bounds__(STEP_BLOCK) void k_step_f32(Consts c, FieldArgs f, Push32Args a, int field_blocks)
{
    const int b = (int)blockIdx.x;
    if (b < field_blocks) {
        if (UPD) field_tile(c, f, b, STEP_BLOCK);
        else step_first_fields(c, f.jnext, f.ctr, f.sc, f.rec, b);
        return;
    }
    const int64_t n = UPD ? f.sc->n[f.n_in] : f.ctr->n_slots;
    push_item_f32<STEP_BLOCK, 1, UPD>(c, a, b - field_blocks, n, f.ctr->n_slots_hi);
}

// The arguments of kernel s of a run (s = m + 1: the closing field update) that
// depend on its place in the run alone.
static void place_in_run(FieldArgs &f, int64_t s, bool last)
{
    f.w_in = (int)((s + 1) % 3);            // tally of step s - 1
    f.w_add = (int)((s - 1) % 3);
    f.w_zero = (int)(s % 3);
    f.n_in = (int)(s & 1);
    f.push = s > 1 && !last;
}

static unsigned field_blocks_of(const Consts &c, int bs) { return (unsigned)((c.N + bs * FIELD_CPT - 1) / (bs * FIELD_CPT)); }

hipError_t launch_run_step(pic_handle *h, int64_t m, int64_t s, const RunPtrs &r, bool hist, int64_t *rec)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    const bool f32 = h->p.precision == PIC_FP32_BULK;
    const int jb = h->jbuf, b = h->pbuf;
    unsigned long long *J = (unsigned long long *)w.j[run_j(jb, m, s)];
    unsigned long long *cnt = hist ? (unsigned long long *)w.cell_count : nullptr;
    FieldArgs f{};
    f.ezo = r.ez; f.ero = r.er; f.bo = r.b;
    f.ezn = r.ezn; f.ern = r.ern; f.bn = r.bn;
    f.j = s > 1 ? w.j[run_j(jb, m, s - 1)] : nullptr;
    f.jnext = w.j[run_j(jb, m, s + 1)];
    f.k32 = f32 ? w.k32 : nullptr;
    f.X = r.X; f.U = r.U; f.Xo = r.Xo; f.Uo = r.Uo;
    if (f32) { f.CL = w.cl[b]; f.OL = w.ol[b]; f.UL = w.ul[b]; }
    f.ctr = w.ctr;
    f.sched = h->d_sched; f.sched_first = h->sched_first; f.sched_n = h->sched_n;
    f.sc = w.sc;
    f.rec = rec;
    f.Jn = J;
    f.push_hist = cnt;
    f.u_hi = h->u_hi;
    place_in_run(f, s, false);
    const PrevStep prev{r.ez, r.er, r.b, f.j};
    const unsigned fb = field_blocks_of(c, STEP_BLOCK);
    if (f32) {
        Push32Args a{w.cl[b], w.ol[b], w.ul[b], w.hp[b], w.hw[b], w.hg[b], w.uh[b], w.k32, r.ez, J, w.ctr,
                     &w.sc->w0[f.w_add], cnt, h->u_hi, prev};
        const unsigned g = fb + (unsigned)((c.cap + STEP_TILE_F32 - 1) / STEP_TILE_F32 + 1);
        if (s > 1) hipLaunchKernelGGL((k_step_f32<1>), dim3(g), dim3(STEP_BLOCK), 0, h->stream, c, f, a, (int)fb);
        else hipLaunchKernelGGL((k_step_f32<0>), dim3(g), dim3(STEP_BLOCK), 0, h->stream, c, f, a, (int)fb);
    } else {
        PushArgs a{r.X, r.U, r.Xo, r.Uo, r.ez, J, w.ctr, &w.sc->w0[f.w_add], cnt, prev};
        const unsigned g = fb + (unsigned)((c.cap + STEP_TILE_F64 - 1) / STEP_TILE_F64);
        if (s > 1) hipLaunchKernelGGL((k_step_f64<1>), dim3(g), dim3(STEP_BLOCK), 0, h->stream, c, f, a, (int)fb);
        else hipLaunchKernelGGL((k_step_f64<0>), dim3(g), dim3(STEP_BLOCK), 0, h->stream, c, f, a, (int)fb);
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_run_end(Consts c, FieldArgs f)
{
    field_tile(c, f, blockIdx.x, 256);
}

// The closing field update of a run of m steps.
hipError_t launch_run_end(pic_handle *h, int64_t m, const RunPtrs &r, bool hist, int64_t *rec)
{
    const Consts &c = h->c;
    Workspace &w = h->ws;
    const bool f32 = h->p.precision == PIC_FP32_BULK;
    const int jb = h->jbuf, b = h->pbuf;
    FieldArgs f{};
    f.ezo = r.ez; f.ero = r.er; f.bo = r.b;
    f.ezn = r.ezn; f.ern = r.ern; f.bn = r.bn;
    f.j = w.j[run_j(jb, m, m)];
    f.jnext = w.j[run_j(jb, m, run_moves(m) ? m : m - 1)];
    f.jmove = run_moves(m) ? w.j[run_j(jb, m, m - 1)] : nullptr;
    f.k32 = f32 ? w.k32 : nullptr;
    f.X = r.X; f.U = r.U;
    if (f32) { f.CL = w.cl[b]; f.OL = w.ol[b]; f.UL = w.ul[b]; }
    f.ctr = w.ctr;
    f.sched = h->d_sched; f.sched_first = h->sched_first; f.sched_n = h->sched_n;
    f.hist = hist ? (unsigned long long *)w.cell_count : nullptr;
    f.inj_key = f32 && 0.0 >= h->u_hi ? sort_low_keys(c) : 0;
    f.sc = w.sc;
    f.rec = rec;
    place_in_run(f, m + 1, true);
    hipLaunchKernelGGL(k_run_end, dim3(field_blocks_of(c, 256)), dim3(256), 0, h->stream, c, f);
    h->jbuf ^= (int)(m & 1);
    return hipGetLastError();
}

// ------------------------------------------------------------------------
// batches: every tube's field and push blocks in one grid
// ------------------------------------------------------------------------

struct BatchRunArgs {
    const TubeDev *tubes;
    const int64_t *pref;     // [n_tubes + 1] first block of each tube (its field blocks, then its push blocks at capacity)
    const int32_t *map;      // block -> tube
    int fb, pb;              // field and particle buffer parities
    int j_in, j_add, j_clear, j_move;   // j_move: -1, or the buffer that receives j_in
    int w_in, w_add, w_zero, n_in;
    int hist;                // the last step before a sort
};

// PART 0: the first kernel of a run, 1: field update and push, 2: the closing field update.
template <int F32, int PART>
__global__ __launch_bounds__(STEP_BLOCK) void k_batch_step(BatchRunArgs r)
{
    const int t = r.map[blockIdx.x];
    const TubeDev &T = r.tubes[t];
    const Consts c = T.c;
    const int64_t b = blockIdx.x - r.pref[t], fblocks = (c.N + STEP_FACES - 1) / STEP_FACES;
    DevCounters *ctr = generic(T.ctr);
    StepScratch *sc = generic(T.sc);
    unsigned long long *J = (unsigned long long *)generic(T.j[r.j_add]);
    unsigned long long *cnt = r.hist ? (unsigned long long *)generic(T.cell_count) : nullptr;
    const int g = r.fb ^ 1;
    if (b < fblocks) {
        if (PART == 0) {
            step_first_fields(c, generic(T.j[r.j_clear]), ctr, sc, nullptr, b);
            return;
        }
        FieldArgs f{};
        f.ezo = generic(T.ez[r.fb]); f.ero = generic(T.er[r.fb]); f.bo = generic(T.b[r.fb]);
        f.ezn = generic(T.ez[g]); f.ern = generic(T.er[g]); f.bn = generic(T.b[g]);
        f.j = generic(T.j[r.j_in]);
        f.jnext = generic(T.j[r.j_clear]);
        if (PART == 2 && r.j_move >= 0) f.jmove = generic(T.j[r.j_move]);
        f.ctr = ctr;
        f.sc = sc;
        f.w_in = r.w_in; f.w_add = r.w_add; f.w_zero = r.w_zero; f.n_in = r.n_in;
        if (F32) {
            f.k32 = generic(T.k32);
            f.CL = generic(T.cl[r.pb]); f.OL = generic(T.ol[r.pb]); f.UL = generic(T.ul[r.pb]);
            f.u_hi = T.u_hi;
        } else {
            f.X = f.Xo = generic(T.x[r.pb]);
            f.U = f.Uo = generic(T.u[r.pb]);
        }
        if (PART == 1) {
            f.push = 1;
            f.Jn = J;
            f.push_hist = cnt;
        } else {
            f.hist = cnt;
            f.inj_key = F32 && 0.0 >= T.u_hi ? sort_low_keys(c) : 0;
        }
        field_tile(c, f, b, STEP_BLOCK);
        return;
    }
    if (PART == 2) return;
    const int64_t n = PART == 1 ? sc->n[r.n_in] : ctr->n_slots;
    const PrevStep prev{generic(T.ez[r.fb]), generic(T.er[r.fb]), generic(T.b[r.fb]), generic(T.j[r.j_in])};
    if (F32) {
        Push32Args a{generic(T.cl[r.pb]), generic(T.ol[r.pb]), generic(T.ul[r.pb]), generic(T.hp[r.pb]),
                     generic(T.hw[r.pb]), generic(T.hg[r.pb]), generic(T.uh[r.pb]), generic(T.k32), generic(T.ez[r.fb]),
                     J, ctr, &sc->w0[r.w_add], cnt, T.u_hi, prev};
        push_item_f32<STEP_BLOCK, 1, PART == 1>(c, a, b - fblocks, n, ctr->n_slots_hi);
    } else {
        const int64_t tile0 = (b - fblocks) * STEP_TILE_F64;
        if (tile0 >= n) return;
        PushArgs a{generic(T.x[r.pb]), generic(T.u[r.pb]), generic(T.x[r.pb]), generic(T.u[r.pb]), generic(T.ez[r.fb]),
                   J, ctr, &sc->w0[r.w_add], cnt, prev};
        push_tile_f64<STEP_BLOCK, 2, 1, 0, PART == 1>(c, a, n, tile0);
    }
}

// Blocks of one tube of a batch in a run's kernels.
int64_t run_blocks(const pic_params &p)
{
    const int64_t f = (p.n_cells + STEP_FACES - 1) / STEP_FACES;
    return f + (p.precision == PIC_FP32_BULK ? (p.capacity + STEP_TILE_F32 - 1) / STEP_TILE_F32 + 1
                                             : (p.capacity + STEP_TILE_F64 - 1) / STEP_TILE_F64);
}

// m steps of every tube of a batch (the caller moves the tubes' buffers on).
hipError_t launch_batch_run(pic_handle *h, int64_t m, bool hist_last)
{
    pic_handle *t0 = h->tubes[0];
    const bool f32 = t0->p.precision == PIC_FP32_BULK;
    const int jb = t0->jbuf;
    const dim3 g((unsigned)h->batch_run_blocks), bl(STEP_BLOCK);
    int fb = t0->fbuf;
    for (int64_t s = 1; s <= m + 1; ++s) {
        FieldArgs f{};
        place_in_run(f, s, s > m);
        const bool move = s > m && run_moves(m);
        BatchRunArgs r{h->d_tubes, h->d_run_pref, h->d_run_map, fb, t0->pbuf,
                       run_j(jb, m, s - 1), run_j(jb, m, s), run_j(jb, m, s <= m ? s + 1 : (move ? m : m - 1)),
                       move ? run_j(jb, m, m - 1) : -1,
                       f.w_in, f.w_add, f.w_zero, f.n_in, hist_last && s >= m ? 1 : 0};
        if (f32) {
            if (s == 1) hipLaunchKernelGGL((k_batch_step<1, 0>), g, bl, 0, h->stream, r);
            else if (s <= m) hipLaunchKernelGGL((k_batch_step<1, 1>), g, bl, 0, h->stream, r);
            else hipLaunchKernelGGL((k_batch_step<1, 2>), g, bl, 0, h->stream, r);
        } else {
            if (s == 1) hipLaunchKernelGGL((k_batch_step<0, 0>), g, bl, 0, h->stream, r);
            else if (s <= m) hipLaunchKernelGGL((k_batch_step<0, 1>), g, bl, 0, h->stream, r);
            else hipLaunchKernelGGL((k_batch_step<0, 2>), g, bl, 0, h->stream, r);
        }
        if (s > 1) fb ^= 1;
    }
    return hipGetLastError();
}

// m steps of a tube in place; rec (or null): the slot counts before each step and
// after the last, m + 1 of them.
hipError_t launch_run(pic_handle *h, int64_t m, bool hist_last, int64_t *rec)
{
    Workspace &w = h->ws;
    hipError_t e = hipSuccess;
    for (int64_t s = 1; s <= m + 1 && e == hipSuccess; ++s) {
        const int f = h->fbuf, b = h->pbuf;
        const RunPtrs r{w.ez[f], w.er[f], w.b[f], w.ez[f ^ 1], w.er[f ^ 1], w.b[f ^ 1], w.x[b], w.u[b], w.x[b], w.u[b]};
        int64_t *n = rec ? rec + s - 1 : nullptr;
        if (s <= m) e = launch_run_step(h, m, s, r, hist_last && s == m, n);
        else e = launch_run_end(h, m, r, hist_last, n);
        if (s > 1) h->fbuf ^= 1;
    }
    return e;
}

}  // namespace pcpic
