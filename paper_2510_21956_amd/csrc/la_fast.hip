// D = 256 as passes of the D = 128 matrix-core kernels (la_split.hip) over blocks of 128 columns
// (split_forward, split_backward, split_prefill).
#include "la_blocks.h"

namespace la {

// Head size 256 on the D = 128 kernels.  With q = [q1 q2], k = [k1 k2] (halves of 128) the
// weight a + b q.k is (a + b q1.k1) + (0 + b q2.k2), and with v = [v1 v2] every sum of
// Sec. 3.1 / 3.2 splits into blocks: the numerator of output half j is the sum over i of
// the numerators of the D = 128 problems (q_i, k_i, v_j) with coefficients (a, b) for i = 1
// and (0, b) for i = 2, g is the sum of their denominators, and likewise
//   dq_i = sum_j dq(q_i, k_i, v_j; o_j, dO_j, g),   dk_i = sum_j dk(...),   dv_j = sum_i dv(...)
// where the blocks (o_j, dO_j) and the full g stand for the stored set of the block problem
// (delta = o . OmegaHat splits over j as well).  Four passes of the D = 128 kernels over column
// blocks of the 256-wide rows, each adding to what the previous ones left in the outputs.
// `pl` is the plan of the D = 128 problem; behind that plan's workspace the forward pass keeps
// the first pass's share of g and, for bf16, its undivided numerator in fp32, and the backward
// pass, for bf16, the first share of every gradient block in fp32 (split_scratch).  With `saved` every
// forward pass hands its sums at the segment boundaries to the backward pass on the same blocks, which
// then runs no sums kernel and no scan (64 slices of 4096 rows, a step without and with: fp32 3390 and 3125 us,
// bf16 1700 and 1556; 8 of 8000, bf16 650 and 580).
static const void *col_block(const void *p, int j, la_dtype dt)
{
    return (const char *)p + (size_t)128 * j * (dt == LA_F32 ? 4 : 2);
}
static void *col_block(void *p, int j, la_dtype dt)
{
    return (char *)p + (size_t)128 * j * (dt == LA_F32 ? 4 : 2);
}

la_status split_prefill(const Problem &pr, const Plan &pl, const void *K, const void *V, float *ws,
                        float *state, int accumulate, hipStream_t st)
{
    Problem p = pr;
    p.D = 128;
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            la_status s = planes_totals(p, pl, 256, col_block(K, i, pr.dt), col_block(V, j, pr.dt), ws, st);
            if (s != LA_OK) return s;
            s = state_block_from_totals(ws, state, pr.BH, pl.nseg, pl.slot_floats, i, j, pr.N,
                                        accumulate, st);
            if (s != LA_OK) return s;
        }
    return LA_OK;
}

// Hand-over of pass (i, j) inside the buffer of all four.
static float *saved_block(float *saved, const Plan &pl, int i, int j)
{
    return saved ? saved + (size_t)(2 * i + j) * (pl.saved_bytes / sizeof(float)) : nullptr;
}

la_status split_forward(const Problem &pr, const Plan &pl, const void *Q, const void *K,
                        const void *V, void *O, float *G, float *ws, float *saved, hipStream_t st,
                        Tracer &tc)
{
    const SplitScratch sc = split_scratch(pl, (size_t)pr.BH * pr.N, pr.dt, 0);
    float *gpart = ws + sc.g_off, *fraw = ws + sc.f_off;
    Problem p = pr;
    p.D = 128;
    Tracer quiet(nullptr, st);  // the caller's trace gets one mark per pass, not per kernel
    for (int j = 0; j < 2; ++j) {
        const void *Vj = col_block(V, j, pr.dt);
        void *Oj = col_block(O, j, pr.dt);
        for (int i = 0; i < 2; ++i) {
            p.a = i == 0 ? pr.a : 0.f;
            const la_status s = planes_forward(p, pl, 256, col_block(Q, i, pr.dt), col_block(K, i, pr.dt),
                                               Vj, Oj, i == 0 ? gpart : (j == 1 ? G : nullptr), ws,
                                               saved_block(saved, pl, i, j), st, quiet, i == 0 ? XF_RAW : XF_ACC,
                                               i == 0 ? nullptr : gpart, fraw);
            if (s != LA_OK) return s;
            tc.mark("fwd_block_pass");
        }
    }
    return LA_OK;
}

// dK == nullptr: the ascending sweeps only (dQ).
la_status split_backward(const Problem &pr, const Plan &pl, const void *Q, const void *K,
                         const void *V, const void *O, const float *G, const void *dO, void *dQ,
                         void *dK, void *dV, float *ws, const float *saved, hipStream_t st, Tracer &tc)
{
    const SplitScratch sc = split_scratch(pl, (size_t)pr.BH * pr.N, pr.dt, 1);
    Problem p = pr;
    p.D = 128;
    Tracer quiet(nullptr, st);  // the caller's trace gets one mark per pass, not per kernel
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            p.a = i == 0 ? pr.a : 0.f;
            BlockPass bp;
            // dQ_i and dK_i are complete after j = 1, dV_j after i = 1
            bp.xflags = (j == 1 ? 1 | 2 : 0) | (i == 1 ? 4 : 0);
            bp.Pq = ws + sc.q_off;
            bp.Pk = ws + sc.k_off;
            bp.Pv = ws + sc.v_off + (size_t)j * pr.BH * pr.N * 128;
            const la_status s = planes_backward(
                p, pl, 256, col_block(Q, i, pr.dt), col_block(K, i, pr.dt), col_block(V, j, pr.dt),
                col_block(O, j, pr.dt), G, col_block(dO, j, pr.dt), col_block(dQ, i, pr.dt),
                dK ? col_block(dK, i, pr.dt) : nullptr, dK ? col_block(dV, j, pr.dt) : nullptr, ws,
                saved_block(const_cast<float *>(saved), pl, i, j), st, quiet, bp);
            if (s != LA_OK) return s;
            tc.mark("bwd_block_pass");
        }
    return LA_OK;
}

}  // namespace la
