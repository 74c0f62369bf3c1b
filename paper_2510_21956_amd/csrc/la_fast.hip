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
// then forms none (a step without and with, us: 64 slices of 4096 rows, fp32 3568 and 3328, bf16 1661 and 1584; 8 of
// 8000, bf16 652 and 608).
//
// Whether a hand-over buffer holds this problem's sums is for the backward pass to find out: the buffer is
// optional, and a forward call that was given none (or one it could not use) succeeds all the same.  So the
// forward pass leaves the last row of every slice's O in it, under a key of the problem, and the backward pass
// compares that with the O it is given: sums of other inputs, or memory that no forward pass wrote, are passed
// over, slice by slice.  The sums kernels are launched either way and return at once where the sums hold (20 us
// a step, witness included).
namespace {

// What the segments and the layout of the sums depend on.
uint32_t problem_key(const Problem &pr, const Plan &pl)
{
    uint32_t k = 0x9e3779b9u;
    for (uint32_t x : {(uint32_t)pr.BH, (uint32_t)pr.N, (uint32_t)pr.causal, (uint32_t)pr.dt, (uint32_t)pl.nseg,
                       (uint32_t)pl.seg_len, (uint32_t)(pl.map.cost_seg > 0)}) {
        k = (k ^ x) * 0x85ebca6bu;
        k ^= k >> 15;
    }
    return k;
}
// One wave a slice; a row of O is `words` (128 or 256) words.
__global__ __launch_bounds__(64) void k_leave_witness(const uint32_t *__restrict__ O, uint32_t *__restrict__ wit,
                                                      int N, int words, uint32_t key)
{
    const uint32_t *row = O + ((size_t)blockIdx.x * N + N - 1) * words;
    uint32_t *w = wit + (size_t)blockIdx.x * kWitnessWords;
    for (int i = threadIdx.x; i < words; i += 64) w[i] = row[i] ^ key;
}
__global__ __launch_bounds__(64) void k_check_witness(const uint32_t *__restrict__ O,
                                                      const uint32_t *__restrict__ wit, int *__restrict__ handed,
                                                      int N, int words, uint32_t key)
{
    const uint32_t *row = O + ((size_t)blockIdx.x * N + N - 1) * words;
    const uint32_t *w = wit + (size_t)blockIdx.x * kWitnessWords;
    uint32_t diff = 0;
    for (int i = threadIdx.x; i < words; i += 64) diff |= w[i] ^ row[i] ^ key;
    const int same = __all(diff == 0);
    if (threadIdx.x == 0) handed[blockIdx.x] = same;
}
int row_words(la_dtype dt) { return dt == LA_F32 ? 256 : 128; }

}  // namespace

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

// Hand-over of pass (i, j) inside the buffer of all four; block 4 is the witness.
template <typename F>
static F *saved_block(F *saved, const Plan &pl, int block)
{
    return saved ? saved + (size_t)block * (pl.saved_bytes / sizeof(float)) : nullptr;
}

la_status split_forward(const Problem &pr, const Plan &pl, const void *Q, const void *K,
                        const void *V, void *O, float *G, float *ws, float *saved, hipStream_t st,
                        Tracer &tc)
{
    const SplitScratch sc = split_scratch(pl, pr.BH, pr.N, pr.dt, 0);
    float *gpart = ws + sc.g_off, *fraw = ws + sc.f_off;
    Problem p = pr;
    p.D = 128;
    Tracer quiet(nullptr, st);  // the caller's trace gets one mark per pass, not per kernel
    if (pr.causal && pl.nseg == 1) saved = nullptr;  // no segment starts from another's sums
    for (int j = 0; j < 2; ++j) {
        const void *Vj = col_block(V, j, pr.dt);
        void *Oj = col_block(O, j, pr.dt);
        for (int i = 0; i < 2; ++i) {
            p.a = i == 0 ? pr.a : 0.f;
            const la_status s = planes_forward(p, pl, 256, col_block(Q, i, pr.dt), col_block(K, i, pr.dt),
                                               Vj, Oj, i == 0 ? gpart : (j == 1 ? G : nullptr), ws,
                                               saved_block(saved, pl, 2 * i + j), st, quiet, i == 0 ? XF_RAW : XF_ACC,
                                               i == 0 ? nullptr : gpart, fraw);
            if (s != LA_OK) return s;
            tc.mark("fwd_block_pass");
        }
    }
    if (!saved) return LA_OK;
    k_leave_witness<<<dim3(pr.BH), dim3(64), 0, st>>>((const uint32_t *)O, (uint32_t *)saved_block(saved, pl, 4),
                                                      pr.N, row_words(pr.dt), problem_key(pr, pl));
    return launch_status();
}

// dK == nullptr: the ascending sweeps only (dQ).
la_status split_backward(const Problem &pr, const Plan &pl, const void *Q, const void *K,
                         const void *V, const void *O, const float *G, const void *dO, void *dQ,
                         void *dK, void *dV, float *ws, const float *saved, hipStream_t st, Tracer &tc)
{
    const SplitScratch sc = split_scratch(pl, pr.BH, pr.N, pr.dt, 1);
    Problem p = pr;
    p.D = 128;
    Tracer quiet(nullptr, st);  // the caller's trace gets one mark per pass, not per kernel
    if (pr.causal && pl.nseg == 1) saved = nullptr;
    int *handed = saved ? (int *)(ws + sc.flag_off) : nullptr;
    if (saved)
        k_check_witness<<<dim3(pr.BH), dim3(64), 0, st>>>(
            (const uint32_t *)O, (const uint32_t *)saved_block(saved, pl, 4), handed, pr.N, row_words(pr.dt),
            problem_key(pr, pl));
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            p.a = i == 0 ? pr.a : 0.f;
            BlockPass bp;
            // dQ_i and dK_i are complete after j = 1, dV_j after i = 1
            bp.xflags = (j == 1 ? 1 | 2 : 0) | (i == 1 ? 4 : 0);
            bp.Pq = ws + sc.q_off;
            bp.Pk = ws + sc.k_off;
            bp.Pv = ws + sc.v_off + (size_t)j * pr.BH * pr.N * 128;
            bp.handed = handed;
            const la_status s = planes_backward(
                p, pl, 256, col_block(Q, i, pr.dt), col_block(K, i, pr.dt), col_block(V, j, pr.dt),
                col_block(O, j, pr.dt), G, col_block(dO, j, pr.dt), col_block(dQ, i, pr.dt),
                dK ? col_block(dK, i, pr.dt) : nullptr, dK ? col_block(dV, j, pr.dt) : nullptr, ws,
                saved_block(saved, pl, 2 * i + j), st, quiet, bp);
            if (s != LA_OK) return s;
            tc.mark("bwd_block_pass");
        }
    return LA_OK;
}

}  // namespace la
