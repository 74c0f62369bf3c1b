// D = 256 on the D = 128 matrix-core kernels (la_split.hip), over blocks of 128 columns (split_forward,
// split_backward, split_prefill).
#include "la_blocks.h"

namespace la {

// Head size 256 on the D = 128 kernels.  With q = [q1 q2], k = [k1 k2] (halves of 128) the
// weight a + b q.k is (a + b q1.k1) + (0 + b q2.k2), and with v = [v1 v2] every sum of
// Sec. 3.1 / 3.2 splits into blocks: the numerator of output half j is the sum over i of
// the numerators of the D = 128 problems (q_i, k_i, v_j) with coefficients (a, b) for i = 1
// and (0, b) for i = 2, g is the sum of their denominators, and likewise
//   dq_i = sum_j dq(q_i, k_i, v_j; o_j, dO_j, g),   dk_i = sum_j dk(...),   dv_j = sum_i dv(...)
// where the blocks (o_j, dO_j) and the full g stand for the stored set of the block problem
// (delta = o . OmegaHat splits over j as well).  The four block problems run on the D = 128 kernels over column
// blocks of the 256-wide rows and build the outputs up in two launches each: all sums in one launch, all scans in
// one, then the two block problems that begin the output blocks and the two that add to them (run_forward,
// run_backward).  What two block problems of a launch read in common is then in the last-level cache, and half
// the segments fill the chip.  One block problem after another, 12 launches forward and 20 backward, took, a step,
// us, and take now: 64 slices of 4096 rows, fp32 3029 and 2790, bf16 1425 and 1200, without the mask 1925 and 1820,
// 1109 and 968; 100 of 400, fp32 631 and 441, bf16 345 and 212; one of 300, bf16 165 and 80.
// `pl` is the plan of the D = 128 problem; behind the slots the forward pass keeps the first share of g and, for
// bf16, the undivided numerators in fp32, and the backward pass, for bf16, the first share of every gradient block
// in fp32 (split_scratch).  la_forward_static, whose scratch may not hold four sets of slots, runs one block problem
// after another where it does not.  With `saved` the forward pass hands its sums at the segment boundaries to the
// backward pass, which then forms none.
//
// Whether a hand-over buffer holds this problem's sums is for the backward pass to find out: the buffer is
// optional, and a forward call that was given none (or one it could not use) succeeds all the same.  So the
// forward pass leaves the last row of every slice's O in it, under a key of the problem, and the backward pass
// compares that with the O it is given: sums of other inputs, or memory that no forward pass wrote, are passed
// over, slice by slice.  The sums kernel is launched either way and returns at once where the sums hold.
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

la_status split_prefill(const Problem &pr, const Plan &pl, const void *K, const void *V, float *ws,
                        float *state, int accumulate, hipStream_t st)
{
    Problem p = pr;
    p.D = 128;
    // fp32: one block after another, each in as many segments as fit the slots of all four, where the shared launch
    // leaves units idle for more rows than six more launches cost (65 to 85 slices, whose blocks are a round and a little
    // more; us, shared and one after another: 66 slices of 2000 rows 237 and 189, 76 of 3509 405 and 341, 84 of 6000 718
    // and 614).  The shared launch reads half of the rows out of the last-level cache: bf16 is faster in it everywhere
    // (76 of 3509 113 and 128), fp32 where that is all there is to gain (35 of 10000 401 and 413).
    Plan one = make_plan(1, pr.BH, pr.N, 128, pr.dt, 0, 0, true, kCoarse);
    one.together = false;
    const auto rows = [&](long problems, const Plan &x) {
        return (problems * pr.BH * x.nseg + 255) / 256 * min(x.seg_len, pr.N);
    };
    const bool shared = pr.dt != LA_F32 || one.nseg > 4 * pl.nseg || rows(4, pl) <= 5 * rows(1, one) ||
                        rows(4, pl) <= 4 * rows(1, one) + 600;
    la_status s = shared ? planes_totals(p, pl, 256, K, V, ws, st) : LA_OK;
    for (int b = 0; b < 4 && s == LA_OK; ++b) {
        if (!shared) s = planes_totals(p, one, 256, K, V, ws, st, b);
        const Plan &x = shared ? pl : one;
        if (s == LA_OK)
            s = state_block_from_totals(ws + (shared ? b * split_slots(pl, pr.BH) : 0), state, pr.BH, x.nseg, x.slot_floats,
                                        b / 2, b % 2, pr.N, accumulate, st);
    }
    return s;
}

// The witness, behind the hand-over buffers of the four block problems.
template <typename F>
static uint32_t *witness(F *saved, const Plan &pl)
{
    return (uint32_t *)(saved + 4 * (pl.saved_bytes / sizeof(float)));
}

la_status split_forward(const Problem &pr, const Plan &pl, const void *Q, const void *K,
                        const void *V, void *O, float *G, float *ws, float *saved, hipStream_t st,
                        Tracer &tc)
{
    const SplitScratch sc = split_scratch(pl, pr.BH, pr.N, pr.dt, 0);
    Problem p = pr;
    p.D = 128;
    if (pr.causal && pl.nseg == 1) saved = nullptr;  // no segment starts from another's sums
    BlockScratch bs;
    bs.together = sc.together;
    bs.g = ws + sc.g_off;
    bs.f = ws + sc.f_off;
    const la_status s = planes_forward(p, pl, 256, Q, K, V, O, G, ws, saved, st, tc, bs);
    if (s != LA_OK || !saved) return s;
    k_leave_witness<<<dim3(pr.BH), dim3(64), 0, st>>>((const uint32_t *)O, witness(saved, pl), pr.N, row_words(pr.dt),
                                                      problem_key(pr, pl));
    tc.mark("leave_witness");
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
    if (pr.causal && pl.nseg == 1) saved = nullptr;
    BlockScratch bs;
    bs.q = ws + sc.q_off;
    bs.k = ws + sc.k_off;
    bs.v = ws + sc.v_off;
    bs.delta = ws + sc.delta_off;
    if (saved) {
        int *handed = (int *)(ws + sc.flag_off);
        k_check_witness<<<dim3(pr.BH), dim3(64), 0, st>>>((const uint32_t *)O, witness((float *)saved, pl), handed,
                                                          pr.N, row_words(pr.dt), problem_key(pr, pl));
        tc.mark("check_witness");
        bs.handed = handed;
    }
    return planes_backward(p, pl, 256, Q, K, V, O, G, dO, dQ, dK, dV, ws, saved, st, tc, bs);
}

}  // namespace la
