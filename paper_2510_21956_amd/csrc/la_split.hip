// Matrix-core kernels for gfx950: the chunk algebra of the three phases (per-segment sums, scan,
// apply) with every contraction on the bf16 matrix pipe, on tiles of one to three bf16 planes
// (la_planes.h).
//   fp32 tensors take three planes everywhere, which is fp32 arithmetic;
//   bf16 tensors are tiles of one plane as they stand; intermediates (weight blocks, running
//     states, the 1/g scaling) take two planes in the first rows of a sequence and one beyond
//     (lo_rows_of);
//   bf16 tensors whose Q, K rows are normalised on the way stay one-plane tiles of the raw rows:
//     the factors 1/|q|, 1/|k| go to the weight blocks, to the outputs and to the wave's own
//     operand of the running sums' updates, which are fp32 in three planes here.
//
// Head size 16 runs on the kernels of D = 32 with columns 16 .. 31 zero (LD < D).  In bf16 it takes
// three planes for every intermediate, in all rows (W16): its matrix work is a few percent of a
// step, and the rounding of a single plane does not average out over 16 columns (dK without the
// mask: 2.8e-3 against 64 bits with one plane, 1.7e-3, the rounding of the output, with three).
//
// A workgroup handles one (slice, segment) in chunks of 32 rows.  Of its waves, one for every 16 columns
// of the D x D running state (wave w: [16w, 16w+16)) keeps them in its accumulators for the whole
// segment; the descending sweep (ks_bwd_dkv) and, up to D = 32, the ascending one (ks_bwd_dq_halves)
// have twice as many, one half for each of their two products with a state; bf16 at D = 128 descends
// with 32 columns a wave (ks_bwd_dkv_wide).  Output blocks are computed transposed (accumulator rows =
// output columns): a lane then holds four columns of a row, which an exchange between lanes turns into
// whole runs of a row (store_block).  The backward sweeps of fp32, which have no registers to spare,
// compute them the other way round, store single floats and need no exchange (SWAP).
//
// The descending sums weight row i by 1/g_i.  With split rows of Q (QT) the kernels stage
// q_i / g_i instead of q_i, and everything follows from that one tile:
//   R = sum (q/g) dO^T,   dK_n = b (sum_i Cm'_in (q_i/g_i) + ...),  Cm'_in = dO_i . v_n - dprime_i,
//   dV_n = sum_i (a/g_i + b (q_i/g_i) . k_n) dO_i + ...,   u = sum dprime (q/g),  w = sum dO / g,
// so no scaled copy of dO is kept next to dO itself.  With one-plane tiles, which must stay
// exact, the weight blocks carry the 1/g, and the wave's own 32 x 16 operand of R's update is
// scaled in registers.
//
// What bounds them (counters of the masked kernels): issue and traffic.  A wave issues one instruction every
// 5.3 clocks, two waves of a SIMD together one vector instruction every 2.9; with two waves a SIMD and a
// chunk's phases in turn between barriers, the matrix pipe, the vector ALU (splitting inputs and states)
// and LDS reads take 25 to 45 % of the clocks each in fp32, 14 to 38 % in bf16, where waits make up the
// rest (barriers, and memory with 40 KB in flight per CU); at D = 64 in fp32 and in bf16 the sweeps move their own
// traffic at 4.2 to 5.0 TB/s, where a copy reaches 5.0.  Four waves a SIMD in the descending sweep and wider
// columns for bf16 at D = 128 are what moved them.  Forward / ascending / descending sweep, us, on waves that
// hold both states of a sweep and now (one card, medians of five runs each; cards differ by up to 8 %):
//   fp32, D = 64, 64 slices of 4096 rows         72 / 95 / 117 -> 74 / 95 / 104
//   fp32, D = 128, 64 slices of 1000             51 / 64 / 80 -> 50 / 64 / 74
//   bf16, D = 64, 36 slices of 5003              28 / 34 / 39 -> 28 / 33 / 31
//   bf16, D = 128, 128 slices of 2048            66 / 89 / 112 -> 66 / 88 / 104
//   bf16, D = 128, 16 slices of 131072           498 / 683 / 918 -> 504 / 690 / 843
//   bf16 normalised, D = 128, 128 of 2048        106 / 153 / 196 -> 108 / 156 / 194
//   fp32, D = 16, one slice of 256 in one piece  12.6 / 14.6 / 17.5 -> 12.5 / 11.4 / 13.0
//   fp32 without the mask, D = 64, 64 of 16384   96 / 242 / 205 -> 96 / 232 / 205
#include "la_wave32.h"

namespace la {
namespace {

// fp32, fp32 normalised, bf16, bf16 normalised, bf16 with 32-bit intermediates throughout
enum { P32, N32, P16, N16, W16 };
// Planes of Q and K (LQ), of V and dO (LV), of intermediates (LX).
template <int MODE>
struct Mode {
    typedef typename std::conditional<MODE == P32 || MODE == N32, float, __bf16>::type TIO;
    static constexpr bool NORM = MODE == N32 || MODE == N16;
    static constexpr int LQ = sizeof(TIO) == 4 ? 3 : 1, LV = LQ, LX = MODE == P16 ? 2 : 3;
    static constexpr bool QT = sizeof(TIO) == 4, SWAP = QT;
    // bf16 rows are normalised through factors 1/|q|, 1/|k| on what is fp32 anyway (RN)
    static constexpr bool RN = MODE == N16;
    // Chunks requested ahead.  A CU keeps 5 TB/s / 256 busy with some 40 KB in flight; a chunk of
    // the four tensors of the descending sweep is 64 KB in fp32 but 32 KB in bf16 (D = 128).
    static constexpr int DEPTH = sizeof(TIO) == 2 ? 2 : 1;
};

// A wave's 16 entries of a vector sum (z, p, u, w) in the layout of its output blocks: one
// column a lane (SWAP), or the columns 4g .. 4g+3 of the lane group.
// LONG: summed with what the additions lose (a sum that only leaves the kernel).
template <bool SWAP, bool LONG = false>
struct Sum {
    typedef typename std::conditional<SWAP, float, f4v>::type T;
    T v;
    LongSum<T> run;
    __device__ __forceinline__ Sum()
    {
        v = T{};
        run = LongSum<T>{};
    }
    // where the lane's share is in an array of D
    static __device__ __forceinline__ int at(int w, int c, int g) { return w * 16 + (SWAP ? c : 4 * g); }
    __device__ __forceinline__ void load(const float *p, int w, int c, int g)
    {
        v = *reinterpret_cast<const T *>(p + at(w, c, g));
    }
    __device__ __forceinline__ void store(float *p, int w, int c, int g) const
    {
        T x = v;
        if constexpr (LONG) x = total(run);
        if constexpr (SWAP) {
            if (g == 0) p[w * 16 + c] = x;
        } else {
            if (c == 0) *reinterpret_cast<f4v *>(p + w * 16 + 4 * g) = x;
        }
    }
    // += sum over the chunk rows of f's columns, weighted by the factor planes in wgt
    template <int LF, int LW>
    __device__ __forceinline__ void add(const bf8v (&f)[LF], const bf8v (&wgt)[LW])
    {
        if constexpr (LONG) {
            f4v hi = {0.f, 0.f, 0.f, 0.f}, lo = hi;
            if constexpr (SWAP) {
                mma_planes<LW, LF>(hi, lo, wgt, f);
                run.add(hi[0], lo[0]);
            } else {
                mma_planes<LF, LW>(hi, lo, f, wgt);
                run.add(hi, lo);
            }
        } else if constexpr (SWAP) {
            v += step_product<LW, LF>(wgt, f)[0];
        } else {
            v += step_product<LF, LW>(f, wgt);
        }
    }
};
// Per-row factors of the chunk for output block m: the lane's four rows (SWAP) or its one row.
template <bool SWAP>
__device__ __forceinline__ auto row_factor(const float *x, int m, int c, int g)
{
    if constexpr (SWAP) return *reinterpret_cast<const f4v *>(x + m * 16 + 4 * g);
    else return x[m * 16 + c];
}
// own columns (x) of the weight block (p) or the other way round
template <bool SWAP, int LA, int LB>
__device__ __forceinline__ f4v own_product(const bf8v (&own)[LA], const bf8v (&p)[LB])
{
    if constexpr (SWAP) return step_product<LB, LA>(p, own);
    else return step_product<LA, LB>(own, p);
}
// One 16-row block of a gradient; LD > D builds it up over two launches (store_grad_block), of which the second
// (`add`) asks for the share of the first ahead (load_grad).
template <bool SWAP, int D, int LD, typename TIO>
__device__ __forceinline__ f4v load_grad(const TIO *out, const float *part, int w, int rows_valid, int l)
{
    if constexpr (SWAP) return load_cols_block(out, LD, w * 16, rows_valid, l % 16, l / 16);
    else return load_block(part, D, w * 16, rows_valid, l);
}
template <bool SWAP, int D, int LD, typename TIO>
__device__ __forceinline__ void store_grad(TIO *out, float *part, bool add, int w, int rows_valid, int l,
                                           f4v x, f4v old)
{
    if (LD < D && w * 16 >= LD) return;  // columns that are not there
    if constexpr (SWAP) {
        if (LD > D && add) {
            keep_branch();
            x += old;
        }
        store_cols_block(out, LD, w * 16, rows_valid, l % 16, l / 16, x);
    } else {
        store_grad_block<D, LD>(out, part, add, w * 16, rows_valid, l, x, old);
    }
}
// Backward of the row normalisation on the two output blocks; xhat = scale * the tile's rows.
template <bool SWAP, bool OP, int D, int LQ, typename LN>
__device__ __forceinline__ void project_chunk(f4v (&x)[2], const __bf16 *tile, const LN &ln,
                                              const float *scale, float *dots, const float *inv, int w,
                                              int c, int g)
{
    if constexpr (SWAP) {
        bf8v f[LQ];
        f4v xh[2];
        if constexpr (OP) load_cols_op<D, LQ>(f, tile, ln.local(ln.ocol), w);
        else load_cols<D, LQ>(f, tile, ln.local(ln.col), w);
        frag_values<LQ>(xh, f);
        if (scale) {
#pragma unroll
            for (int m = 0; m < 2; ++m) xh[m] *= *reinterpret_cast<const f4v *>(scale + m * 16 + 4 * g);
        }
        project_cols<D / 16>(x, xh, dots, inv, w, c, g);
    } else {
        float y[2][4], xh[2][4];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int r = m * 16 + c;
            quad_values<D, LQ>(xh[m], tile + (OP ? Tile<D>::op_quad(r, 4 * w + g) : Tile<D>::nat_quad(r, 4 * w + g)));
            const float sc = scale ? scale[r] : 1.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                xh[m][e] *= sc;
                y[m][e] = x[m][e];
            }
        }
        project_blocks<D / 16, CR, 2>(y, xh, dots, inv, w, c, g);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[m][e] = y[m][e];
    }
}
// The wave's own column fragment f (one plane) times the row factors in r1 and, if given, r2,
// split again.
template <int L>
__device__ __forceinline__ void scale_frag(bf8v (&o)[L], const bf8v (&f)[1], const float *r1, int g,
                                           const float *r2 = nullptr)
{
    f4v x[2];
    frag_values<1>(x, f);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        x[m] *= *reinterpret_cast<const f4v *>(r1 + 16 * m + 4 * g);
        if (r2) x[m] *= *reinterpret_cast<const f4v *>(r2 + 16 * m + 4 * g);
    }
    split_frag<L>(x[0], x[1], o);
}
// A per-row factor array (32 floats) as an operand: three planes.
__device__ __forceinline__ void factor_frag(bf8v (&o)[3], const float *r, int g)
{
    split_frag<3>(*reinterpret_cast<const f4v *>(r + 4 * g),
                  *reinterpret_cast<const f4v *>(r + 16 + 4 * g), o);
}

// The state a workgroup starts from: the sum of `n` slots, `step` floats from one to the next, in that order,
// as four rows of one column a lane (COLS; rows 16 rb + 4 g .., column 16 w + c of the D x D block p) or its
// transpose, and NV vectors (the lane's share at v[k], a float or four).  n = 1 reads a slot that
// launch_scan_slots has summed up.
template <int D, bool COLS, int NV, typename T>
__device__ __forceinline__ void add_slots(Blk (&st)[D / 16], const float *p, T (&sum)[NV],
                                          const float *const (&v)[NV], ptrdiff_t step, int n, int w, int c, int g)
{
    constexpr int NRB = D / 16, BATCH = 2;
    const float *q = COLS ? p + 4 * g * D + w * 16 + c : p + (w * 16 + c) * D + 4 * g;
    const auto read = [&](ptrdiff_t at, Blk (&x)[NRB], T (&y)[NV]) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            if constexpr (COLS) {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[rb].set(e, q[at + (rb * 16 + e) * D]);
            } else {
                x[rb].v = *reinterpret_cast<const f4v *>(q + at + rb * 16);
            }
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) y[k] = *reinterpret_cast<const T *>(v[k] + at);
    };
    if (n > 0) read(0, st, sum);
    if constexpr (D > 64) return;
    for (int i0 = 1; i0 < n; i0 += BATCH) {
        Blk x[BATCH][NRB];
        T y[BATCH][NV];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) read(min(i0 + i, n - 1) * step, x[i], y[i]);
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            if (i0 + i < n) {
#pragma unroll
                for (int rb = 0; rb < NRB; ++rb) st[rb].v += x[i][rb].v;
#pragma unroll
                for (int k = 0; k < NV; ++k) sum[k] += y[i][k];
            }
    }
}

// The waves that form weight blocks are the last to reach the barrier behind them: between the two calls
// their instructions go first.  Time of the forward / ascending / descending sweep with it: fp32, D = 64 (64 slices
// of 4096 rows) - 2 / - 0.5 / - 1 %; bf16 (36 of 5003) - 1 / - 1 / - 2 %; normalised - 3 / - 2 / - 2 %; D = 32, bf16 (64 of
// 4096), descending - 5 %.  At D = 128 it moves nothing (fp32, 64 of 1000 0 / + 0.5 / + 1 %; bf16, 128 of 2048 0 / 0 / 0).
template <int D>
__device__ __forceinline__ void go_first(bool on)
{
    if (D <= 64 && on) __builtin_amdgcn_s_setprio(2);
}
template <int D>
__device__ __forceinline__ void go_in_turn()
{
    if (D <= 64) __builtin_amdgcn_s_setprio(0);
}

// Of the ascending sweeps: 1/g and g of a chunk of `rows` rows, of which thread t < 32 holds row t's g.
__device__ __forceinline__ void post_ascending(float *rs, float *gb, __bf16 *fr, int t, int rows, float gn)
{
    if (t < CR) {
        const bool ok = t < rows;
        const float r = ok ? __builtin_amdgcn_rcpf(gn) : 0.f;
        rs[t] = r;
        gb[t] = ok ? gn : 0.f;
        store_factor<3>(fr, t, r);
    }
}
// Their weight blocks Cm' (rows n, columns i) on or below the diagonal, one a wave w of D / 16.
template <int MODE, int D, typename LN>
__device__ __forceinline__ void ascending_weights(__bf16 *Ct, const __bf16 *Vt, const __bf16 *dOt, const float *dl,
                                                  const float *ik, int w, bool lo_on, const LN &ln, int c, int g)
{
    typedef Mode<MODE> MD;
#pragma unroll 1
    for (int pidx = w; pidx < 3; pidx += D / 16) {
        const int ib = pidx ? 1 : 0, nb = pidx == 2 ? 1 : 0;
        const f4v pa = block_product<D, MD::LV, MD::LV>(Vt, nb, dOt, ib, ln);
        const float di = dl[ib * 16 + c];
        const int last = nb == ib ? c : 15;  // last row n at or before row i
        f4v x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = 4 * g + e > last ? 0.f : pa[e] - di;
        if constexpr (MD::RN) x *= *reinterpret_cast<const f4v *>(ik + nb * 16 + 4 * g);
        with_planes<MD::LX>(lo_on, [&](auto n) { store_weights<n.value>(Ct, ib * 16 + c, nb, g, x); });
    }
}
// Of the descending sweeps: thread t < 32 holds row t's g, thread 32 + r dprime of row r.  Returns the row's factor
// in w (1/g) or u (dprime, over g where the staged rows are not).
template <bool QT>
__device__ __forceinline__ float post_descending(float *rs, float *dl, int t, int rows, float gd)
{
    const int r = t % CR;
    float y = r < rows ? (t < CR ? __builtin_amdgcn_rcpf(gd) : gd) : 0.f;
    (t < CR ? rs : dl)[r] = y;
    if constexpr (!QT) {
        const float inv = __shfl(y, r);
        if (t >= CR) y *= inv;
    }
    return y;
}
// Weights of block (ib, nb) from its products x (rows i = 4 g + e, column n): of Cm' (cm) or W.
template <bool QT, bool RN>
__device__ __forceinline__ f4v descending_weight(f4v x, bool cm, int ib, int nb, const float *rs, const float *dl,
                                                 const float *iq, const float *kinv, float a, float b, int n, int g)
{
    const int row = ib * 16 + 4 * g;
    const f4v r4 = *reinterpret_cast<const f4v *>(rs + row);
    f4v iq4 = {1.f, 1.f, 1.f, 1.f};
    if constexpr (RN) iq4 = *reinterpret_cast<const f4v *>(iq + row);
    if (cm) {
        x -= *reinterpret_cast<const f4v *>(dl + row);
        if constexpr (!QT) x *= r4;
        if constexpr (RN) x *= iq4;
    } else {
        if constexpr (RN) x = (x * kinv[nb * 16 + n]) * iq4;
        if constexpr (QT) x = a * r4 + b * x;
        else x = (a + b * x) * r4;
    }
    const int first = nb == ib ? n : 0;  // first row i that sees column n
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = 4 * g + e < first ? 0.f : x[e];
    return x;
}

// Head size 256 (LD > D): the block problems of one launch, 1 << lg of them, block problem 2 i + j on columns 128 i
// .. of Q and K and 128 j .. of V.  Workgroups of the same rows follow one another, so that what they read in
// common comes out of the last-level cache.  Strides between the block problems' slots, hand-over buffers (or
// slots) and, between column blocks, of the fp32 shares and the token-heads.
struct Blocks {
    int lg = 0;
    unsigned ids = 0;
    size_t slots = 0, sinit = 0, part = 0, rows = 0;
};
struct Block {
    int id = 0, i = 0, j = 0;
};
template <bool ON>
__device__ __forceinline__ Block block_of(const Blocks &bl, int &wg)
{
    Block b;
    if constexpr (ON) {
        b.id = bl.ids >> 2 * (wg & ((1 << bl.lg) - 1)) & 3;
        b.i = b.id >> 1;
        b.j = b.id & 1;
        wg >>= bl.lg;
    }
    return b;
}

// One tensor's chunk into its tile: normalised (NORM, fp32) and times scale[row], if given, on
// the way.  1 / |row| goes to inv_out.
template <bool NORM, bool OP, int L, typename CH>
__device__ __forceinline__ void stage(const CH &ch, __bf16 *tile, float *inv_out = nullptr,
                                      const float *scale = nullptr, int t = threadIdx.x)
{
    f4v x[CH::NQ];
    ch.values(x);
    if constexpr (L == 1) {  // bf16 as it stands; NORM: 1 / |row| to inv_out
        if constexpr (NORM) normalise_quads<CH>(x, inv_out, t);
        ch.template store<OP, L>(tile, t);
    } else {
        if constexpr (NORM) normalise_quads<CH>(x, inv_out, t);
        if (scale) {
#pragma unroll
            for (int k = 0; k < CH::NQ; ++k) x[k] *= scale[CH::row(k, t)];
        }
        CH::template store_values<OP, L>(tile, x, t);
    }
}

// ---------------------------------------------------------------------------
// Phase 1: per-segment S = sum k v^T, z = sum k, p = sum v (Eq. xy without the factors), to
// slot `seg + slot_shift` as [S | z | p], or [S^T | z] (TRANSPOSED) for the backward pass.  LONG: z and p
// with what their additions lose (unmasked passes and prompt states; masked rows see them through
// plain running sums anyway).  STREAM: K and V by non-temporal loads (kv_state).
// ---------------------------------------------------------------------------
template <int MODE, int D, bool TRANSPOSED, int LD, bool LONG, bool STREAM>
__global__ __launch_bounds__(4 * D, 2) void ks_kv_state(
    const typename Mode<MODE>::TIO *__restrict__ K, const typename Mode<MODE>::TIO *__restrict__ V,
    float *__restrict__ ws, int N, int nseg, int nseg_run, SegMap sm, size_t slot_floats, int slot_shift,
    const int *__restrict__ skip, Blocks bl)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int LQ = MD::LQ, LV = MD::LV, NRB = D / 16, PL = Tile<D>::PLANE;
    constexpr int NT = MD::DEPTH, TP = (LQ + LV) * PL;  // tile pairs staged at a time, elements of one
    typedef Chunk<TIO, D, LD> CH;
    __shared__ __align__(16) __bf16 lds[NT * TP];
    __shared__ __align__(16) float ikb[MD::RN ? NT * CR : 4];  // 1 / |k|
    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    const int bh = wg / nseg_run, seg = wg % nseg_run;
    if constexpr (LD > D) {  // slices whose sums were handed over
        if (skip && skip[bh]) return;
        K += D * at.i;
        V += D * at.j;
        ws += at.id * bl.slots;
    }
    const TIO *Kp = K + (size_t)bh * N * LD, *Vp = V + (size_t)bh * N * LD;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const Lanes<D, (D == 64 && LV == 3)> ln(c, g);
    const bf8v one[1] = {ones_frag()};

    Blk st[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) st[rb].zero();
    LongSum<f4v> zacc{}, pacc{};  // z, p [16w + 4g + e]
    const f4v zero = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](LongSum<f4v> &x, f4v hi, f4v lo) __attribute__((always_inline)) {
        if constexpr (LONG) x.add(hi, lo);
        else x.s += hi + lo;
    };
    struct Set {
        CH k, v;
    } sets[NT];
    const long c_last = row0 + (row1 - row0 - 1) / CR * CR;
    auto request = [&](long c0, int i) __attribute__((always_inline)) {
        sets[i].k.template load<STREAM>(Kp, min(c0 + i * CR, c_last), N);
        sets[i].v.template load<STREAM>(Vp, min(c0 + i * CR, c_last), N);
    };
    auto put = [&](int i) __attribute__((always_inline)) {
        __bf16 *Kt = lds + i * TP, *Vt = Kt + LQ * PL;
        stage<MD::NORM, false, LQ>(sets[i].k, Kt, MD::RN ? ikb + i * CR : nullptr);
        sets[i].v.template store<false, LV>(Vt);
        if (__builtin_expect(sets[i].v.top() > kLargestBf16, 0)) sets[i].v.template store_any<false>(Vt);
    };
    // One tile pair into the sums.  In bf16, z and p take their products in when the update of S has
    // run; fp32 has no registers to keep them that long (128 at D = 64, four workgroups a CU).
    constexpr bool DEFER = LV == 1;
    auto one_tile = [&](int i) __attribute__((always_inline)) {
        const __bf16 *Kt = lds + i * TP, *Vt = Kt + LQ * PL;
        const float *ik = ikb + (MD::RN ? i * CR : 0);
        f4v zh = zero, zl = zero, ph = zero, pl = zero;
        bf8v kf[LQ];
        load_cols<D, LQ>(kf, Kt, ln.local(ln.col), w);
        if constexpr (MD::RN) {
            bf8v fk[3];
            factor_frag(fk, ik, g);
            mma_planes<LQ, 3>(zh, zl, kf, fk);
        } else {
            mma_planes<LQ, 1>(zh, zl, kf, one);
        }
        if constexpr (!DEFER) add(zacc, zh, zl);
        if constexpr (TRANSPOSED) {
            if constexpr (MD::RN) {
                bf8v kh[3];
                scale_frag<3>(kh, kf, ik, g);
                rank_update<D, LV, 3>(st, Vt, kh, ln);
            } else {
                rank_update<D, LV, LQ>(st, Vt, kf, ln);
            }
        } else {
            bf8v vf[LV];
            load_cols<D, LV>(vf, Vt, ln.local(ln.col), w);
            mma_planes<LV, 1>(ph, pl, vf, one);
            if constexpr (!DEFER) add(pacc, ph, pl);
            if constexpr (MD::RN) {
                bf8v vh[3];
                scale_frag<3>(vh, vf, ik, g);
                rank_update<D, LQ, 3>(st, Kt, vh, ln);
            } else {
                rank_update<D, LQ, LV>(st, Kt, vf, ln);
            }
            if constexpr (DEFER) add(pacc, ph, pl);
        }
        if constexpr (DEFER) add(zacc, zh, zl);
    };
#pragma unroll
    for (int i = 0; i < NT; ++i) request(row0, i);
    for (long c0 = row0; c0 < row1; c0 += NT * CR) {
        const bool two = NT == 2 && c0 + CR < row1;
        block_sync();
        put(0);
        if (NT == 2) request(c0 + NT * CR, 0);
        if (two) put(NT - 1);
        block_sync();
        request(c0 + NT * CR, NT - 1);
        if (LQ * LV == 1 && !MD::RN && two) {
            const __bf16 *K0 = lds, *V0 = K0 + LQ * PL, *K1 = lds + (NT - 1) * TP, *V1 = K1 + LQ * PL;
            bf8v k0[1], k1[1], v0[1], v1[1];
            load_cols<D, 1>(k0, K0, ln.local(ln.col), w);
            load_cols<D, 1>(k1, K1, ln.local(ln.col), w);
            const f4v zh = mfma(k1[0], one[0], mfma(k0[0], one[0], zero));
            if constexpr (TRANSPOSED) {
                rank_update_two<D>(st, V0, V1, k0[0], k1[0], ln);
            } else {
                load_cols<D, 1>(v0, V0, ln.local(ln.col), w);
                load_cols<D, 1>(v1, V1, ln.local(ln.col), w);
                const f4v ph = mfma(v1[0], one[0], mfma(v0[0], one[0], zero));
                rank_update_two<D>(st, K0, K1, v0[0], v1[0], ln);
                add(pacc, ph, zero);
            }
            add(zacc, zh, zero);
        } else {
            one_tile(0);
            if (two) one_tile(NT - 1);
        }
    }
    float *slot = ws + ((size_t)bh * nseg + seg + slot_shift) * slot_floats;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) slot[(rb * 16 + 4 * g + i) * D + w * 16 + c] = st[rb].get(i);
    if (c == 0) {
        *reinterpret_cast<f4v *>(slot + D * D + w * 16 + 4 * g) = total(zacc);
        if constexpr (!TRANSPOSED) *reinterpret_cast<f4v *>(slot + D * D + D + w * 16 + 4 * g) = total(pacc);
    }
}

// ---------------------------------------------------------------------------
// Phase 3 (forward, masked): Eq. fglast / div chunk by chunk.
//   f = tril(a + b Q_c K_c^T) V_c + a 1 p^T + b Q_c S ;  g = rowsum(tril) + a n + b Q_c z
//   then S += K_c^T V_c, z += sum k, p += sum v
// LD > D: the call works on D columns of rows LD wide and is one of several launches that
// build O up: the first leaves the numerator undivided in O and its share of g in G; the second (ADD) adds
// the numerator that O holds and the share of g in Gin first.  bf16 tensors keep the undivided numerator
// in Fraw instead (fp32, B*H*N rows of D): O is rounded once.
// ---------------------------------------------------------------------------
template <int MODE, int D, int LD, bool ADD>
__global__ __launch_bounds__(4 * D, 2) void ks_fwd_apply(
    const typename Mode<MODE>::TIO *__restrict__ Q, const typename Mode<MODE>::TIO *__restrict__ K,
    const typename Mode<MODE>::TIO *__restrict__ V, typename Mode<MODE>::TIO *__restrict__ O,
    float *__restrict__ G, const float *__restrict__ ws, float *__restrict__ saved, int N, int nseg,
    SegMap sm, size_t slot_floats, int fold, size_t saved_floats, float a, float b,
    const float *__restrict__ Gin, float *__restrict__ Fraw, Blocks bl)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int LQ = MD::LQ, LV = MD::LV, LX = MD::LX;
    constexpr bool RAW32 = LD > D && sizeof(TIO) == 2;
    constexpr int NW = D / 16, NRB = D / 16, PL = Tile<D>::PLANE, WPL = Tile<32>::PLANE;
    typedef Chunk<TIO, D, LD> CH;
    __shared__ __align__(16) __bf16 lds[(2 * LQ + LV) * PL + LX * WPL];
    __shared__ __align__(16) float zs[D], qzs[CR], psum[2][CR], ginv[NW][CR];
    __shared__ __align__(16) float iq[MD::RN ? CR : 4], ik[MD::RN ? CR : 4];  // 1 / |q|, 1 / |k|
    __bf16 *Qt = lds;  // operand-ordered; K and V natural
    __bf16 *Kt = Qt + LQ * PL, *Vt = Kt + LQ * PL, *Pt = Vt + LV * PL;

    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    if constexpr (LD > D) {
        Q += D * at.i;
        K += D * at.i;
        V += D * at.j;
        O += D * at.j;
        ws += at.id * bl.slots;
        if (saved) saved += at.id * bl.sinit;
        if (at.i) a = 0.f;
        if (at.j) G = nullptr;  // both blocks have the same
        Fraw += at.j * bl.part;
    }
    const int bh = wg / nseg, seg = wg % nseg;
    const size_t base = (size_t)bh * N * LD;
    const TIO *Qp = Q + base, *Kp = K + base, *Vp = V + base;
    TIO *Op = O + base;
    float *Gp = G + (size_t)bh * N;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const Lanes<D> ln(c, g);
    const Lanes<32> lw(c, g);
    const bf8v one[1] = {ones_frag()};

    // initial state: S[r][j], j = 16w + c
    const int nsum = fold ? seg : min(seg, 1);
    const float *slot = ws + ((size_t)bh * nseg + seg - max(nsum - 1, 0)) * slot_floats;
    Blk st[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) st[rb].zero();
    f4v vec[2] = {};  // p, z [16w + 4g + e]
    const float *const vp[2] = {slot + D * D + D + w * 16 + 4 * g, slot + D * D + w * 16 + 4 * g};
    add_slots<D, true>(st, slot, vec, vp, slot_floats, nsum, w, c, g);
    f4v pacc = vec[0], zacc = vec[1];
    if (c == 0) *reinterpret_cast<f4v *>(zs + w * 16 + 4 * g) = zacc;
    // the block above the diagonal stays zero
    if (t < 64) store_weights<LX>(Pt, c, 1, g, f4v{0.f, 0.f, 0.f, 0.f});

    struct Set {
        CH q, k, v;
    } sets[MD::DEPTH];
    const long c_last = row0 + (row1 - row0 - 1) / CR * CR;
#pragma unroll
    for (int i = 0; i < MD::DEPTH; ++i) {
        const long ci = min(row0 + i * CR, c_last);
        sets[i].q.load(Qp, ci, N);
        sets[i].k.load(Kp, ci, N);
        sets[i].v.load(Vp, ci, N);
    }
    auto chunk = [&](long c0, Set &cur) __attribute__((always_inline)) {
        const bool lo_on = c0 < sm.lo_rows;  // second plane of the intermediates: early rows
        block_sync();  // every wave is done with the previous chunk's tiles; zs is written
        {
            f4v x[2] = {cur.q.value(0), cur.q.value(1)};
            if constexpr (MD::NORM) normalise_quads<CH>(x, MD::RN ? iq : nullptr);
            float s[2];
#pragma unroll
            for (int k = 0; k < 2; ++k)
                s[k] = dot4(x[k], *reinterpret_cast<const f4v *>(zs + 4 * CH::quad(k)));
            CH::row_totals(s);
            if (CH::leader()) {
#pragma unroll
                for (int k = 0; k < 2; ++k) qzs[CH::row(k)] = s[k];
            }
            if constexpr (LQ == 1) cur.q.template store<true, 1>(Qt);
            else CH::template store_values<true, LQ>(Qt, x);
        }
        stage<MD::NORM, false, LQ>(cur.k, Kt, MD::RN ? ik : nullptr);
        cur.v.template store<false, LV>(Vt);
        if (__builtin_expect(cur.v.top() > kLargestBf16, 0)) cur.v.template store_any<false>(Vt);
        block_sync();
        const long cn = min(c0 + MD::DEPTH * CR, c_last);
        f4v old[2] = {};  // numerators that the launch before left
        if constexpr (ADD) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int nrows = (int)(row1 - c0) - m * 16;
                if constexpr (RAW32) old[m] = load_block(Fraw + ((size_t)bh * N + c0 + m * 16) * D, D, w * 16, nrows, l);
                else old[m] = load_block(Op + (size_t)(c0 + m * 16) * LD, LD, w * 16, nrows, l);
            }
        }
        cur.q.load(Qp, cn, N);

        go_first<D>(w < 3);
        // ---- phase A: weight blocks P = tril(a + b Q K^T), rows n, columns i ----
#pragma unroll 1
        for (int pidx = w; pidx < 3; pidx += NW) {
            const int ib = pidx ? 1 : 0, nb = pidx == 2 ? 1 : 0;
            f4v pa = block_product<D, LQ, LQ>(Kt, nb, Qt, ib, ln);
            if constexpr (MD::RN)  // one factor after the other: their product may overflow
                pa = (pa * iq[ib * 16 + c]) * *reinterpret_cast<const f4v *>(ik + nb * 16 + 4 * g);
            const int last = nb == ib ? c : 15;  // last row n at or before row i
            f4v x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = 4 * g + e > last ? 0.f : a + b * pa[e];
            with_planes<LX>(lo_on, [&](auto n) { store_weights<n.value>(Pt, ib * 16 + c, nb, g, x); });
            const float rs = reduce_lane_groups((x[0] + x[1]) + (x[2] + x[3]));
            if (g == 0) psum[nb][ib * 16 + c] = rs;
        }
        cur.k.load(Kp, cn, N);
        // The product with the state needs nothing of phase A.
        f4v fh[2], fl[2];  // rows j = 16w + 4g + e, columns i
#pragma unroll
        for (int m = 0; m < 2; ++m) fh[m] = fl[m] = f4v{0.f, 0.f, 0.f, 0.f};
        with_planes<LX>(lo_on, [&](auto n) { state_product<D, n.value, LQ, false>(fh, fl, st, Qt, ln); });
        bf8v vf[LV];
        load_cols<D, LV>(vf, Vt, ln.local(ln.col), w);
        cur.v.load(Vp, cn, N);
        block_sync();

        go_in_turn<D>();
        // ---- phase B: denominators; V^T P^T on top, divide, store ----
        if (l < CR) {
            const float ps = psum[0][l] + (l >= 16 ? psum[1][l] : 0.f);
            float gv = b * qzs[l] + a * (float)c0 + ps;
            const bool valid = l < (int)(row1 - c0);
            if constexpr (ADD) {
                if (valid) gv += (Gin + (size_t)bh * N + c0)[l];
            }
            ginv[w][l] = LD > D && !ADD ? 1.f : 1.f / gv;
            if (w == 0 && G && valid) (Gp + c0)[l] = gv;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            f4v f = (MD::RN ? b * iq[m * 16 + c] : b) * (fh[m] + fl[m]);
            with_planes<LX>(lo_on, [&](auto n) {
                bf8v pf[n.value];
                load_rows<32, n.value>(pf, Pt, lw.row, m, 0);
                f += step_product<LV, n.value>(vf, pf);
            });
            const f4v y = (f + a * pacc) * ginv[w][m * 16 + c];
            if (LD < D && w * 16 >= LD) break;  // columns that are not there
            const int nrows = (int)(row1 - c0) - m * 16;
            float *fr = RAW32 ? Fraw + ((size_t)bh * N + c0 + m * 16) * D : nullptr;
            if (RAW32 && !ADD)
                store_block<float>(fr, D, w * 16, nrows, l, y[0], y[1], y[2], y[3]);
            else
                store_block<TIO>(Op + (size_t)(c0 + m * 16) * LD, LD, w * 16, nrows, l, y[0], y[1], y[2],
                                 y[3], ADD, old[m], &ginv[w][m * 16]);
        }
        pacc += step_product<LV, 1>(vf, one);
        bf8v kf[LQ];
        load_cols<D, LQ>(kf, Kt, ln.local(ln.col), w);
        if constexpr (MD::RN) {
            bf8v fk[3], vh[3];
            factor_frag(fk, ik, g);
            zacc += step_product<LQ, 3>(kf, fk);
            scale_frag<3>(vh, vf, ik, g);
            rank_update<D, LQ, 3>(st, Kt, vh, ln);
        } else {
            zacc += step_product<LQ, 1>(kf, one);
            rank_update<D, LQ, LV>(st, Kt, vf, ln);
        }
        // zs was read while this chunk was staged; it is read again behind the barrier at
        // the top of the next one
        if (c == 0) *reinterpret_cast<f4v *>(zs + w * 16 + 4 * g) = zacc;
    };
    for (long c0 = row0; c0 < row1; c0 += MD::DEPTH * CR) {
        chunk(c0, sets[0]);
        if (MD::DEPTH == 2 && c0 + CR < row1) chunk(c0 + CR, sets[MD::DEPTH - 1]);
    }
    // hand-over to the backward pass: entry s = [S^T | z] over all rows before segment s
    if (saved && seg + 1 < nseg) {
        float *dst = saved + ((size_t)bh * nseg + seg + 1) * saved_floats;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
            *reinterpret_cast<f4v *>(dst + (w * 16 + c) * D + rb * 16 + 4 * g) = st[rb].v;
        if (c == 0) *reinterpret_cast<f4v *>(dst + D * D + w * 16 + 4 * g) = zacc;
    }
}

// ---------------------------------------------------------------------------
// Phase 3 (forward, unmasked): every row reads the same sums, f = a p + b Q S, g = a N + b Q z.
// The rows are cut as fills the chip best, rows_wg a workgroup, whatever the segments were; the
// state is split into planes once.  Bound by memory and by what a workgroup needs before its first
// row (the 4 D^2 bytes of the state, out of L2).  bf16 stages 64 rows between its two barriers.
// LD > D, ADD, Gin and Fraw as above.
// ---------------------------------------------------------------------------
template <int MODE, int D, int LD, bool ADD>
__global__ __launch_bounds__(4 * D, 2) void ks_fwd_read(
    const typename Mode<MODE>::TIO *__restrict__ Q, typename Mode<MODE>::TIO *__restrict__ O,
    float *__restrict__ G, const float *__restrict__ ws, float *__restrict__ saved, int N, int nseg,
    int nwg, int rows_wg, int lo_rows, size_t slot_floats, size_t saved_floats, float a, float b,
    const float *__restrict__ Gin, float *__restrict__ Fraw, Blocks bl)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int LQ = MD::LQ, LX = MD::LX, NT = MD::DEPTH;
    constexpr bool RAW32 = LD > D && sizeof(TIO) == 2;
    constexpr int NW = D / 16, NRB = D / 16, PL = Tile<D>::PLANE;
    typedef Chunk<TIO, D, LD> CH;
    __shared__ __align__(16) __bf16 lds[NT * LQ * PL];  // operand-ordered tiles of Q
    __shared__ __align__(16) float zs[D], qzs[NT * CR], ginv[NW][NT * CR], iqb[MD::RN ? NT * CR : 4];

    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    if constexpr (LD > D) {
        Q += D * at.i;
        O += D * at.j;
        ws += at.id * bl.slots;
        if (saved) saved += at.id * bl.sinit;
        if (at.i) a = 0.f;
        if (at.j) G = nullptr;  // both blocks have the same
        Fraw += at.j * bl.part;
    }
    const int bh = wg / nwg, part = wg % nwg;
    const size_t base = (size_t)bh * N * LD;
    const TIO *Qp = Q + base;
    TIO *Op = O + base;
    float *Gp = G + (size_t)bh * N;
    const long row0 = (long)part * rows_wg, row1 = min(row0 + rows_wg, (long)N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const Lanes<D> ln(c, g);

    CH sets[NT];
    const long c_last = row0 + (row1 - row0 - 1) / CR * CR;
#pragma unroll
    for (int i = 0; i < NT; ++i) sets[i].load(Qp, min(row0 + i * CR, c_last), N);

    const float *slot = ws + (size_t)bh * nseg * slot_floats;
    Blk st[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) st[rb].set(i, slot[(rb * 16 + 4 * g + i) * D + w * 16 + c]);
    const f4v pacc = *reinterpret_cast<const f4v *>(slot + D * D + D + w * 16 + 4 * g);
    const f4v zacc = *reinterpret_cast<const f4v *>(slot + D * D + w * 16 + 4 * g);
    if (c == 0) *reinterpret_cast<f4v *>(zs + w * 16 + 4 * g) = zacc;
    // hand-over to the backward pass: entry 0 = [S^T | z] over the whole sequence
    if (saved && part == 0) {
        float *dst = saved + (size_t)bh * nseg * saved_floats;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
            *reinterpret_cast<f4v *>(dst + (w * 16 + c) * D + rb * 16 + 4 * g) = st[rb].v;
        if (c == 0) *reinterpret_cast<f4v *>(dst + D * D + w * 16 + 4 * g) = zacc;
    }
    bf8v sp[D / 32][LX];
#pragma unroll
    for (int kt = 0; kt < D / 32; ++kt) split_frag<LX>(st[2 * kt].v, st[2 * kt + 1].v, sp[kt]);

    auto put = [&](int i) __attribute__((always_inline)) {
        f4v x[2] = {sets[i].value(0), sets[i].value(1)};
        if constexpr (MD::NORM) normalise_quads<CH>(x, MD::RN ? iqb + i * CR : nullptr);
        float s[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) s[k] = dot4(x[k], *reinterpret_cast<const f4v *>(zs + 4 * CH::quad(k)));
        CH::row_totals(s);
        if (CH::leader()) {
#pragma unroll
            for (int k = 0; k < 2; ++k) qzs[i * CR + CH::row(k)] = s[k];
        }
        if constexpr (LQ == 1) sets[i].template store<true, 1>(lds + i * PL);
        else CH::template store_values<true, LQ>(lds, x);
    };
    f4v old[NT][2] = {};  // numerators that the launch before left
    const auto request_old = [&](long c0) __attribute__((always_inline)) {
        if constexpr (!ADD) return;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const long r = c0 + i * CR + m * 16;
                if constexpr (ADD && RAW32) old[i][m] = load_block(Fraw + ((size_t)bh * N + r) * D, D, w * 16, (int)(row1 - r), l);
                else if constexpr (ADD) old[i][m] = load_block(Op + (size_t)r * LD, LD, w * 16, (int)(row1 - r), l);
            }
    };
    auto rows = [&](long c0, int i) __attribute__((always_inline)) {
        f4v fh[2], fl[2];  // rows j = 16w + 4g + e, columns i
#pragma unroll
        for (int m = 0; m < 2; ++m) fh[m] = fl[m] = f4v{0.f, 0.f, 0.f, 0.f};
        with_planes<LX>(c0 < lo_rows, [&](auto n) {
            fixed_product<D, n.value, LX, LQ>(fh, fl, sp, lds + i * LQ * PL, ln);
        });
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int r = i * CR + m * 16;
            const f4v f = (MD::RN ? b * iqb[r + c] : b) * (fh[m] + fl[m]);
            const f4v y = (f + a * pacc) * ginv[w][r + c];
            if (LD < D && w * 16 >= LD) break;  // columns that are not there
            const int nrows = (int)(row1 - c0) - m * 16;
            float *fr = RAW32 ? Fraw + ((size_t)bh * N + c0 + m * 16) * D : nullptr;
            if (RAW32 && !ADD)
                store_block<float>(fr, D, w * 16, nrows, l, y[0], y[1], y[2], y[3]);
            else
                store_block<TIO>(Op + (size_t)(c0 + m * 16) * LD, LD, w * 16, nrows, l, y[0], y[1], y[2],
                                 y[3], ADD, old[i][m], &ginv[w][r]);
        }
    };
    for (long c0 = row0; c0 < row1; c0 += NT * CR) {
        const bool two = NT == 2 && c0 + CR < row1;
        block_sync();  // zs is written; every wave is done with the tiles, qzs and the factors
        put(0);
        request_old(c0);  // ahead of the next rows: loads are waited for in order
        if (NT == 2) sets[0].load(Qp, min(c0 + 2 * CR, c_last), N);
        if (two) put(NT - 1);
        block_sync();
        sets[NT - 1].load(Qp, min(c0 + (2 * NT - 1) * CR, c_last), N);
        if (l < (two ? 2 * CR : CR)) {
            float gv = b * qzs[l] + a * (float)N;
            const bool valid = l < (int)(row1 - c0);
            if constexpr (ADD) {
                if (valid) gv += (Gin + (size_t)bh * N + c0)[l];
            }
            ginv[w][l] = LD > D && !ADD ? 1.f : 1.f / gv;
            if (w == 0 && G && valid) (Gp + c0)[l] = gv;
        }
        __builtin_amdgcn_wave_barrier();
        rows(c0, 0);
        if (two) rows(c0 + CR, NT - 1);
    }
}

// ---------------------------------------------------------------------------
// Backward, ascending sweep: dQ (Eq. back1), dprime, and the segment's reverse sums.
//   Cm'_in = dO_i . v_n - dprime_i,  dprime_i = o_i . dO_i
//   dQ_c = diag(b / g) (tril(Cm') K_c + dO_c S^T - dprime z^T);  then S += K_c^T V_c, z += sum k
//   R += (Q/g)_c^T dO_c,  u += sum dprime (q/g),  w += sum dO / g
// The state is held transposed (rows j, columns r): the product contracts over j.
// LD > D: ADD marks the second of the two launches that build dQ up; handed as in BlockScratch.
// fp32 at D = 128 holds S^T, R and two chunks in 234 to 256 registers; normalised, with the mask, one more
// goes to scratch (a state in its accumulators less would cost a pass over Q and dO).
// ---------------------------------------------------------------------------
template <int MODE, int D, bool CAUSAL, int LD, bool ADD>
__global__ __launch_bounds__(4 * D, 2) void ks_bwd_dq(
    const typename Mode<MODE>::TIO *__restrict__ Q, const typename Mode<MODE>::TIO *__restrict__ K,
    const typename Mode<MODE>::TIO *__restrict__ V, const typename Mode<MODE>::TIO *__restrict__ O,
    const float *__restrict__ G, const typename Mode<MODE>::TIO *__restrict__ dO,
    typename Mode<MODE>::TIO *__restrict__ dQ, float *ws, const float *sinit, size_t sinit_floats,
    float *__restrict__ dprime, int N, int nseg, SegMap sm, size_t slot_floats, int fold, float b,
    float *__restrict__ Pq, const int *__restrict__ handed, Blocks bl)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int LQ = MD::LQ, LV = MD::LV, LX = MD::LX;
    constexpr bool SWAP = MD::SWAP, QT = MD::QT, PROJ = MD::NORM, F32 = sizeof(TIO) == 4;
    constexpr int NW = D / 16, NRB = D / 16, PL = Tile<D>::PLANE, WPL = Tile<32>::PLANE;
    constexpr int TS = CAUSAL ? 1 : 0;
    typedef Chunk<TIO, D, LD> CH;
    typedef BwdSlot<D> SL;
    __shared__ __align__(16) __bf16 lds[LV * PL + LQ * PL + TS * (LV * PL + LQ * PL + LX * WPL)];
    __shared__ __align__(16) __bf16 frs[2][3 * CR], fdl[3 * CR];  // 1/g, dprime as operands
    __shared__ __align__(16) float rsb[2][CR], gb[2][CR], dl[CR];
    __shared__ __align__(16) float qinv[PROJ ? CR : 4], dots[PROJ ? NW * CR : 4];  // 1 / |q|
    __shared__ __align__(16) float ik[MD::RN ? CR : 4];                            // 1 / |k|
    __bf16 *dOt = lds;  // operand-ordered; the others natural
    __bf16 *Qt = dOt + LV * PL, *Vt = Qt + LQ * PL, *Kt = Vt + TS * LV * PL, *Ct = Kt + TS * LQ * PL;

    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    if constexpr (LD > D) {
        Q += D * at.i;
        K += D * at.i;
        dQ += D * at.i;
        V += D * at.j;
        O += D * at.j;
        dO += D * at.j;
        ws += at.id * bl.slots;
        sinit += at.id * bl.sinit;
        dprime += at.j * bl.rows;
        Pq += at.i * bl.part;
    }
    const int bh = wg / nseg, seg = wg % nseg;
    const size_t base = (size_t)bh * N * LD;
    const TIO *Qp = Q + base, *Kp = K + base, *Vp = V + base, *Op = O + base, *dOp = dO + base;
    TIO *dQp = dQ + base;
    const float *Gp = G + (size_t)bh * N;
    float *dp = dprime + (size_t)bh * N;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const Lanes<D, (D >= 128)> ln(c, g);
    const Lanes<32> lw(c, g);
    const bf8v one[1] = {ones_frag()};
    const bool need_R = CAUSAL ? (seg > 0) : true;  // segment 0's sums start no one
    const bool need_Q = need_R || PROJ;

    const bool zero_init = CAUSAL && seg == 0;
    const float *slot = sinit + ((size_t)bh * nseg + (CAUSAL ? seg : 0)) * sinit_floats;
    if constexpr (LD > D) {
        if (handed && !handed[bh]) slot = ws + ((size_t)bh * nseg + (CAUSAL ? seg : 0)) * slot_floats;
    }
    Blk st[NRB], accR[NRB];  // S^T: rows j, columns r = 16w + c;  R: rows r, columns j
#pragma unroll
    for (int jb = 0; jb < NRB; ++jb) {
        accR[jb].zero();
        st[jb].zero();
    }
    Sum<SWAP> zacc, uacc;      // z, u
    Sum<SWAP, !CAUSAL && QT> wacc;  // w: without the mask, most of dV (fp32: bf16 rounds it anyway)
    if (!zero_init) {
        const int nsum = CAUSAL && fold ? seg : 1;
        slot -= (nsum - 1) * sinit_floats;
        typename Sum<SWAP>::T x[1] = {};
        const float *const vp[1] = {slot + SL::Z + Sum<SWAP>::at(w, c, g)};
        add_slots<D, true>(st, slot + SL::ST, x, vp, sinit_floats, nsum, w, c, g);
        zacc.v = x[0];
    }
    if constexpr (CAUSAL) {
        if (t < 64) store_weights<LX>(Ct, c, 1, g, f4v{0.f, 0.f, 0.f, 0.f});
    }

    struct Set {
        CH d, o, k, v, q;
        float g;  // g of row t % 32
    } sets[MD::DEPTH];
    const long c_last = row0 + (row1 - row0 - 1) / CR * CR;
    // 1/g of the chunk starting at c0, whose g is gn, into buffer `par`
    auto post_factors = [&](long c0, float gn, int par) {
        post_ascending(rsb[par], gb[par], frs[par], t, (int)(row1 - c0), gn);
    };
#pragma unroll
    for (int i = 0; i < MD::DEPTH; ++i) {
        const long ci = min(row0 + i * CR, c_last);
        sets[i].g = load_row_float(Gp, ci, N, t % CR);
        sets[i].d.load(dOp, ci, N);
        sets[i].o.load(Op, ci, N);
        if constexpr (CAUSAL) {
            sets[i].v.load(Vp, ci, N);
            sets[i].k.load(Kp, ci, N);
        }
        sets[i].q.load(Qp, ci, N);
    }
    post_factors(row0, sets[0].g, 0);
    // nxt: the set that holds the chunk after this one
    auto chunk = [&](long c0, Set &cur, Set &nxt, int par) __attribute__((always_inline)) {
        block_sync();
        const float *rs = rsb[par];
        const bool lo_on = c0 < sm.lo_rows;  // second plane of the intermediates: early rows
        if (need_Q) stage<MD::NORM, false, LQ>(cur.q, Qt, PROJ ? qinv : nullptr, QT ? rs : nullptr);
        {
            float s[2] = {dot4(cur.d.value(0), cur.o.value(0)), dot4(cur.d.value(1), cur.o.value(1))};
            CH::row_totals(s);
            if (CH::leader()) {
#pragma unroll
                for (int k = 0; k < CH::NLD; ++k) {
                    const int r = CH::row(k);
                    dl[r] = s[k];
                    // the row's weight in u: the staged rows are q/g (QT), or q (times 1/|q|;
                    // this lane wrote that factor)
                    float wu = QT ? s[k] : s[k] * rs[r];
                    if constexpr (MD::RN) wu *= qinv[r];
                    store_factor<3>(fdl, r, wu);
                    if (r < (int)(row1 - c0) && at.i == 0) (dp + c0)[r] = s[k];
                }
            }
            cur.d.template store<true, LV>(dOt);
        }
        if constexpr (CAUSAL) {
            cur.v.template store<false, LV>(Vt);
            stage<MD::NORM, false, LQ>(cur.k, Kt, MD::RN ? ik : nullptr);
        }
        if (__builtin_expect(max(cur.d.top(), CAUSAL ? cur.v.top() : 0.f) > kLargestBf16, 0)) {
            cur.d.template store_any<true>(dOt);
            if constexpr (CAUSAL) cur.v.template store_any<false>(Vt);
        }
        block_sync();
        const long cn = min(c0 + MD::DEPTH * CR, c_last);
        f4v old[2] = {};  // shares that the launch before left
        if constexpr (ADD) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
                old[m] = load_grad<SWAP, D, LD>(dQp + (size_t)(c0 + m * 16) * LD, Pq + ((size_t)bh * N + c0 + m * 16) * D,
                                                w, (int)(row1 - c0) - m * 16, l);
        }
        // Under a branch the load stays here; as a plain load the compiler moves it into post_factors, behind this
        // chunk's stores, where the first wave waits for both.  Time of the sweep under a branch: fp32 without the
        // mask - 3 % (D = 64, 64 x 16384) and - 8 % (D = 32, 64 x 8192), bf16 with it - 1.5 % (D = 64, 36 x 5003); bf16
        // without, which requests two chunks ahead, + 3 % (64 x 16384); fp32 with it, where the load stays put
        // either way, no less, and at D = 128 normalised a register goes to scratch.
        if (F32 == CAUSAL || w == 0) cur.g = load_row_float(Gp, cn, N, t % CR);
        cur.d.load(dOp, cn, N);
        cur.o.load(Op, cn, N);
        if constexpr (!CAUSAL) cur.q.load(Qp, cn, N);

        if constexpr (CAUSAL) go_first<D>(w < 3);
        // ---- phase A: weight blocks Cm' (rows n, columns i) ----
        if constexpr (CAUSAL) {
            ascending_weights<MODE, D>(Ct, Vt, dOt, dl, ik, w, lo_on, ln, c, g);
            cur.v.load(Vp, cn, N);
        }
        f4v fh[2], fl[2];  // rows i, columns r (SWAP), or rows r, columns i
#pragma unroll
        for (int m = 0; m < 2; ++m) fh[m] = fl[m] = f4v{0.f, 0.f, 0.f, 0.f};
        with_planes<LX>(lo_on, [&](auto n) { state_product<D, n.value, LV, SWAP>(fh, fl, st, dOt, ln); });
        bf8v kf[LQ];
        if constexpr (CAUSAL) {
            load_cols<D, LQ>(kf, Kt, ln.local(ln.col), w);
            cur.k.load(Kp, cn, N);
            block_sync();
        }

        if constexpr (CAUSAL) go_in_turn<D>();
        // ---- phase B: K^T Cm'^T on top, scale, store ----
        f4v x[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            f4v f = fh[m] + fl[m];
            if constexpr (CAUSAL) {
                with_planes<LX>(lo_on, [&](auto n) {
                    bf8v pf[n.value];
                    load_rows<32, n.value>(pf, Ct, lw.row, m, 0);
                    f += own_product<SWAP, LQ, n.value>(kf, pf);
                });
            }
            x[m] = (b * row_factor<SWAP>(rs, m, c, g)) * (f - zacc.v * row_factor<SWAP>(dl, m, c, g));
        }
        if constexpr (PROJ)  // qhat = g (q/g), or q / |q|
            project_chunk<SWAP, false, D, LQ>(x, Qt, ln, QT ? gb[par] : qinv, dots, qinv, w, c, g);
#pragma unroll
        for (int m = 0; m < 2; ++m)
            store_grad<SWAP, D, LD>(dQp + (size_t)(c0 + m * 16) * LD,
                                    Pq + ((size_t)bh * N + c0 + m * 16) * D, ADD, w,
                                    (int)(row1 - c0) - m * 16, l, x[m], old[m]);
        if constexpr (CAUSAL) {
            cur.q.load(Qp, cn, N);
            if constexpr (MD::RN) {
                bf8v fk[3], kh[3];
                factor_frag(fk, ik, g);
                zacc.add(kf, fk);
                scale_frag<3>(kh, kf, ik, g);
                rank_update<D, LV, 3>(st, Vt, kh, ln);
            } else {
                zacc.add(kf, one);
                rank_update<D, LV, LQ>(st, Vt, kf, ln);
            }
        }
        if (need_R) {
            bf8v df[LV], qf[LQ], fr[3], fd[3];
            load_cols_op<D, LV>(df, dOt, ln.local(ln.ocol), w);
            load_cols<D, LQ>(qf, Qt, ln.local(ln.col), w);
            load_factor<3>(fr, frs[par], g);
            load_factor<3>(fd, fdl, g);
            wacc.add(df, fr);
            uacc.add(qf, fd);
            if constexpr (QT) {
                rank_update<D, LQ, LV>(accR, Qt, df, ln);
            } else {
                with_planes<LX>(lo_on, [&](auto n) {
                    bf8v oh[n.value];
                    scale_frag<n.value>(oh, df, rs, g, MD::RN ? qinv : nullptr);
                    rank_update<D, LQ, n.value>(accR, Qt, oh, ln);
                });
            }
        }
        post_factors(min(c0 + CR, row1), nxt.g, par ^ 1);
    };
    if constexpr (MD::DEPTH == 2) {
        for (long c0 = row0; c0 < row1; c0 += 2 * CR) {
            chunk(c0, sets[0], sets[MD::DEPTH - 1], 0);
            if (c0 + CR < row1) chunk(c0 + CR, sets[MD::DEPTH - 1], sets[0], 1);
        }
    } else {
        int par = 0;
        for (long c0 = row0; c0 < row1; c0 += CR, par ^= 1) chunk(c0, sets[0], sets[0], par);
    }
    if (need_R) {
        float *out = ws + ((size_t)bh * nseg + seg - (CAUSAL ? 1 : 0)) * slot_floats;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) out[SL::R + (rb * 16 + 4 * g + i) * D + w * 16 + c] = accR[rb].get(i);
        wacc.store(out + SL::W, w, c, g);
        uacc.store(out + SL::U, w, c, g);
    }
}

// ---------------------------------------------------------------------------
// Backward, ascending sweep, masked: dQ (Eq. back1), dprime, and the segment's reverse sums.
//   Cm'_in = dO_i . v_n - dprime_i,  dprime_i = o_i . dO_i
//   dQ_c = diag(b / g) (tril(Cm') K_c + dO_c S^T - dprime z^T);  then S += K_c^T V_c, z += sum k
//   R += (Q/g)_c^T dO_c,  u += sum dprime (q/g),  w += sum dO / g
// Half the waves make dQ and hold the state transposed (rows j, columns r: the product contracts over j);
// the others form the weight blocks and hold R.  Only at D = 32 (and 16), where a chunk's latencies are
// most of its time: one slice of 256 rows, D = 16, 14.6 -> 11.4 us.  Beyond, waves that hold both states are
// as fast or faster: fp32, 64 slices of 4096 rows, D = 64 88 us against 92 in halves; bf16, 36 of 5003 33.2
// against 35.2, 128 of 2048, D = 128 86 against 94.
// ---------------------------------------------------------------------------
template <int MODE, int D, int LD>
__global__ __launch_bounds__(8 * D, 4) void ks_bwd_dq_halves(
    const typename Mode<MODE>::TIO *__restrict__ Q, const typename Mode<MODE>::TIO *__restrict__ K,
    const typename Mode<MODE>::TIO *__restrict__ V, const typename Mode<MODE>::TIO *__restrict__ O,
    const float *__restrict__ G, const typename Mode<MODE>::TIO *__restrict__ dO,
    typename Mode<MODE>::TIO *__restrict__ dQ, float *ws, const float *sinit, size_t sinit_floats,
    float *__restrict__ dprime, int N, int nseg, SegMap sm, size_t slot_floats, int fold, float b,
    float *__restrict__ Pq, const int *, Blocks)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int L = MD::LQ, LX = MD::LX;
    constexpr bool SWAP = MD::SWAP, QT = MD::QT, PROJ = MD::NORM, F32 = sizeof(TIO) == 4;
    static_assert(D == 32 && LD <= D, "the larger head sizes have a kernel of their own");
    constexpr bool TIGHT = PROJ;
    constexpr int DEPTH = MD::DEPTH;
    constexpr int NW = D / 16, NRB = D / 16, PL = Tile<D>::PLANE, WPL = Tile<32>::PLANE;
    typedef Chunk<TIO, D, LD, true> CH;
    typedef BwdSlot<D> SL;
    __shared__ __align__(16) __bf16 lds[4 * L * PL + LX * WPL];
    __shared__ __align__(16) __bf16 frs[2][3 * CR], fdl[3 * CR];  // 1/g, dprime as operands
    __shared__ __align__(16) float rsb[2][CR], gb[2][CR], dl[CR];
    __shared__ __align__(16) float qinv[PROJ ? CR : 4], dots[PROJ ? NW * CR : 4];  // 1 / |q|
    __shared__ __align__(16) float ik[MD::RN ? CR : 4];                            // 1 / |k|
    __bf16 *dOt = lds;  // operand-ordered; the others natural
    __bf16 *Qt = dOt + L * PL, *Vt = Qt + L * PL, *Kt = Vt + L * PL, *Ct = Kt + L * PL;

    const int bh = blockIdx.x / nseg, seg = blockIdx.x % nseg;
    const size_t base = (size_t)bh * N * LD;
    const TIO *Qp = Q + base, *Kp = K + base, *Vp = V + base, *Op = O + base, *dOp = dO + base;
    TIO *dQp = dQ + base;
    const float *Gp = G + (size_t)bh * N;
    float *dp = dprime + (size_t)bh * N;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int wv = __builtin_amdgcn_readfirstlane(t / 64);
    const int half = wv / NW, w = wv % NW;  // half 0: dQ; half 1: R; columns 16 w ..
    const Lanes<D, TIGHT> ln(c, g);
    const bf8v one[1] = {ones_frag()};
    const bool need_R = seg > 0;  // segment 0's sums start no one
    const bool need_Q = need_R || PROJ;

    const float *slot = sinit + ((size_t)bh * nseg + seg) * sinit_floats;
    Blk st[NRB];  // half 0: S^T, rows j, columns r = 16w + c;  half 1: R, rows r, columns j
    Sum<SWAP> vec, vec2;  // z; u, w
#pragma unroll
    for (int jb = 0; jb < NRB; ++jb) st[jb].zero();
    if (seg > 0 && half == 0) {
        const int nsum = fold ? seg : 1;
        slot -= (nsum - 1) * sinit_floats;
        typename Sum<SWAP>::T x[1] = {};
        const float *const vp[1] = {slot + SL::Z + Sum<SWAP>::at(w, c, g)};
        add_slots<D, true>(st, slot + SL::ST, x, vp, sinit_floats, nsum, w, c, g);
        vec.v = x[0];
    }
    if (t < 64) store_weights<LX>(Ct, c, 1, g, f4v{0.f, 0.f, 0.f, 0.f});

    // fp32: all five tensors in every thread (dO, O, Q, V, K); bf16: dO, O and Q in half 0, V and K in
    // half 1
    struct Set {
        CH x[F32 ? 5 : 3];
        float g;  // g of row t % 32 (first wave)
    } sets[DEPTH];
    const long c_last = row0 + (row1 - row0 - 1) / CR * CR;
    auto request = [&](Set &s, long c0, bool first, bool second) __attribute__((always_inline)) {
        const int th = ln.local(t);
        if (first) {
            if (F32 || half == 0) {
                s.x[0].load(dOp, c0, N, th);
                s.x[1].load(Op, c0, N, th);
            } else {
                s.x[0].load(Vp, c0, N, th);
                s.x[1].load(Kp, c0, N, th);
            }
        }
        if (second) {
            if (need_Q && (F32 || half == 0)) s.x[2].load(Qp, c0, N, th);
            if constexpr (F32) {
                s.x[3].load(Vp, c0, N, th);
                s.x[4].load(Kp, c0, N, th);
            }
            if (wv == 0) s.g = load_row_float(Gp, c0, N, th % CR);
        }
    };
    // 1/g of the chunk starting at c0, whose g is gn, into buffer `par`
    auto post_factors = [&](long c0, float gn, int par) {
        post_ascending(rsb[par], gb[par], frs[par], ln.local(t), (int)(row1 - c0), gn);
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) request(sets[i], min(row0 + i * CR, c_last), true, true);
    post_factors(row0, sets[0].g, 0);
    // nxt: the set that holds the chunk after this one
    auto chunk = [&](long c0, Set &cur, Set &nxt, int par) __attribute__((always_inline)) {
        block_sync();
        const int th = ln.local(t), l = th % 64, c = l % 16, g = l / 16;
        const Lanes<32> lw(c, g);
        const float *rs = rsb[par];
        const bool lo_on = c0 < sm.lo_rows;  // second plane of the intermediates: early rows
        if (F32 || half == 0) {
            if (need_Q) stage<MD::NORM, false, L>(cur.x[2], Qt, PROJ ? qinv : nullptr, QT ? rs : nullptr, th);
            f4v d[CH::NQ], o[CH::NQ];
            cur.x[0].values(d);
            cur.x[1].values(o);
            float s[CH::NQ];
#pragma unroll
            for (int k = 0; k < CH::NQ; ++k) s[k] = dot4(d[k], o[k]);
            CH::row_totals(s);
            if (CH::leader(th)) {
                const int r = CH::row(0, th);
                dl[r] = s[0];
                // the row's weight in u: the staged rows are q/g (QT), or q (times 1/|q|;
                // this lane wrote that factor)
                float wu = QT ? s[0] : s[0] * rs[r];
                if constexpr (MD::RN) wu *= qinv[r];
                store_factor<3>(fdl, r, wu);
                if (r < (int)(row1 - c0)) (dp + c0)[r] = s[0];
            }
            cur.x[0].template store<true, L>(dOt, th);
        }
        if (F32 || half == 1) {
            constexpr int I = F32 ? 3 : 0;
            cur.x[I].template store<false, L>(Vt, th);
            stage<MD::NORM, false, L>(cur.x[I + 1], Kt, MD::RN ? ik : nullptr, nullptr, th);
            if constexpr (F32) {
                if (__builtin_expect(max(cur.x[0].top(), cur.x[I].top()) > kLargestBf16, 0)) {
                    cur.x[0].template store_any<true>(dOt, th);
                    cur.x[I].template store_any<false>(Vt, th);
                }
            }
        }
        block_sync();
        const long cn = min(c0 + DEPTH * CR, c_last);
        request(cur, cn, true, false);

        if (half) {
            // ---- phase A: weight blocks Cm' (rows n, columns i) ----
            ascending_weights<MODE, D>(Ct, Vt, dOt, dl, ik, w, lo_on, ln, c, g);
            block_sync();
            bf8v df[L];
            if (need_R) {
                load_cols_op<D, L>(df, dOt, ln.local(ln.ocol), w);
                {
                    bf8v fr[3];
                    load_factor<3>(fr, frs[par], g);
                    vec2.add(df, fr);
                }
                __builtin_amdgcn_sched_barrier(0);
                bf8v qf[L], fd[3];
                load_cols<D, L>(qf, Qt, ln.local(ln.col), w);
                load_factor<3>(fd, fdl, g);
                vec.add(qf, fd);
                __builtin_amdgcn_sched_barrier(0);
            }
            request(cur, cn, false, true);
            if (need_R) {
                if constexpr (QT) {
                    rank_steps<D, L, L>(st, Qt, df, ln);
                } else {
                    with_planes<LX>(lo_on, [&](auto n) {
                        bf8v oh[n.value];
                        scale_frag<n.value>(oh, df, rs, g, MD::RN ? qinv : nullptr);
                        rank_steps<D, L, n.value>(st, Qt, oh, ln);
                    });
                }
            }
            if constexpr (PROJ) block_sync();  // the one inside project_chunk
        } else {
            f4v fh[2], fl[2];  // rows i, columns r (SWAP), or rows r, columns i
#pragma unroll
            for (int m = 0; m < 2; ++m) fh[m] = fl[m] = f4v{0.f, 0.f, 0.f, 0.f};
            with_planes<LX>(lo_on, [&](auto n) { state_steps<D, n.value, L, SWAP>(fh, fl, st, dOt, ln); });
            bf8v kf[L];
            load_cols<D, L>(kf, Kt, ln.local(ln.col), w);
            block_sync();

            // ---- phase B: K^T Cm'^T on top, scale, store ----
            f4v x[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                f4v f = fh[m] + fl[m];
                with_planes<LX>(lo_on, [&](auto n) {
                    bf8v pf[n.value];
                    load_rows<32, n.value>(pf, Ct, lw.row, m, 0);
                    f += own_product<SWAP, L, n.value>(kf, pf);
                });
                x[m] = (b * row_factor<SWAP>(rs, m, c, g)) * (f - vec.v * row_factor<SWAP>(dl, m, c, g));
            }
            if constexpr (PROJ)  // qhat = g (q/g), or q / |q|
                project_chunk<SWAP, false, D, L>(x, Qt, ln, QT ? gb[par] : qinv, dots, qinv, w, c, g);
#pragma unroll
            for (int m = 0; m < 2; ++m)
                store_grad<SWAP, D, LD>(dQp + (size_t)(c0 + m * 16) * LD,
                                        Pq + ((size_t)bh * N + c0 + m * 16) * D, false, w,
                                        (int)(row1 - c0) - m * 16, l, x[m], f4v{});
            request(cur, cn, false, true);
            if constexpr (MD::RN) {
                bf8v fk[3], kh[3];
                factor_frag(fk, ik, g);
                vec.add(kf, fk);
                scale_frag<3>(kh, kf, ik, g);
                rank_steps<D, L, 3>(st, Vt, kh, ln);
            } else {
                vec.add(kf, one);
                rank_steps<D, L, L>(st, Vt, kf, ln);
            }
            post_factors(min(c0 + CR, row1), nxt.g, par ^ 1);
        }
    };
    if constexpr (DEPTH == 2) {
        for (long c0 = row0; c0 < row1; c0 += 2 * CR) {
            chunk(c0, sets[0], sets[DEPTH - 1], 0);
            if (c0 + CR < row1) chunk(c0 + CR, sets[DEPTH - 1], sets[0], 1);
        }
    } else {
        int par = 0;
        for (long c0 = row0; c0 < row1; c0 += CR, par ^= 1) chunk(c0, sets[0], sets[0], par);
    }
    if (need_R && half) {
        float *out = ws + ((size_t)bh * nseg + seg - 1) * slot_floats;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) out[SL::R + (rb * 16 + 4 * g + i) * D + w * 16 + c] = st[rb].get(i);
        vec2.store(out + SL::W, w, c, g);
        vec.store(out + SL::U, w, c, g);
    }
}

// ---------------------------------------------------------------------------
// Backward, descending sweep, masked: dK and dV (Eq. back1 / back2).
//   dK_c = b (tril(Cm')^T (Q/g)_c + V_c R^T - 1 u^T),   Cm'_in = dO_i . v_n - dprime_i
//   dV_c = tril(W)^T dO_c + a 1 w^T + b K_c R,          W_in = a / g_i + b (q_i/g_i) . k_n
//   then R += (Q/g)_c^T dO_c, u += sum dprime (q/g), w += sum dO / g.
// R is held twice.  2 D/16 waves: half make dK and hold R^T (rows j, columns r) and u, the others make dV
// and hold R (rows r, columns j) and w; both run the same code on exchanged tiles, 16 columns a wave.
// Four waves a SIMD instead of two that hold both states: more of what the waves issue and wait for in turn
// overlaps (fp32, D = 64: vector ALU 30 -> 38 %, LDS 38 -> 46 %, matrix pipe 31 -> 38 % of the clocks; times at the
// top).  Half the registers a wave have to do (TIGHT).
// LD > D: ADD marks the second of the two launches that build them up.
// ---------------------------------------------------------------------------
template <int MODE, int D, int LD, bool ADD>
__global__ __launch_bounds__(8 * D, 4) void ks_bwd_dkv(
    const typename Mode<MODE>::TIO *__restrict__ Q, const typename Mode<MODE>::TIO *__restrict__ K,
    const typename Mode<MODE>::TIO *__restrict__ V, const float *__restrict__ G,
    const typename Mode<MODE>::TIO *__restrict__ dO, typename Mode<MODE>::TIO *__restrict__ dK,
    typename Mode<MODE>::TIO *__restrict__ dV, const float *__restrict__ ws, const float *__restrict__ dprime, int N,
    int nseg, SegMap sm, size_t slot_floats, int fold, float a, float b, float *__restrict__ Pk, float *__restrict__ Pv,
    Blocks bl)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int L = MD::LQ, LX = MD::LX;  // planes of a tile, of intermediates
    constexpr bool SWAP = MD::SWAP, QT = MD::QT, PROJ = MD::NORM, F32 = sizeof(TIO) == 4;
    constexpr bool TIGHT = D == 128 || (D == 64 && PROJ);  // registers are short
    constexpr int DEPTH = D == 128 ? 1 : MD::DEPTH;
    constexpr int NW = D / 16, NRB = D / 16, PL = Tile<D>::PLANE, WPL = Tile<32>::PLANE;
    typedef Chunk<TIO, D, LD, true> CH;
    typedef BwdSlot<D> SL;
    __shared__ __align__(16) __bf16 lds[4 * L * PL + 2 * LX * WPL];
    __shared__ __align__(16) __bf16 frs[2][3 * CR], fdl[2][3 * CR];  // 1/g, dprime as operands
    __shared__ __align__(16) float rsb[2][CR], dlb[2][CR];
    __shared__ __align__(16) float kinv[PROJ ? CR : 4], dots[PROJ ? NW * CR : 4];  // 1 / |k|
    __shared__ __align__(16) float iq[MD::RN ? CR : 4];                            // 1 / |q|
    __bf16 *Kt = lds, *Vt = Kt + L * PL;  // operand-ordered; Q/g and dO natural
    __bf16 *Qt = Vt + L * PL, *dOt = Qt + L * PL, *Ct = dOt + L * PL, *Wt = Ct + LX * WPL;

    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    if constexpr (LD > D) {
        Q += D * at.i;
        K += D * at.i;
        dK += D * at.i;
        V += D * at.j;
        dO += D * at.j;
        dV += D * at.j;
        ws += at.id * bl.slots;
        dprime += at.j * bl.rows;
        if (at.i) a = 0.f;
        Pk += at.i * bl.part;
        Pv += at.j * bl.part;
    }
    const int bh = wg / nseg, seg = wg % nseg;
    const size_t base = (size_t)bh * N * LD;
    const TIO *Qp = Q + base, *Kp = K + base, *Vp = V + base, *dOp = dO + base;
    const float *Gp = G + (size_t)bh * N, *dp = dprime + (size_t)bh * N;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int wv = __builtin_amdgcn_readfirstlane(t / 64);
    const int half = wv / NW, w = wv % NW;  // half 0: dK; half 1: dV; columns 16 w ..
    const Lanes<D, TIGHT> ln(c, g);

    // the half's tiles: of the state product, of the own columns, of the update; its weights
    const __bf16 *Yt = half ? Kt : Vt, *Et = half ? dOt : Qt, *At = half ? Qt : dOt,
                 *Xt = half ? Wt : Ct;
    Blk st[NRB];
    Sum<SWAP> vec;  // u or w
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) st[rb].zero();
    if (seg < nseg - 1) {
        const int nsum = fold ? nseg - 1 - seg : 1;
        const ptrdiff_t step = -(ptrdiff_t)slot_floats;
        const float *slot = ws + ((size_t)bh * nseg + seg + nsum - 1) * slot_floats;
        typename Sum<SWAP>::T x[1] = {};
        const float *const vp[1] = {slot + (half ? SL::W : SL::U) + Sum<SWAP>::at(w, c, g)};
        if (half) add_slots<D, true>(st, slot + SL::R, x, vp, step, nsum, w, c, g);
        else add_slots<D, false>(st, slot + SL::R, x, vp, step, nsum, w, c, g);
        vec.v = x[0];
    }
    if (t < 64) {
        store_weights<LX>(Ct, 16 + c, 0, g, f4v{0.f, 0.f, 0.f, 0.f});
        store_weights<LX>(Wt, 16 + c, 0, g, f4v{0.f, 0.f, 0.f, 0.f});
    }

    const long nchunks = (row1 - row0 + CR - 1) / CR;
    // fp32: all four tensors in every thread; bf16: K and Q in half 0, V and dO in half 1
    struct Set {
        CH x[F32 ? 4 : 2];
        float gd;  // first wave: g of row l (l < 32), dprime of row l - 32
    } sets[DEPTH];
    // in two parts: registers are short while the state product runs
    auto request = [&](Set &s, long c0, bool first, bool second) __attribute__((always_inline)) {
        const int th = ln.local(t);
        if (first) {
            if constexpr (F32) {
                s.x[0].load(Kp, c0, N, th);
                s.x[1].load(Vp, c0, N, th);
            } else {
                s.x[0].load(half ? Vp : Kp, c0, N, th);
            }
        }
        if (second) {
            if constexpr (F32) {
                s.x[2].load(Qp, c0, N, th);
                s.x[3].load(dOp, c0, N, th);
            } else {
                s.x[1].load(half ? dOp : Qp, c0, N, th);
            }
            if (wv == 0) s.gd = (th < CR ? Gp : dp)[min((unsigned)c0 + th % CR, (unsigned)N - 1)];
        }
    };
    // 1/g and dprime of the chunk starting at c0 into buffer `par`
    auto post_factors = [&](long c0, const Set &x, int par) {
        if (wv != 0) return;
        const int th = ln.local(t), r = th % CR;
        const float y = post_descending<QT>(rsb[par], dlb[par], th, (int)(row1 - c0), x.gd);
        store_factor<3>((th < CR ? frs : fdl)[par], r, y);
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) request(sets[i], row0 + max(nchunks - 1 - i, 0L) * CR, true, true);
    post_factors(row0 + (nchunks - 1) * CR, sets[0], 0);
    // nxt: the set that holds the chunk after this one
    auto chunk = [&](long ci, Set &cur, Set &nxt, int par) __attribute__((always_inline)) {
        const long c0 = row0 + ci * CR;
        const float *rs = rsb[par], *dl = dlb[par];
        const bool lo_on = c0 < sm.lo_rows;  // second plane of the intermediates: early rows
        block_sync();
        const int th = ln.local(t), l = th % 64, c = l % 16, g = l / 16;
        const Lanes<32> lw(c, g);
        if constexpr (F32) {
            stage<MD::NORM, true, L>(cur.x[0], Kt, PROJ ? kinv : nullptr, nullptr, th);
            cur.x[1].template store<true, L>(Vt, th);
            stage<MD::NORM, false, L>(cur.x[2], Qt, nullptr, rs, th);
            cur.x[3].template store<false, L>(dOt, th);
            if (__builtin_expect(max(cur.x[1].top(), cur.x[3].top()) > kLargestBf16, 0)) {
                cur.x[1].template store_any<true>(Vt, th);
                cur.x[3].template store_any<false>(dOt, th);
            }
        } else {
            if (MD::RN && half == 0) {
                f4v x[2];
                cur.x[0].values(x);
                normalise_quads<CH>(x, kinv, th);
                cur.x[1].values(x);
                normalise_quads<CH>(x, iq, th);
                // the weights in u take the factor this lane just wrote
                const int r = CH::row(0, th);
                if (CH::leader(th)) store_factor<3>(fdl[par], r, dl[r] * rs[r] * iq[r]);
            }
            if constexpr (L == 1) {
                cur.x[0].template store_raw<true>(half ? Vt : Kt, th);
                cur.x[1].template store_raw<false>(half ? dOt : Qt, th);
            }
        }
        block_sync();
        const long cn = row0 + max(ci - DEPTH, 0L) * CR;
        const auto out = [&] { return (half ? dV : dK) + base + (size_t)c0 * LD; };
        const auto part = [&] { return (half ? Pv : Pk) + ((size_t)bh * N + c0) * D; };
        f4v old[2] = {};  // shares that the launch before left
        if constexpr (ADD) {
            {
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    old[m] = load_grad<SWAP, D, LD>(out() + (size_t)(m * 16) * LD, part() + m * 16 * D, w,
                                                    (int)(row1 - c0) - m * 16, l);
            }
        }
        request(cur, cn, true, false);

        go_first<D>(wv < 6);
        // ---- phase A: weight blocks Cm' and W (rows i, columns n) ----
#pragma unroll 1
        for (int pidx = wv; pidx < 6; pidx += 2 * NW) {
            const int q = pidx >= 3 ? pidx - 3 : pidx, ib = q ? 1 : 0, nb = q == 2 ? 1 : 0;
            const bool cm = pidx < 3;
            f4v x = block_product<D, L, L>(cm ? dOt : Qt, ib, cm ? Vt : Kt, nb, ln);
            x = descending_weight<QT, MD::RN>(x, cm, ib, nb, rs, dl, iq, kinv, a, b, c, g);
            with_planes<LX>(lo_on, [&](auto n) { store_weights<n.value>(cm ? Ct : Wt, nb * 16 + c, ib, g, x); });
        }
        f4v fh[2], fl[2];  // rows n, the wave's columns (SWAP), or the other way round
#pragma unroll
        for (int m = 0; m < 2; ++m) fh[m] = fl[m] = f4v{0.f, 0.f, 0.f, 0.f};
        with_planes<LX>(lo_on, [&](auto n) { state_steps<D, n.value, L, SWAP>(fh, fl, st, Yt, ln); });
        bf8v own[L];
        load_cols<D, L>(own, Et, ln.local(ln.col), w);
        request(cur, cn, false, true);
        block_sync();

        go_in_turn<D>();
        // ---- phase B ----
        f4v x[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            f4v f = fh[m] + fl[m], y = {0.f, 0.f, 0.f, 0.f};
            with_planes<LX>(lo_on, [&](auto n) {
                bf8v pf[n.value];
                load_rows<32, n.value>(pf, Xt, lw.row, m, 0);
                y = own_product<SWAP, L, n.value>(own, pf);
            });
            if (half) x[m] = (a * vec.v + (MD::RN ? b * kinv[m * 16 + c] : b) * f) + y;
            else x[m] = b * ((f + y) - vec.v);
        }
        if constexpr (PROJ) {
            if (half)
                block_sync();  // the one inside project_chunk
            else
                project_chunk<SWAP, true, D, L>(x, Kt, ln, QT ? nullptr : kinv, dots, kinv, w, c, g);
        }
#pragma unroll
        for (int m = 0; m < 2; ++m)
            store_grad<SWAP, D, LD>(out() + (size_t)(m * 16) * LD, part() + m * 16 * D, ADD, w,
                                    (int)(row1 - c0) - m * 16, l, x[m], old[m]);
        bf8v fac[3];
        load_factor<3>(fac, half ? frs[par] : fdl[par], g);
        vec.add(own, fac);
        if constexpr (QT) {
            rank_steps<D, L, L>(st, At, own, ln);
        } else {
            with_planes<LX>(lo_on, [&](auto n) {
                bf8v og[n.value];
                scale_frag<n.value>(og, own, rs, g, MD::RN ? iq : nullptr);
                rank_steps<D, L, n.value>(st, At, og, ln);
            });
        }
        post_factors(row0 + max(ci - 1, 0L) * CR, nxt, par ^ 1);
    };
    if constexpr (DEPTH == 2) {
        for (long ci = nchunks - 1; ci >= 0; ci -= 2) {
            chunk(ci, sets[0], sets[DEPTH - 1], 0);
            if (ci > 0) chunk(ci - 1, sets[DEPTH - 1], sets[0], 1);
        }
    } else {
        int par = 0;
        for (long ci = nchunks - 1; ci >= 0; --ci, par ^= 1) chunk(ci, sets[0], sets[0], par);
    }
}

// ---------------------------------------------------------------------------
// The same for bf16 at D = 128: waves of 32 columns (la_wave32.h), half of them for dK, half for dV, on
// natural tiles; two chunks requested ahead.  Half the LDS reads of 16 columns a wave (LDS 33 -> 25 % of the
// clocks); waits are what is left (43 % of a wave's life).
// ---------------------------------------------------------------------------
template <int D, int LD, bool ADD>
__global__ __launch_bounds__(4 * D, 2) void ks_bwd_dkv_wide(
    const __bf16 *__restrict__ Q, const __bf16 *__restrict__ K, const __bf16 *__restrict__ V,
    const float *__restrict__ G, const __bf16 *__restrict__ dO, __bf16 *__restrict__ dK, __bf16 *__restrict__ dV,
    const float *__restrict__ ws, const float *__restrict__ dprime, int N, int nseg, SegMap sm,
    size_t slot_floats, int, float a, float b, float *__restrict__ Pk, float *__restrict__ Pv,
    Blocks bl)
{
    constexpr int LX = Mode<P16>::LX, NW = D / 16, NC = D / 32, PL = NTile<D>::PLANE, WPL = NTile<32>::PLANE;
    typedef Chunk<__bf16, D, LD> CH;
    typedef BwdSlot<D> SL;
    __shared__ __align__(16) __bf16 lds[4 * PL + 2 * LX * WPL];
    __shared__ __align__(16) __bf16 frs[2][3 * CR], fdl[2][3 * CR];  // 1/g, dprime/g as operands
    __shared__ __align__(16) float rsb[2][CR], dlb[2][CR], vecs[2 * D];  // 1/g, dprime; u and w
    __bf16 *Kt = lds, *Vt = Kt + PL, *Qt = Vt + PL, *dOt = Qt + PL, *Ct = dOt + PL, *Wt = Ct + LX * WPL;

    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    if constexpr (LD > D) {
        Q += D * at.i;
        K += D * at.i;
        dK += D * at.i;
        V += D * at.j;
        dO += D * at.j;
        dV += D * at.j;
        ws += at.id * bl.slots;
        dprime += at.j * bl.rows;
        if (at.i) a = 0.f;
        Pk += at.i * bl.part;
        Pv += at.j * bl.part;
    }
    const int bh = wg / nseg, seg = wg % nseg;
    const size_t base = (size_t)bh * N * LD;
    const __bf16 *Qp = Q + base, *Kp = K + base, *Vp = V + base, *dOp = dO + base;
    const float *Gp = G + (size_t)bh * N, *dp = dprime + (size_t)bh * N;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 32, h = l / 32;
    const int wv = __builtin_amdgcn_readfirstlane(t / 64);
    const int half = wv / NC, w = wv % NC;  // half 0: dK; half 1: dV; columns 32 w ..
    const Lanes32<D> ln(l);
    const int wrow = Lanes32<32>(l).row;

    // the half's tiles: of the state product, of the own columns, of the update; its weights
    const __bf16 *Yt = half ? Kt : Vt, *Et = half ? dOt : Qt, *At = half ? Qt : dOt, *Xt = half ? Wt : Ct;
    f16v st[NC];  // half 0: R^T, rows j, columns r;  half 1: R, rows r, columns j
    float vec = 0.f;  // u or w, column c
#pragma unroll
    for (int rb = 0; rb < NC; ++rb) st[rb] = zero16();
    if (seg < nseg - 1) {
        const float *slot = ws + ((size_t)bh * nseg + seg) * slot_floats, *R = slot + SL::R;
#pragma unroll
        for (int rb = 0; rb < NC; ++rb)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int r = 32 * rb + 16 * (k / 2) + 8 * h + 4 * (k % 2);
                if (half) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[rb][4 * k + e] = R[(r + e) * D + 32 * w + c];
                } else {
                    const f4v x = *reinterpret_cast<const f4v *>(R + (32 * w + c) * D + r);
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[rb][4 * k + e] = x[e];
                }
            }
        vec = slot[(half ? SL::W : SL::U) + 32 * w + c];
    }
    vecs[half * D + 32 * w + c] = vec;
    if (t < 64) {  // weight blocks that stay zero: rows n 16 .., columns i 0 .. 15
        put_weights<LX>(Ct, 16 + l % 16, 0, l / 16, f4v{0.f, 0.f, 0.f, 0.f});
        put_weights<LX>(Wt, 16 + l % 16, 0, l / 16, f4v{0.f, 0.f, 0.f, 0.f});
    }

    const long nchunks = (row1 - row0 + CR - 1) / CR;
    struct Set {
        CH k, v, q, d;
    } sets[2];
    float gd = 0.f;  // first wave: g of row l (l < 32), dprime of row l - 32 of the next chunk
    auto request_gd = [&](long c0) __attribute__((always_inline)) {
        if (wv == 0) gd = (t < CR ? Gp : dp)[min((unsigned)c0 + t % CR, (unsigned)N - 1)];
    };
    // 1/g and dprime of the chunk starting at c0 into buffer `par`
    auto post_factors = [&](long c0, int par) {
        if (wv != 0) return;
        const float y = post_descending<false>(rsb[par], dlb[par], t, (int)(row1 - c0), gd);
        store_row_factor<3>((t < CR ? frs : fdl)[par], t % CR, y);
    };
    auto put = [&](const CH &x, __bf16 *tile) __attribute__((always_inline)) {
        *reinterpret_cast<u4v *>(tile + NTile<D>::quad(CH::row(0), CH::quad(0))) = x.raw[0];
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const long cl = row0 + max(nchunks - 1 - i, 0L) * CR;
        sets[i].k.load(Kp, cl, N);
        sets[i].v.load(Vp, cl, N);
        sets[i].q.load(Qp, cl, N);
        sets[i].d.load(dOp, cl, N);
    }
    request_gd(row0 + (nchunks - 1) * CR);
    post_factors(row0 + (nchunks - 1) * CR, 0);
    auto chunk = [&](long ci, Set &cur, int par) __attribute__((always_inline)) {
        const long c0 = row0 + ci * CR;
        const float *rs = rsb[par], *dl = dlb[par];
        const bool lo_on = c0 < sm.lo_rows;  // second plane of the intermediates: early rows
        block_sync();
        put(cur.k, Kt);
        put(cur.v, Vt);
        put(cur.q, Qt);
        put(cur.d, dOt);
        block_sync();
        const long cn = row0 + max(ci - 2, 0L) * CR;
        f16v old = zero16();  // shares that the launch before left
        if constexpr (ADD) {
            old = load_cols32((half ? Pv : Pk) + ((size_t)bh * N + c0) * D, D, 32 * w, (int)(row1 - c0), l);
        }
        cur.k.load(Kp, cn, N);
        cur.v.load(Vp, cn, N);
        request_gd(row0 + max(ci - 1, 0L) * CR);
        // ---- phase A: weight blocks Cm' and W (rows i, columns n) ----
#pragma unroll 1
        for (int pidx = wv; pidx < 6; pidx += NW) {
            const int q = pidx >= 3 ? pidx - 3 : pidx, ib = q ? 1 : 0, nb = q == 2 ? 1 : 0;
            const int n = l % 16, g = l / 16;
            const bool cm = pidx < 3;
            f4v x = block16<D>(cm ? dOt : Qt, ib, cm ? Vt : Kt, nb, ln.row16);
            x = descending_weight<false, false>(x, cm, ib, nb, rs, dl, nullptr, nullptr, a, b, n, g);
            with_planes<LX>(lo_on, [&](auto np) { put_weights<np.value>(cm ? Ct : Wt, nb * 16 + n, ib, g, x); });
        }
        f16v f;  // rows = the wave's columns, columns n
        with_planes<LX>(lo_on, [&](auto np) { f = state_rows<D, np.value>(st, Yt, ln.row); });
        bf8v own[2][1];
#pragma unroll
        for (int kr = 0; kr < 2; ++kr) own[kr][0] = load_col_frag<D>(Et, ln.own, w, kr);
        cur.q.load(Qp, cn, N);
        cur.d.load(dOp, cn, N);
        block_sync();
        // ---- phase B ----
        f16v y;
        with_planes<LX>(lo_on, [&](auto np) { y = weight_product<np.value>(own, Xt, wrow); });
        // dK: b (f + y - u);  dV: b f + y + a w
        const float ys = half ? 1.f : b, vs = half ? a : -b;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f4v vq = *reinterpret_cast<const f4v *>(vecs + half * D + 32 * w + 8 * q + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) f[4 * q + e] = b * f[4 * q + e] + (ys * y[4 * q + e] + vs * vq[e]);
        }
        if constexpr (ADD) {
            f += old;
        }
        store_grad32<D, LD>((half ? dV : dK) + base + (size_t)c0 * LD, (half ? Pv : Pk) + ((size_t)bh * N + c0) * D,
                            ADD, 32 * w, (int)(row1 - c0), l, f);
        vec += weighted_sum(own, half ? frs[par] : fdl[par], h);
        vecs[half * D + 32 * w + c] = vec;
        with_planes<LX>(lo_on, [&](auto np) {
            bf8v og[2][np.value];
            scale_own<np.value>(og, own, rs, h);
            update_rows<D, np.value>(st, At, ln.upd, og);
        });
        post_factors(row0 + max(ci - 1, 0L) * CR, par ^ 1);
    };
    for (long ci = nchunks - 1; ci >= 0; ci -= 2) {
        chunk(ci, sets[0], 0);
        if (ci > 0) chunk(ci - 1, sets[1], 1);
    }
}

// ---------------------------------------------------------------------------
// Backward without the mask: dK_c = b (V_c R^T - 1 u^T), dV_c = a 1 w^T + b K_c R, R, u, w the sums
// over the whole sequence.
// LD > D: ADD as above.
// ---------------------------------------------------------------------------
template <int MODE, int D, int LD, bool ADD>
__global__ __launch_bounds__(4 * D, 2) void ks_bwd_dkv_read(
    const typename Mode<MODE>::TIO *__restrict__ K, const typename Mode<MODE>::TIO *__restrict__ V,
    typename Mode<MODE>::TIO *__restrict__ dK, typename Mode<MODE>::TIO *__restrict__ dV,
    const float *__restrict__ ws, int N, int nseg, SegMap sm, size_t slot_floats, float a, float b,
    float *__restrict__ Pk, float *__restrict__ Pv, Blocks bl)
{
    typedef Mode<MODE> MD;
    typedef typename MD::TIO TIO;
    constexpr int LQ = MD::LQ, LV = MD::LV, LX = MD::LX;
    constexpr bool SWAP = MD::SWAP, QT = MD::QT, PROJ = MD::NORM;
    constexpr int NW = D / 16, NRB = D / 16, PL = Tile<D>::PLANE;
    typedef Chunk<TIO, D, LD> CH;
    typedef BwdSlot<D> SL;
    __shared__ __align__(16) __bf16 lds[LQ * PL + LV * PL];
    __shared__ __align__(16) float kinv[PROJ ? CR : 4], dots[PROJ ? NW * CR : 4];  // 1 / |k|
    __bf16 *Kt = lds, *Vt = Kt + LQ * PL;  // operand-ordered

    int wg = blockIdx.x;
    const Block at = block_of<(LD > D)>(bl, wg);
    if constexpr (LD > D) {
        K += D * at.i;
        dK += D * at.i;
        V += D * at.j;
        dV += D * at.j;
        ws += at.id * bl.slots;
        if (at.i) a = 0.f;
        Pk += at.i * bl.part;
        Pv += at.j * bl.part;
    }
    const int bh = wg / nseg, seg = wg % nseg;
    const size_t base = (size_t)bh * N * LD;
    const TIO *Kp = K + base, *Vp = V + base;
    TIO *dKp = dK + base, *dVp = dV + base;
    const long row0 = seg_row(sm, seg, nseg, N), row1 = seg_row(sm, seg + 1, nseg, N);
    const int t = threadIdx.x, l = t % 64, c = l % 16, g = l / 16;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const Lanes<D, (D >= 128)> ln(c, g);

    const float *slot = ws + (size_t)bh * nseg * slot_floats;
    Blk Ra[NRB], Rb[NRB];  // R: rows r, columns j = 16w + c;  R^T: rows j, columns r = 16w + c
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) Ra[rb].set(i, slot[SL::R + (rb * 16 + 4 * g + i) * D + w * 16 + c]);
        Rb[rb].v = *reinterpret_cast<const f4v *>(slot + SL::R + (w * 16 + c) * D + rb * 16 + 4 * g);
    }
    Sum<SWAP> uacc, wacc;  // u, w
    uacc.load(slot + SL::U, w, c, g);
    wacc.load(slot + SL::W, w, c, g);

    const long nchunks = (row1 - row0 + CR - 1) / CR;
    struct Set {
        CH k, v;
    } sets[MD::DEPTH];
#pragma unroll
    for (int i = 0; i < MD::DEPTH; ++i) {
        const long cl = row0 + max(nchunks - 1 - i, 0L) * CR;
        sets[i].k.load(Kp, cl, N);
        sets[i].v.load(Vp, cl, N);
    }
    auto chunk = [&](long ci, Set &cur) __attribute__((always_inline)) {
        const long c0 = row0 + ci * CR;
        const bool lo_on = c0 < sm.lo_rows;  // second plane of the intermediates: early rows
        block_sync();
        stage<MD::NORM, true, LQ>(cur.k, Kt, PROJ ? kinv : nullptr);
        cur.v.template store<true, LV>(Vt);
        if (__builtin_expect(cur.v.top() > kLargestBf16, 0)) cur.v.template store_any<true>(Vt);
        block_sync();
        const long cn = row0 + max(ci - MD::DEPTH, 0L) * CR;
        f4v oldk[2] = {}, oldv[2] = {};  // shares that the launch before left
        if constexpr (ADD) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const size_t at = (size_t)(c0 + m * 16) * LD, pat = ((size_t)bh * N + c0 + m * 16) * D;
                const int nrows = (int)(row1 - c0) - m * 16;
                oldk[m] = load_grad<SWAP, D, LD>(dKp + at, Pk + pat, w, nrows, l);
                oldv[m] = load_grad<SWAP, D, LD>(dVp + at, Pv + pat, w, nrows, l);
            }
        }
        cur.k.load(Kp, cn, N);
        cur.v.load(Vp, cn, N);
        f4v kh[2], kl[2];  // rows n, columns r (SWAP), or rows r, columns n
#pragma unroll
        for (int m = 0; m < 2; ++m) kh[m] = kl[m] = f4v{0.f, 0.f, 0.f, 0.f};
        with_planes<LX>(lo_on, [&](auto n) { state_product<D, n.value, LV, SWAP>(kh, kl, Rb, Vt, ln); });
        f4v x[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) x[m] = b * (kh[m] + kl[m] - uacc.v);
        if constexpr (PROJ)
            project_chunk<SWAP, true, D, LQ>(x, Kt, ln, QT ? nullptr : kinv, dots, kinv, w, c, g);
#pragma unroll
        for (int m = 0; m < 2; ++m)
            store_grad<SWAP, D, LD>(dKp + (size_t)(c0 + m * 16) * LD,
                                    Pk + ((size_t)bh * N + c0 + m * 16) * D, ADD, w,
                                    (int)(row1 - c0) - m * 16, l, x[m], oldk[m]);
        f4v vh[2], vl[2];  // rows n, columns j (SWAP), or rows j, columns n
#pragma unroll
        for (int m = 0; m < 2; ++m) vh[m] = vl[m] = f4v{0.f, 0.f, 0.f, 0.f};
        with_planes<LX>(lo_on, [&](auto n) { state_product<D, n.value, LQ, SWAP>(vh, vl, Ra, Kt, ln); });
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const f4v f = a * wacc.v + (MD::RN ? b * kinv[m * 16 + c] : b) * (vh[m] + vl[m]);
            store_grad<SWAP, D, LD>(dVp + (size_t)(c0 + m * 16) * LD,
                                    Pv + ((size_t)bh * N + c0 + m * 16) * D, ADD, w,
                                    (int)(row1 - c0) - m * 16, l, f, oldv[m]);
        }
    };
    for (long ci = nchunks - 1; ci >= 0; ci -= MD::DEPTH) {
        chunk(ci, sets[0]);
        if (MD::DEPTH == 2 && ci > 0) chunk(ci - 1, sets[MD::DEPTH - 1]);
    }
}

// Rows a workgroup of ks_fwd_read takes, 128 at least: eight workgroups a CU at D <= 32, four beyond
// (as many as registers allow).  At D = 128 a workgroup reads a state of 64 KB first, as much as 128
// bf16 rows in and out, so that short sequences get two or one a CU instead of less than 160 rows.
// bf16, D = 128, forward pass, 192 slices of 300 rows: 25.8 us at 128 rows, 22.5 at 300; 80 of 1000:
// 35.3 at 128, 33.0 at 192, 35.1 at 320; 12 of 500: 16.8 at 128, 20.2 at 320.
int read_rows(int BH, int N, int D)
{
    for (int per_cu = D <= 32 ? 8 : 4;; per_cu /= 2) {
        const long want = max((256L * per_cu + BH / 2) / BH, 1L), rows = (N + want - 1) / want;
        if (D < 128 || rows >= 160 || per_cu == 1) return (int)((max(rows, 128L) + 63) / 64 * 64);
    }
}

// Whether the masked apply kernels add the segments' slots up themselves (add_slots) instead of a scan between
// the kernels: up to five segments at D = 64, where a workgroup reads four slots of 16 KB at most, up to nine below
// (4 KB a slot).  A step, us, scan / in the kernels: D = 64, bf16, 128 slices of 600 rows (four segments) 64.1 / 59.8,
// 120 of 1000 73.7 / 69.8, fp32, 128 of 600 108.4 / 103.4; D = 32, fp32, 8 of 300 (five) 28.4 / 26.6; eight segments,
// fp32, D = 64, 64 of 4096 280 / 282, fourteen, bf16, 36 of 5003 98 / 113; sixteen, bf16, D = 32, 64 of 4096 81 / 90.  At
// D = 128, 64 KB a slot, it is no faster with four (fp32, 64 of 1000 201 / 199) and slower with eight (16 of 1000
// 103 / 117).
bool folds_scan(const Problem &pr, int nseg)
{
    return pr.causal && nseg <= (pr.D <= 32 ? 9 : pr.D == 64 ? 5 : 1);
}

// ks_kv_state with non-temporal loads where what it reads is not found in the last-level cache (256 MB) afterwards:
// K and V (tensors = 2) exceed it, or, where the pass reads them once, all four tensors do.  It then reads 4.8
// to 6.5 TB/s, and 4.0 to 5.5 with plain loads; where the pass before left that cache full of stores, part of that is
// their way to memory, left to the next kernel (step without the mask, fp32, D = 64, 64 slices of 16384 rows: sums 137
// and 112, apply kernel 95 and 117).  Plain / non-temporal, us, 64 slices, K and V of 300 MB: bf16, D = 64, forward
// 205 / 182, without the mask 154 / 129, prefill and forward 259 / 236, step 601 / 586; fp32, D = 64, 220 / 208,
// 148 / 133, 289 / 276, 670 / 660; fp32, D = 128, 273 / 268, 182 / 178.  Of 90 and 200 MB, where the apply kernel still
// finds some of K and V: bf16, D = 64, forward 60.0 / 62.3, 119 / 123, prefill 151 / 160.  Without the mask the line
// shows at K and V of 128 MB: forward, bf16, D = 64, of 100 MB 42.4 / 42.3, of 135 64.1 / 55.0, of 170 88.3 / 67.9.
// At head size 256 the block problems of a launch read K and V after one another: plain loads.
template <int MODE, int D, bool TRANSPOSED, int LD, bool LONG>
auto kv_state(const Problem &pr, int tensors)
{
    const size_t bytes = sizeof(typename Mode<MODE>::TIO) * (size_t)pr.BH * pr.N * LD * tensors;
    return LD <= D && bytes > (size_t)256 << 20 ? ks_kv_state<MODE, D, TRANSPOSED, LD, LONG, (LD <= D)>
                                                : ks_kv_state<MODE, D, TRANSPOSED, LD, LONG, false>;
}

template <int MODE, int D, int LD>
la_status run_forward(const Problem &pr, const Plan &pl, const void *Qv, const void *Kv,
                      const void *Vv, void *Ov, float *G, float *ws, float *saved, hipStream_t st,
                      Tracer &tc, const BlockScratch &bs)
{
    typedef typename Mode<MODE>::TIO TIO;
    const TIO *Q = (const TIO *)Qv, *K = (const TIO *)Kv, *V = (const TIO *)Vv;
    TIO *O = (TIO *)Ov;
    const int nseg = pl.nseg, nrun = pr.causal ? nseg - 1 : nseg;
    const dim3 block(4 * D);
    const bool fold = folds_scan(pr, nseg);
    const size_t slots = bs.together ? split_slots(pl, pr.BH) : 0;
    const auto blocks = [&](int lg, unsigned ids) {
        return Blocks{lg, ids, slots, pl.saved_bytes / sizeof(float), bs.together ? (size_t)pr.BH * pr.N * D : 0, 0};
    };
    const auto sums = [&](const Blocks &bl) {
        if (nrun == 0) return;
        (pr.causal ? kv_state<MODE, D, false, LD, false>(pr, 2) : kv_state<MODE, D, false, LD, true>(pr, 4))<<<
            dim3(pr.BH * nrun << bl.lg), block, 0, st>>>(
            K, V, ws, pr.N, nseg, nrun, pl.map, pl.slot_floats, pr.causal ? 1 : 0, nullptr, bl);
        tc.mark("fwd_state");
        if (fold) return;
        launch_scan_slots(ws, pr.BH << bl.lg, nseg, pl.slot_floats, 0, D * D + 2 * D, pr.causal ? 0 : 2,
                          pr.causal ? 1 : 0, nseg - 1, st);
        tc.mark("scan_slots");
    };
    const auto apply = [&](const Blocks &bl, bool add) {
        float *g = LD > D && !add ? bs.g : G;
        if (pr.causal) {
            auto *kernel = add ? ks_fwd_apply<MODE, D, LD, (LD > D)> : ks_fwd_apply<MODE, D, LD, false>;
            kernel<<<dim3(pr.BH * nseg << bl.lg), block, 0, st>>>(
                Q, K, V, O, g, ws, saved, pr.N, nseg, pl.map, pl.slot_floats, fold, pl.saved_floats, pr.a, pr.b, bs.g,
                bs.f, bl);
        } else {
            const int rows_wg = read_rows(pr.BH << bl.lg, pr.N, D), nwg = (pr.N + rows_wg - 1) / rows_wg;
            auto *kernel = add ? ks_fwd_read<MODE, D, LD, (LD > D)> : ks_fwd_read<MODE, D, LD, false>;
            kernel<<<dim3(pr.BH * nwg << bl.lg), block, 0, st>>>(
                Q, O, g, ws, saved, pr.N, nseg, nwg, rows_wg, pl.map.lo_rows, pl.slot_floats, pl.saved_floats, pr.a,
                pr.b, bs.g, bs.f, bl);
        }
        tc.mark("fwd_apply");
    };
    if (LD <= D) {
        sums(Blocks());
        apply(Blocks(), false);
    } else if (bs.together) {
        sums(blocks(2, 0xe4));          // all four
        apply(blocks(1, 0x4), false);   // 0 and 1: the shares of the first halves of Q and K
        apply(blocks(1, 0xe), true);    // 2 and 3
    } else {
        for (unsigned j = 0; j < 2; ++j)
            for (unsigned i = 0; i < 2; ++i) {
                sums(blocks(0, 2 * i + j));
                apply(blocks(0, 2 * i + j), i == 1);
            }
    }
    return launch_status();
}

// The ascending masked sweep: two halves of a workgroup at D = 32, one kind of waves beyond.
template <int MODE, int D, int LD, bool ADD>
constexpr auto ks_bwd_dq_masked()
{
    if constexpr (D == 32) return ks_bwd_dq_halves<MODE, D, LD>;
    else return ks_bwd_dq<MODE, D, true, LD, ADD>;
}

// The descending masked sweep: 32 columns a wave for bf16 at D = 128, whose tiles and states leave room for
// it (us, 32 columns and 16 with four waves a SIMD, medians of six runs: 128 slices of 2048 rows 109 and 118, 16
// of 131072 825 and 911, 64 of 500 31.0 and 32.5; a step at head size 256, 64 of 4096, one block problem after
// another, 1596 and 1609).  fp32 at D = 128 is within 2 % either way; at D = 64 the four waves are faster
// (bf16, 36 slices of 5003 rows 30.0 against 34.2).
template <int MODE, int D, int LD, bool ADD>
constexpr auto ks_bwd_dkv_masked()
{
    if constexpr (MODE == P16 && D == 128) return ks_bwd_dkv_wide<D, LD, ADD>;
    else return ks_bwd_dkv<MODE, D, LD, ADD>;
}

// dK == nullptr: the ascending sweep alone (dQ and the per-row o . dO).
template <int MODE, int D, int LD>
la_status run_backward(const Problem &pr, const Plan &pl, const void *Qv, const void *Kv,
                       const void *Vv, const void *Ov, const float *G, const void *dOv, void *dQv,
                       void *dKv, void *dVv, float *ws, const float *saved, hipStream_t st,
                       Tracer &tc, const BlockScratch &bs)
{
    typedef typename Mode<MODE>::TIO TIO;
    typedef BwdSlot<D> SL;
    const TIO *Q = (const TIO *)Qv, *K = (const TIO *)Kv, *V = (const TIO *)Vv,
              *O = (const TIO *)Ov, *dO = (const TIO *)dOv;
    TIO *dQ = (TIO *)dQv, *dK = (TIO *)dKv, *dV = (TIO *)dVv;
    const int nseg = pl.nseg, nrun = pr.causal ? nseg - 1 : nseg;
    constexpr bool SPLIT = LD > D;
    float *dprime = SPLIT ? bs.delta : ws + pl.delta_offset_floats;
    const bool fold = folds_scan(pr, nseg);
    const dim3 block(4 * D), block2(8 * D);
    const size_t slots = split_slots(pl, pr.BH), T = (size_t)pr.BH * pr.N;
    const auto blocks = [&](int lg, unsigned ids) {
        return SPLIT ? Blocks{lg, ids, slots, saved ? pl.saved_bytes / sizeof(float) : slots, T * D, (T + 63) / 64 * 64}
                     : Blocks();
    };
    const int all = SPLIT ? 2 : 0;  // all four block problems
    // forward-running sums before every segment: handed over by the forward pass, or
    // per-segment sums (none needed from a masked pass's last segment) and a scan here
    if ((!saved || bs.handed) && nrun > 0) {
        (pr.causal ? kv_state<MODE, D, true, LD, false>(pr, 2) : kv_state<MODE, D, true, LD, true>(pr, 4))<<<
            dim3(pr.BH * nrun << all), block, 0, st>>>(
            K, V, ws, pr.N, nseg, nrun, pl.map, pl.slot_floats, pr.causal ? 1 : 0, bs.handed, blocks(all, 0xe4));
        if (!bs.handed) tc.mark("bwd_state");  // one entry with the scan where both return at once (LA_MAX_TRACE)
        if (saved || !fold) {
            launch_scan_slots(ws, pr.BH << all, nseg, pl.slot_floats, SL::ST, SL::R - SL::ST, pr.causal ? 0 : 2,
                              pr.causal ? 1 : 0, nseg - 1, st, bs.handed, pr.BH);
            tc.mark(bs.handed ? "bwd_state_scan" : "scan_slots");
        }
    }
    const float *sinit = saved ? saved : ws;
    const size_t sinit_floats = saved ? pl.saved_floats : pl.slot_floats;
    const auto ascend = [&](const Blocks &bl, auto add) {
        constexpr bool ADD = decltype(add)::value;
        auto *dq = !pr.causal ? ks_bwd_dq<MODE, D, false, LD, ADD> : ks_bwd_dq_masked<MODE, D, LD, ADD>();
        dq<<<dim3(pr.BH * nseg << bl.lg), pr.causal && D == 32 ? block2 : block, 0, st>>>(
            Q, K, V, O, G, dO, dQ, ws, sinit, sinit_floats, dprime, pr.N, nseg, pl.map, pl.slot_floats,
            fold && !saved, pr.b, bs.q, bs.handed, bl);
        tc.mark("bwd_dq");
    };
    const auto descend = [&](const Blocks &bl, auto add) {
        constexpr bool ADD = decltype(add)::value;
        const dim3 grid(pr.BH * nseg << bl.lg);
        if (pr.causal) {
            auto *dkv = ks_bwd_dkv_masked<MODE, D, LD, ADD>();
            dkv<<<grid, MODE == P16 && D == 128 ? block : block2, 0, st>>>(
                Q, K, V, G, dO, dK, dV, ws, dprime, pr.N, nseg, pl.map, pl.slot_floats, fold, pr.a, pr.b, bs.k, bs.v,
                bl);
        } else {
            ks_bwd_dkv_read<MODE, D, LD, ADD><<<grid, block, 0, st>>>(
                K, V, dK, dV, ws, pr.N, nseg, pl.map, pl.slot_floats, pr.a, pr.b, bs.k, bs.v, bl);
        }
        tc.mark("bwd_dkv");
    };
    ascend(blocks(SPLIT, 0x8), std::false_type());  // D = 256: block problems 0 and 2, which begin dQ
    if constexpr (SPLIT) ascend(blocks(1, 0xd), std::true_type());  // 1 and 3, which add to it
    if (!dK) return launch_status();
    // reverse-running sums left by the ascending sweep
    if (!pr.causal || (nseg > 1 && !fold)) {
        launch_scan_slots(ws, pr.BH << all, nseg, pl.slot_floats, SL::R, SL::END - SL::R, pr.causal ? 1 : 2, 0,
                          pr.causal ? nseg - 2 : nseg - 1, st);
        tc.mark("scan_slots_rev");
    }
    descend(blocks(SPLIT, 0xc), std::false_type());  // 0 and 3, which begin all of dK and dV
    if constexpr (SPLIT) descend(blocks(1, 0x9), std::true_type());  // 1 and 2, which add to them
    return launch_status();
}

template <int MODE, int D, int LD>
la_status run_totals(const Problem &pr, const Plan &pl, const void *K, const void *V, float *ws, int block,
                     hipStream_t st)
{
    typedef typename Mode<MODE>::TIO TIO;
    const bool all = LD > D && pl.together;
    const Blocks bl = all ? Blocks{2, 0xe4, split_slots(pl, pr.BH), 0, 0, 0} : Blocks{0, (unsigned)block, 0, 0, 0, 0};
    kv_state<MODE, D, false, LD, true>(pr, 2)<<<dim3(pr.BH * pl.nseg << bl.lg), dim3(4 * D), 0, st>>>(
        (const TIO *)K, (const TIO *)V, ws, pr.N, pl.nseg, pl.nseg, pl.map, pl.slot_floats, 0, nullptr, bl);
    return launch_status();
}

int mode_of(const Problem &pr)
{
    return pr.dt == LA_F32 ? (pr.norm_qk ? N32 : P32) : (pr.norm_qk ? N16 : P16);
}

}  // namespace

#define LA_BY_MODE(CALL)                                   \
    switch (mode_of(pr) * 1024 + pr.D + (ld == 256)) {     \
        case P32 * 1024 + 16: return CALL(P32, 32, 16);    \
        case P32 * 1024 + 32: return CALL(P32, 32, 32);    \
        case P32 * 1024 + 64: return CALL(P32, 64, 64);    \
        case P32 * 1024 + 128: return CALL(P32, 128, 128); \
        case P32 * 1024 + 129: return CALL(P32, 128, 256); \
        case N32 * 1024 + 16: return CALL(N32, 32, 16);    \
        case N32 * 1024 + 32: return CALL(N32, 32, 32);    \
        case N32 * 1024 + 64: return CALL(N32, 64, 64);    \
        case N32 * 1024 + 128: return CALL(N32, 128, 128); \
        case P16 * 1024 + 16: return CALL(W16, 32, 16);    \
        case P16 * 1024 + 32: return CALL(P16, 32, 32);    \
        case P16 * 1024 + 64: return CALL(P16, 64, 64);    \
        case P16 * 1024 + 128: return CALL(P16, 128, 128); \
        case P16 * 1024 + 129: return CALL(P16, 128, 256); \
        case N16 * 1024 + 16: return CALL(N16, 32, 16);    \
        case N16 * 1024 + 32: return CALL(N16, 32, 32);    \
        case N16 * 1024 + 64: return CALL(N16, 64, 64);    \
        case N16 * 1024 + 128: return CALL(N16, 128, 128); \
    }                                                      \
    return LA_ERR_UNSUPPORTED

la_status planes_forward(const Problem &pr, const Plan &pl, int ld, const void *Q, const void *K,
                         const void *V, void *O, float *G, float *ws, float *saved, hipStream_t st,
                         Tracer &tc, const BlockScratch &bs)
{
#define LA_FORWARD(M, D, LD) \
    (run_forward<M, D, LD>(pr, pl, Q, K, V, O, G, ws, saved, st, tc, bs))
    LA_BY_MODE(LA_FORWARD);
}

la_status planes_backward(const Problem &pr, const Plan &pl, int ld, const void *Q, const void *K,
                          const void *V, const void *O, const float *G, const void *dO, void *dQ,
                          void *dK, void *dV, float *ws, const float *saved, hipStream_t st,
                          Tracer &tc, const BlockScratch &bs)
{
#define LA_BACKWARD(M, D, LD) \
    (run_backward<M, D, LD>(pr, pl, Q, K, V, O, G, dO, dQ, dK, dV, ws, saved, st, tc, bs))
    LA_BY_MODE(LA_BACKWARD);
}

la_status planes_totals(const Problem &pr, const Plan &pl, int ld, const void *K, const void *V,
                        float *ws, hipStream_t st, int block)
{
#define LA_TOTALS(M, D, LD) (run_totals<M, D, LD>(pr, pl, K, V, ws, block, st))
    LA_BY_MODE(LA_TOTALS);
}

}  // namespace la
