// Building blocks of the plane-split kernels (la_split.hip): fp32 arithmetic on the bf16 matrix
// pipe of gfx950.
//
// A float is the exact sum of three bf16 values, x = x0 + x1 + x2 with |x1| <= 2^-8 |x|,
// |x2| <= 2^-16 |x| (each plane the round-to-nearest bf16 of what the ones before it left), so
//     x y = x0 y0 + (x0 y1 + x1 y0) + (x0 y2 + x1 y1 + x2 y0) + O(2^-24 |x y|):
// six bf16 matrix products with fp32 accumulation stand for one fp32 product.  On gfx950 the
// bf16 pipe is sixteen times as fast as the fp32 one (v_mfma_f32_16x16x32_bf16: 16 clocks for
// 16 K flops; v_mfma_f32_16x16x4_f32: 32 clocks for 2 K), so the six take 3/8 of its time.
// A bf16 tensor is its own first plane and takes three products against a split operand.
// Exact means for magnitudes from 2^-109 on: below, x2 is subnormal in bf16 and what is lost of x is up
// to 2^-134.  Above the largest bf16, 3.3895e38, the first plane would be infinite: split4_any.
//
// Tiles.  A tile is 32 chunk rows x D columns of one tensor in bf16, one after another for each
// plane, rows D elements apart without padding.  Fragments are read two ways from the same
// tile, so nothing is stored twice:
//   rows: 16 rows x 32 columns as a product operand contracting over the columns,
//   cols: 16 columns x 32 rows contracting over the rows, through the transposing LDS read
//         (ds_read_b64_tr_b16: the 16 lanes of a group hand in 4 rows x 16 columns and get
//         one column each).
// The 32-byte granules of a row are XOR-swizzled by the row so that both kinds of read touch
// all 64 banks: the eight rows of one pass go to eight different granules of a 256-byte window.
//
// Order of the contraction index inside a 32-wide step: lane group g supplies 4g..4g+3 and
// 16+4g..16+4g+3, which is what a lane holds of two stacked accumulator blocks, so that a
// running state is fed back from its accumulators.  A tile is either "natural" (columns in
// order) or "operand-ordered" (index 16h + 4g + e at position 8g + 4h + e, one 16-byte read a
// fragment); each tensor of a kernel takes the form its most frequent read wants.
#pragma once

#include "la_blocks.h"

namespace la {
namespace {

constexpr int CR = 32;  // chunk rows

// ---- splitting ---------------------------------------------------------------------------------
// Planes of four floats.  The rounded pair is hidden from the compiler before it is widened
// again: it would otherwise convert the upper element a second time on its own instead of
// masking it out of the pair (six instructions a pair and plane instead of five; the staging
// of two tensors took 56 conversions where 24 do).
template <int L>
__device__ __forceinline__ void split4(f4v x, bf4v (&o)[L])
{
#pragma unroll
    for (int p = 0; p < L; ++p) {
        unsigned a = __builtin_bit_cast(unsigned, __builtin_convertvector((f2v{x[0], x[1]}), bf2v));
        unsigned b = __builtin_bit_cast(unsigned, __builtin_convertvector((f2v{x[2], x[3]}), bf2v));
        asm("" : "+v"(a), "+v"(b));
        o[p] = __builtin_bit_cast(bf4v, u2v{a, b});
        if (p + 1 < L)
            x -= f4v{__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u), __uint_as_float(b << 16),
                     __uint_as_float(b & 0xffff0000u)};
    }
}
// Largest magnitude of eight values (a NaN counts as nothing).  split4 leaves NaN behind an infinite
// first plane (infinity minus itself): where this exceeds kLargestBf16.
constexpr float kLargestBf16 = 0x1.fep127f;
__device__ __forceinline__ float largest(f4v x, f4v y)
{
    float m;
    asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(m) : "v"(x[0]), "v"(x[1]), "v"(x[2]));
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(x[3]), "v"(y[0]));
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(y[1]), "v"(y[2]));
    asm("v_max_f32 %0, %1, |%2|" : "=v"(m) : "v"(m), "v"(y[3]));
    return m;
}
// The three planes of any four floats.  A finite value takes the largest bf16 at most as its first
// plane; an infinity becomes +-1, 0, +-infinity: its only infinite product with another split
// value is the one with that value's first plane, which has the sign of the whole product.
__device__ __forceinline__ void split4_any(f4v x, bf4v (&o)[3])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool inf = __builtin_isinf(x[e]);
        const float first = inf ? __builtin_copysignf(1.f, x[e])
                                : __builtin_fminf(__builtin_fmaxf(x[e], -kLargestBf16), kLargestBf16);
        o[0][e] = (__bf16)first;
        const float rest = x[e] - (float)o[0][e];
        o[1][e] = (__bf16)(inf ? 0.f : rest);
        o[2][e] = (__bf16)(inf ? x[e] : rest - (float)o[1][e]);
    }
}
__device__ __forceinline__ bf8v join(bf4v lo, bf4v hi)
{
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// Operand fragment (planes) from two groups of four accumulator rows.
template <int L>
__device__ __forceinline__ void split_frag(f4v g0, f4v g1, bf8v (&o)[L])
{
    bf4v a[L], b[L];
    split4<L>(g0, a);
    split4<L>(g1, b);
#pragma unroll
    for (int p = 0; p < L; ++p) o[p] = join(a[p], b[p]);
}
__device__ __forceinline__ bf8v ones_frag()
{
    bf8v r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)1.f;
    return r;
}

// ---- long sums -----------------------------------------------------------------------------------
// A running sum with what its additions lost (Dekker's fast two-sum: exact where the sum is the larger
// operand, which it is but for the first few additions, whose roundings are small next to the end's).
// A segment's vector sums take one addition per 32 rows, and without the mask they are most of an
// output row: O = (a p + ...) / g with |p| ~ sqrt(N), the rest ~ sqrt(N / D).  Against 64 bits, unmasked
// fp32, O over 16384 rows at D = 64: 2.3e-7 with plain sums, 0.7e-7 with these; 20000 rows at D = 128:
// 2.6e-7 and 0.6e-7.
template <typename V>
struct LongSum {
    V s, lost;
    // += a product of the first planes and the products of the further ones, two accumulators: on
    // one, the small products are cut off at the large one's last bit.
    __device__ __forceinline__ void add(V hi, V lo)
    {
        const V t = s + hi;
        lost += (hi - (t - s)) + lo;
        s = t;
    }
};
// The sum; where it is not finite, neither is a number what it lost.
__device__ __forceinline__ float total(const LongSum<float> &x)
{
    return __builtin_isfinite(x.s) ? x.s + x.lost : x.s;
}
__device__ __forceinline__ f4v total(const LongSum<f4v> &x)
{
    f4v r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = total(LongSum<float>{x.s[e], x.lost[e]});
    return r;
}

// ---- products ----------------------------------------------------------------------------------
__device__ __forceinline__ f4v mfma(bf8v a, bf8v b, f4v c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Two products with the same left operand, X Y_m^T for m = 0, 1:
//   hi[m] += x0 y0;  lo[m] += the products of the further planes up to the order of the
// better-split operand, smallest first.  Two accumulators: the rounding of the small terms
// stays small, and the large one is rounded once per step.  The two blocks alternate, so that
// no product waits for the one before it.
// SWAP: the transposed result, Y_m X^T.
template <int LA, int LB, bool SWAP>
__device__ __forceinline__ void mma_pair(f4v (&hi)[2], f4v (&lo)[2], const bf8v (&a)[LA],
                                         const bf8v (&b)[2][LB])
{
    constexpr int M = (LA > LB ? LA : LB) - 1;  // highest order kept
#pragma unroll
    for (int s = M; s >= 1; --s)
#pragma unroll
        for (int p = 0; p < LA; ++p)
            if (s - p >= 0 && s - p < LB) {
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    lo[m] = SWAP ? mfma(b[m][s - p], a[p], lo[m]) : mfma(a[p], b[m][s - p], lo[m]);
            }
#pragma unroll
    for (int m = 0; m < 2; ++m) hi[m] = SWAP ? mfma(b[m][0], a[0], hi[m]) : mfma(a[0], b[m][0], hi[m]);
}
template <int LA, int LB>
__device__ __forceinline__ void mma_planes(f4v &hi, f4v &lo, const bf8v (&a)[LA], const bf8v (&b)[LB])
{
    constexpr int M = (LA > LB ? LA : LB) - 1;
#pragma unroll
    for (int s = M; s >= 1; --s)
#pragma unroll
        for (int p = 0; p < LA; ++p)
            if (s - p >= 0 && s - p < LB) lo = mfma(a[p], b[s - p], lo);
    hi = mfma(a[0], b[0], hi);
}
// The number of matrix instructions of one such product.
constexpr int products(int LA, int LB)
{
    int n = 0;
    const int M = (LA > LB ? LA : LB) - 1;
    for (int p = 0; p < LA; ++p)
        for (int q = 0; q < LB; ++q) n += p + q <= M;
    return n;
}
// The whole product of one step, smallest terms first, on one accumulator that starts at zero.
template <int LA, int LB>
__device__ __forceinline__ f4v step_product(const bf8v (&a)[LA], const bf8v (&b)[LB])
{
    constexpr int M = (LA > LB ? LA : LB) - 1;
    f4v t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = M; s >= 0; --s)
#pragma unroll
        for (int p = 0; p < LA; ++p)
            if (s - p >= 0 && s - p < LB) t = mfma(a[p], b[s - p], t);
    return t;
}
// The same for two left operands.
template <int LA, int LB>
__device__ __forceinline__ void step_pair(f4v (&t)[2], const bf8v (&a)[2][LA], const bf8v (&b)[LB])
{
    constexpr int M = (LA > LB ? LA : LB) - 1;
    t[0] = t[1] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = M; s >= 0; --s)
#pragma unroll
        for (int p = 0; p < LA; ++p)
            if (s - p >= 0 && s - p < LB) {
                t[0] = mfma(a[0][p], b[s - p], t[0]);
                t[1] = mfma(a[1][p], b[s - p], t[1]);
            }
}

// Order of the instructions of one pipeline step, the code since the last one of these: LDS
// reads first (they are for the next step), then matrix instructions with NV vector
// instructions after each.  A wave issues in order, and a matrix instruction keeps its pipe
// busy for 16 clocks: what stands between two of them is free.
template <int NDS, int NM, int NV>
__device__ __forceinline__ void step_schedule()
{
    if constexpr (NDS > 0) __builtin_amdgcn_sched_group_barrier(0x100, NDS, 0);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (NV > 0) __builtin_amdgcn_sched_group_barrier(0x002, NV, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// ---- tiles -------------------------------------------------------------------------------------
template <int D>
struct Tile {
    static_assert(D == 32 || D == 64 || D == 128, "one, two or four rows per 256 bytes");
    static constexpr int PLANE = CR * D;  // elements from one plane to the next
    static constexpr int SH = D == 128 ? 0 : (D == 64 ? 1 : 2);
    // The same for rows r and r + 16.
    static __device__ __forceinline__ int swz(int row) { return (row >> SH) & (D / 16 - 1); }
    // Offset of the four columns 4q .. 4q+3 of a row.
    static __device__ __forceinline__ int nat_quad(int row, int q)
    {
        return row * D + 16 * ((q >> 2) ^ swz(row)) + 4 * (q & 3);
    }
    static __device__ __forceinline__ int op_quad(int row, int q)
    {
        const int g = q & 3, h = (q >> 2) & 1;
        return row * D + 16 * ((2 * (q >> 3) + (g >> 1)) ^ swz(row)) + 8 * (g & 1) + 4 * h;
    }
};

// The lane's parts of fragment addresses, elements.  Column steps are XORed in: they are
// multiples of a granule, and a row's offset has no bits there.
// LOCAL: a product works its fragment addresses out anew (an XOR each) instead of keeping them
// in registers of their own across the chunk loop; for the kernels that have none to spare.
template <int D, bool LOCAL = false>
struct Lanes {
    int row;   // operand-ordered tile, row fragment: row c, lane group g's unit
    int nat;   // natural tile, row fragment (two 8-byte reads)
    int col;   // natural tile, column fragment (transposing read)
    int ocol;  // operand-ordered tile, column fragment
    __device__ __forceinline__ Lanes(int c, int g)
    {
        typedef Tile<D> T;
        row = c * D + 16 * ((g >> 1) ^ T::swz(c)) + 8 * (g & 1);
        nat = c * D + 16 * T::swz(c) + 4 * g;
        const int r = 4 * g + (c >> 2), q = c & 3;
        col = r * D + 16 * T::swz(r) + 4 * q;
        ocol = r * D + 16 * ((q >> 1) ^ T::swz(r)) + 8 * (q & 1);
    }
    static __device__ __forceinline__ int local(int x)
    {
        if constexpr (LOCAL) asm volatile("" : "+v"(x));  // not recognisable as the same value
        return x;
    }
};

__device__ __forceinline__ bf4v read_tr(const __bf16 *p)
{
    typedef __attribute__((address_space(3))) bf4v lds_bf4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf4 *)p);
}
// Rows 16 ib .. of an operand-ordered tile, columns 32 kt .. , all planes.
template <int D, int L>
__device__ __forceinline__ void load_rows(bf8v (&f)[L], const __bf16 *tile, int row, int ib, int kt)
{
    const __bf16 *p = tile + (row ^ (32 * kt)) + ib * 16 * D;
#pragma unroll
    for (int q = 0; q < L; ++q) f[q] = *reinterpret_cast<const bf8v *>(p + q * Tile<D>::PLANE);
}
// The same from a natural tile.
template <int D, int L>
__device__ __forceinline__ void load_rows_nat(bf8v (&f)[L], const __bf16 *tile, int nat, int ib,
                                              int kt)
{
    const __bf16 *p = tile + (nat ^ (32 * kt)) + ib * 16 * D;
    const __bf16 *p2 = tile + (nat ^ (32 * kt + 16)) + ib * 16 * D;
#pragma unroll
    for (int q = 0; q < L; ++q)
        f[q] = join(*reinterpret_cast<const bf4v *>(p + q * Tile<D>::PLANE),
                    *reinterpret_cast<const bf4v *>(p2 + q * Tile<D>::PLANE));
}
// Columns 16 jb .. of a natural tile, contracting over the 32 rows.
template <int D, int L>
__device__ __forceinline__ void load_cols(bf8v (&f)[L], const __bf16 *tile, int col, int jb)
{
    const __bf16 *p = tile + (col ^ (16 * jb));
#pragma unroll
    for (int q = 0; q < L; ++q)
        f[q] = join(read_tr(p + q * Tile<D>::PLANE), read_tr(p + q * Tile<D>::PLANE + 16 * D));
}
// The same from an operand-ordered tile.
template <int D, int L>
__device__ __forceinline__ void load_cols_op(bf8v (&f)[L], const __bf16 *tile, int ocol, int jb)
{
    const __bf16 *p = tile + (ocol ^ (32 * (jb >> 1))) + 4 * (jb & 1);
#pragma unroll
    for (int q = 0; q < L; ++q)
        f[q] = join(read_tr(p + q * Tile<D>::PLANE), read_tr(p + q * Tile<D>::PLANE + 16 * D));
}

// ---- staging -----------------------------------------------------------------------------------
// One chunk (32 x D) of a tensor in 16-byte loads, whole consecutive rows a wave.  A workgroup of 4 D
// threads holds it as two quads (four columns of a row) per thread: fp32, quad t % (D/4) of rows
// t / (D/4) and that + 16; bf16, two neighbouring quads of row t / (D/8).  With HALVES (8 D threads)
// fp32 is one quad a thread, and a bf16 chunk is held by one half of the workgroup, which the caller
// names.
template <typename TIO, int D, int LD, bool HALVES = false>
struct Chunk {
    static constexpr bool F32 = sizeof(TIO) == 4;
    static constexpr int PER_ROW = F32 ? D / 4 : D / 8;    // lanes that share a row
    static constexpr int NLD = F32 && !HALVES ? 2 : 1;     // 16-byte loads per thread
    static constexpr int NQ = F32 && HALVES ? 1 : 2;       // quads per thread
    static constexpr int COLS = LD < D ? LD : D;           // columns there are; the others read as zeros
    u4v raw[NLD];

    // t: the thread's index.  A kernel short of registers hands in a copy that the compiler does not
    // recognise, so that what follows from it is worked out where it is used and not kept across the
    // chunk loop.
    static __device__ __forceinline__ int row(int k, int t = threadIdx.x)
    {
        if constexpr (F32) return t / PER_ROW + 16 * k;
        else return (HALVES ? t % (4 * D) : t) / PER_ROW;
    }
    static __device__ __forceinline__ int quad(int k, int t = threadIdx.x)
    {
        return F32 ? t % PER_ROW : 2 * (t % PER_ROW) + k;
    }
    // the lane that writes a per-row result
    static __device__ __forceinline__ bool leader(int t = threadIdx.x) { return t % PER_ROW == 0; }

    // Request chunk rows [c0, c0 + 32) of X, the base of a slice of N rows (c0 < N).  The
    // buffer descriptor covers the chunk's valid rows; rows beyond them read as zeros.
    // Nothing looks at the loaded values before the tile is written, so the loads stay in
    // flight over the chunk before.  STREAM: with the non-temporal bit.
    template <bool STREAM = false>
    __device__ __forceinline__ void load(const TIO *X, long c0, int N, int t = threadIdx.x)
    {
        const long rows = (N - c0 < CR) ? N - c0 : CR;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<TIO *>(X + (size_t)c0 * LD), 0, (int)(((rows - 1) * LD + COLS) * sizeof(TIO)),
            kBufferFlags);
        int off = (row(0, t) * LD + 4 * quad(0, t)) * (int)sizeof(TIO);
        if (LD < D && 4 * quad(0, t) >= COLS) off = 1 << 30;  // out of range
#pragma unroll
        for (int k = 0; k < NLD; ++k)
            raw[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + k * 16 * LD * (int)sizeof(TIO),
                                                           0, STREAM ? 2 : 0);
    }
    __device__ __forceinline__ f4v value(int k) const
    {
        if constexpr (F32) {
            return __builtin_bit_cast(f4v, raw[k]);
        } else {
            const uint32_t a = raw[0][2 * k], b = raw[0][2 * k + 1];
            const u4v r = {a << 16, a & 0xffff0000u, b << 16, b & 0xffff0000u};
            return __builtin_bit_cast(f4v, r);
        }
    }
    // Per-quad partial sums -> row totals, in every lane that shares the row.
    static __device__ __forceinline__ void row_totals(float (&s)[NQ])
    {
        if constexpr (F32) {
#pragma unroll
            for (int k = 0; k < NQ; ++k) s[k] = reduce_adjacent<PER_ROW>(s[k]);
        } else {
            s[0] = s[1] = reduce_adjacent<PER_ROW>(s[0] + s[1]);
        }
    }
    // The tensor's own bf16 values into a one-plane tile.
    template <bool OP>
    __device__ __forceinline__ void store_raw(__bf16 *tile, int t = threadIdx.x) const
    {
        static_assert(!F32, "fp32 tensors are split");
        if constexpr (!OP) {
            *reinterpret_cast<u4v *>(tile + Tile<D>::nat_quad(row(0, t), quad(0, t))) = raw[0];
        } else {
            *reinterpret_cast<u2v *>(tile + Tile<D>::op_quad(row(0, t), quad(0, t))) = u2v{raw[0][0], raw[0][1]};
            *reinterpret_cast<u2v *>(tile + Tile<D>::op_quad(row(0, t), quad(1, t))) = u2v{raw[0][2], raw[0][3]};
        }
    }
    __device__ __forceinline__ void values(f4v (&x)[NQ]) const
    {
#pragma unroll
        for (int k = 0; k < NQ; ++k) x[k] = value(k);
    }
    // Values x into a tile of L planes.
    template <bool OP, int L>
    static __device__ __forceinline__ void store_values(__bf16 *tile, const f4v (&x)[NQ],
                                                        int t = threadIdx.x)
    {
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            __bf16 *dst = tile + (OP ? Tile<D>::op_quad(row(k, t), quad(k, t)) : Tile<D>::nat_quad(row(k, t), quad(k, t)));
            bf4v o[L];
            split4<L>(x[k], o);
#pragma unroll
            for (int p = 0; p < L; ++p) *reinterpret_cast<bf4v *>(dst + p * Tile<D>::PLANE) = o[p];
        }
    }
    // The tensor as it is: its own bits (bf16, one plane) or all planes.
    template <bool OP, int L>
    __device__ __forceinline__ void store(__bf16 *tile, int t = threadIdx.x) const
    {
        if constexpr (!F32 && L == 1) {
            store_raw<OP>(tile, t);
        } else {
            f4v x[NQ];
            values(x);
            store_values<OP, L>(tile, x, t);
        }
    }
    // Above kLargestBf16: store<OP, 3> left NaN behind an infinite plane, and the tile is written
    // once more.
    __device__ __forceinline__ float top() const
    {
        if constexpr (F32) return largest(value(0), value(NQ - 1));
        else return 0.f;
    }
    template <bool OP>
    __device__ __forceinline__ void store_any(__bf16 *tile, int t = threadIdx.x) const
    {
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            __bf16 *dst = tile + (OP ? Tile<D>::op_quad(row(k, t), quad(k, t)) : Tile<D>::nat_quad(row(k, t), quad(k, t)));
            bf4v o[3];
            split4_any(value(k), o);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<bf4v *>(dst + p * Tile<D>::PLANE) = o[p];
        }
    }
};

__device__ __forceinline__ float dot4(f4v x, f4v y)
{
    return (x[0] * y[0] + x[1] * y[1]) + (x[2] * y[2] + x[3] * y[3]);
}

// Row normalisation of Sec. 3.3 on the quads a thread holds; rows of zeros stay zeros.
// inv_out (if given) receives 1 / |row|.
template <typename CH>
__device__ __forceinline__ void normalise_quads(f4v (&x)[CH::NQ], float *inv_out, int t = threadIdx.x)
{
    float s[CH::NQ];
#pragma unroll
    for (int k = 0; k < CH::NQ; ++k) s[k] = dot4(x[k], x[k]);
    CH::row_totals(s);
#pragma unroll
    for (int k = 0; k < CH::NQ; ++k) {
        const float inv = s[k] > 0.f ? 1.f / sqrtf(s[k]) : 0.f;
        x[k] *= inv;
        if (inv_out && CH::leader(t)) inv_out[CH::row(k, t)] = inv;
    }
}

// A per-row factor of the chunk as an operand fragment: planes of 32 bf16 each, row
// 16h + 4g + e at position 8g + 4h + e.
template <int L>
__device__ __forceinline__ void store_factor(__bf16 *dst, int r, float x)
{
    const int pos = 8 * ((r >> 2) & 3) + 4 * (r >> 4) + (r & 3);
#pragma unroll
    for (int p = 0; p < L; ++p) {
        const __bf16 h = (__bf16)x;
        dst[p * CR + pos] = h;
        x -= (float)h;
    }
}
template <int L>
__device__ __forceinline__ void load_factor(bf8v (&f)[L], const __bf16 *src, int g)
{
#pragma unroll
    for (int p = 0; p < L; ++p) f[p] = *reinterpret_cast<const bf8v *>(src + p * CR + 8 * g);
}

// ---- whole products over a tile ------------------------------------------------------------------
// {hi, lo}[m] += (y st)^T: rows j = the wave's 16 state columns, columns i = rows 16 m .. of the
// operand-ordered tile y, contracting over D (SWAP: y st, rows i, columns j).  st holds the
// state's D/16 blocks.  The next
// step's fragments are read, and its share of the state is split, under this step's products.
template <int D, int LS, int LY, bool SWAP, typename LN>
__device__ __forceinline__ void state_product(f4v (&hi)[2], f4v (&lo)[2], const Blk (&st)[D / 16],
                                              const __bf16 *y, const LN &ln)
{
    const int row = LN::local(ln.row);
    constexpr int NK = D / 32, NM = 2 * products(LS, LY);
    if constexpr (NM <= 4) {  // few products a step: all fragments at once
        bf8v f[NK][2][LY];
#pragma unroll
        for (int kt = 0; kt < NK; ++kt)
#pragma unroll
            for (int m = 0; m < 2; ++m) load_rows<D, LY>(f[kt][m], y, row, m, kt);
#pragma unroll
        for (int kt = 0; kt < NK; ++kt) {
            bf8v x[LS];
            split_frag<LS>(st[2 * kt].v, st[2 * kt + 1].v, x);
            mma_pair<LS, LY, SWAP>(hi, lo, x, f[kt]);
        }
        return;
    }
    bf8v x[2][LS], f[2][2][LY];
    load_rows<D, LY>(f[0][0], y, row, 0, 0);
    load_rows<D, LY>(f[0][1], y, row, 1, 0);
    split_frag<LS>(st[0].v, st[1].v, x[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kt = 0; kt < NK; ++kt) {
        const int cur = kt & 1, nxt = cur ^ 1;
        if (kt + 1 < NK) {
            load_rows<D, LY>(f[nxt][0], y, row, 0, kt + 1);
            load_rows<D, LY>(f[nxt][1], y, row, 1, kt + 1);
            split_frag<LS>(st[2 * kt + 2].v, st[2 * kt + 3].v, x[nxt]);
        }
        mma_pair<LS, LY, SWAP>(hi, lo, x[cur], f[cur]);
        if (kt + 1 < NK) step_schedule<2 * LY, NM, (20 * LS - 16 + NM - 1) / NM + 1>();
        else __builtin_amdgcn_sched_barrier(0);
    }
}
// The same one step at a time: for four waves a SIMD, which hide each other's latencies and have half
// the registers each.
template <int D, int LS, int LY, bool SWAP, typename LN>
__device__ __forceinline__ void state_steps(f4v (&hi)[2], f4v (&lo)[2], const Blk (&st)[D / 16],
                                            const __bf16 *y, const LN &ln)
{
    const int row = LN::local(ln.row);
#pragma unroll
    for (int kt = 0; kt < D / 32; ++kt) {
        bf8v f[2][LY], x[LS];
        load_rows<D, LY>(f[0], y, row, 0, kt);
        load_rows<D, LY>(f[1], y, row, 1, kt);
        split_frag<LS>(st[2 * kt].v, st[2 * kt + 1].v, x);
        mma_pair<LS, LY, SWAP>(hi, lo, x, f);
        __builtin_amdgcn_sched_barrier(0);
    }
}
// The same with a state that stays as it is, split once: the first LS of its LL planes.
template <int D, int LS, int LL, int LY, typename LN>
__device__ __forceinline__ void fixed_product(f4v (&hi)[2], f4v (&lo)[2], const bf8v (&sp)[D / 32][LL],
                                              const __bf16 *y, const LN &ln)
{
    const int row = LN::local(ln.row);
    constexpr int NK = D / 32, NM = 2 * products(LS, LY), AHEAD = NM <= 4 ? NK : 1;
    bf8v f[AHEAD + 1][2][LY];
#pragma unroll
    for (int kt = 0; kt < AHEAD; ++kt)
#pragma unroll
        for (int m = 0; m < 2; ++m) load_rows<D, LY>(f[kt][m], y, row, m, kt);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kt = 0; kt < NK; ++kt) {
        const int cur = kt % (AHEAD + 1), nxt = (kt + AHEAD) % (AHEAD + 1);
        if (kt + AHEAD < NK) {
#pragma unroll
            for (int m = 0; m < 2; ++m) load_rows<D, LY>(f[nxt][m], y, row, m, kt + AHEAD);
        }
        bf8v x[LS];
#pragma unroll
        for (int p = 0; p < LS; ++p) x[p] = sp[kt][p];
        mma_pair<LS, LY, false>(hi, lo, x, f[cur]);
        if (kt + AHEAD < NK) step_schedule<2 * LY, NM, 0>();
    }
}
// One 16 x 16 block of X_rows . Y_rows^T over D, X natural (rows 16 xb), Y operand-ordered
// (rows 16 yb): accumulator rows = rows of X, columns = rows of Y.
template <int D, int LX, int LY, typename LN>
__device__ __forceinline__ f4v block_product(const __bf16 *xt, int xb, const __bf16 *yt, int yb,
                                             const LN &ln)
{
    const int nat = LN::local(ln.nat), row = LN::local(ln.row);
    constexpr int NK = D / 32;
    f4v hi = {0.f, 0.f, 0.f, 0.f}, lo = hi;
    if constexpr (LX * LY == 1) {
        bf8v x[NK][1], y[NK][1];
#pragma unroll
        for (int kt = 0; kt < NK; ++kt) {
            load_rows_nat<D, 1>(x[kt], xt, nat, xb, kt);
            load_rows<D, 1>(y[kt], yt, row, yb, kt);
        }
#pragma unroll
        for (int kt = 0; kt < NK; ++kt) hi = mfma(x[kt][0], y[kt][0], hi);
        return hi;
    }
    bf8v x[2][LX], y[2][LY];
    load_rows_nat<D, LX>(x[0], xt, nat, xb, 0);
    load_rows<D, LY>(y[0], yt, row, yb, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kt = 0; kt < NK; ++kt) {
        const int cur = kt & 1, nxt = cur ^ 1;
        if (kt + 1 < NK) {
            load_rows_nat<D, LX>(x[nxt], xt, nat, xb, kt + 1);
            load_rows<D, LY>(y[nxt], yt, row, yb, kt + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        mma_planes<LX, LY>(hi, lo, x[cur], y[cur]);
        __builtin_amdgcn_sched_barrier(0);
    }
    return hi + lo;
}
// st[rb] += A_rb^T B over the chunk rows: A = columns of the natural tile `at`, B = the wave's
// own column fragment.  Each step's product is formed on an accumulator of its own and added
// once, a step later, so that the state takes one rounding per chunk and the addition does not
// wait for the matrix pipe.
template <int D, int LA, int LB, typename LN>
__device__ __forceinline__ void rank_update(Blk (&st)[D / 16], const __bf16 *at, const bf8v (&b)[LB],
                                            const LN &ln)
{
    const int col = LN::local(ln.col);
    constexpr int NS = D / 32, NM = 2 * products(LA, LB);
    if constexpr (LA * LB == 1) {  // one product a block: onto the state itself
        bf8v a[2 * NS][1];
#pragma unroll
        for (int rb = 0; rb < 2 * NS; ++rb) load_cols<D, 1>(a[rb], at, col, rb);
#pragma unroll
        for (int rb = 0; rb < 2 * NS; ++rb) st[rb].v = mfma(a[rb][0], b[0], st[rb].v);
        return;
    }
    bf8v a[2][2][LA];
    f4v t[2][2];
    load_cols<D, LA>(a[0][0], at, col, 0);
    load_cols<D, LA>(a[0][1], at, col, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int cur = s & 1, nxt = cur ^ 1;
        if (s + 1 < NS) {
            load_cols<D, LA>(a[nxt][0], at, col, 2 * s + 2);
            load_cols<D, LA>(a[nxt][1], at, col, 2 * s + 3);
        }
        step_pair<LA, LB>(t[cur], a[cur], b);
        if (s > 0) {
            st[2 * s - 2].v += t[nxt][0];
            st[2 * s - 1].v += t[nxt][1];
        }
        if (s + 1 < NS) step_schedule<4 * LA, NM, 1>();
        else __builtin_amdgcn_sched_barrier(0);
    }
    st[2 * NS - 2].v += t[(NS - 1) & 1][0];
    st[2 * NS - 1].v += t[(NS - 1) & 1][1];
}

// The same two blocks at a time (four with single planes), for four waves a SIMD.
template <int D, int LA, int LB, typename LN>
__device__ __forceinline__ void rank_steps(Blk (&st)[D / 16], const __bf16 *at, const bf8v (&b)[LB], const LN &ln)
{
    const int col = LN::local(ln.col);
    constexpr int NR = D / 16;
    constexpr int AT = LA * LB == 1 && NR >= 4 ? 4 : 2;
#pragma unroll
    for (int r = 0; r < NR; r += AT) {
        bf8v a[AT][LA];
#pragma unroll
        for (int i = 0; i < AT; ++i) load_cols<D, LA>(a[i], at, col, r + i);
        if constexpr (LA * LB == 1) {
#pragma unroll
            for (int i = 0; i < AT; ++i) st[r + i].v = mfma(a[i][0], b[0], st[r + i].v);
        } else {
            f4v t[2];
            step_pair<LA, LB>(t, a, b);
            st[r].v += t[0];
            st[r + 1].v += t[1];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}
// The same for two tiles of single planes, b0 and b1: one addition to the state for both.  The matrix
// pipe cuts an accumulator off where the vector ALU rounds, so long sums gain from fewer, rounded
// additions (bf16 D = 128, S over 8192 rows against 64 bits: 1.9e-7 with one instruction a tile onto
// the state itself, 1.1e-7 so).
template <int D, typename LN>
__device__ __forceinline__ void rank_update_two(Blk (&st)[D / 16], const __bf16 *at0, const __bf16 *at1,
                                                bf8v b0, bf8v b1, const LN &ln)
{
    const int col = LN::local(ln.col);
#pragma unroll
    for (int rb = 0; rb < D / 16; ++rb) {
        bf8v a0[1], a1[1];
        load_cols<D, 1>(a0, at0, col, rb);
        load_cols<D, 1>(a1, at1, col, rb);
        st[rb].v += mfma(a1[0], b1, mfma(a0[0], b0, f4v{0.f, 0.f, 0.f, 0.f}));
    }
}

// ---- output blocks -------------------------------------------------------------------------------
// Store a 16 x 16 fp32 block of which lane (c, g) holds rows 4g .. 4g+3 of column col0 + c: the 16
// lanes of a group write one 64-byte run of a row.  The buffer descriptor covers the block's
// first `rows_valid` rows (at most 16, possibly none): stores beyond them are dropped.
__device__ __forceinline__ void store_cols_block(float *base, int ld, int col0, int rows_valid, int c,
                                                 int g, f4v x)
{
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, valid_rows(rows_valid) * ld * 4, kBufferFlags);
    const int off = (4 * g * ld + col0 + c) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[e]), rsrc, off + e * ld * 4, 0, 0);
}
// What the block holds, in the same layout.
__device__ __forceinline__ f4v load_cols_block(const float *base, int ld, int col0, int rows_valid, int c, int g)
{
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(base), 0, valid_rows(rows_valid) * ld * 4, kBufferFlags);
    const int off = (4 * g * ld + col0 + c) * 4;
    f4v x;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off + e * ld * 4, 0, 0));
    return x;
}

// Backward of the row normalisation (Sec. 3.3) on gradient blocks still in registers:
//   dx = (dxhat - xhat (xhat . dxhat)) / |x|     for every row of the chunk.
// x[m], xh[m]: rows 16 m + 4 g .. + 3, column 16 w + c of dxhat and xhat.  The row's dot product
// runs over the 16 lanes of a group and over the waves: per-wave shares meet in dots[NW][32]
// (LDS), which costs one workgroup barrier.  Every thread of the workgroup must call this.
template <int NW>
__device__ __forceinline__ void project_cols(f4v (&x)[2], const f4v (&xh)[2], float *dots,
                                             const float *inv, int w, int c, int g)
{
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        f4v s;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = reduce_adjacent<16>(x[m][e] * xh[m][e]);
        if (c == 0) *reinterpret_cast<f4v *>(dots + w * CR + m * 16 + 4 * g) = s;
    }
    block_sync();
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        f4v dot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < NW; ++v) dot += *reinterpret_cast<const f4v *>(dots + v * CR + m * 16 + 4 * g);
        x[m] = (x[m] - xh[m] * dot) * *reinterpret_cast<const f4v *>(inv + m * 16 + 4 * g);
    }
}
// The values behind a column fragment: rows 4g .. 4g+3 and 16+4g .. of the lane's column.
template <int L>
__device__ __forceinline__ void frag_values(f4v (&x)[2], const bf8v (&f)[L])
{
    x[0] = x[1] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = L - 1; p >= 0; --p) {
        x[0] += bf4_to_float(__builtin_shufflevector(f[p], f[p], 0, 1, 2, 3));
        x[1] += bf4_to_float(__builtin_shufflevector(f[p], f[p], 4, 5, 6, 7));
    }
}

// Values behind a 4-column group of a tile row (all planes).
template <int D, int L>
__device__ __forceinline__ void quad_values(float (&x)[4], const __bf16 *src)
{
    f4v q = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = L - 1; p >= 0; --p)
        q += bf4_to_float(*reinterpret_cast<const bf4v *>(src + p * Tile<D>::PLANE));
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = q[e];
}

// ---- weight blocks -------------------------------------------------------------------------------
// A weight tile holds a 32 x 32 block of intermediates as a 32-column operand-ordered tile.
// Four values of row `row`, columns 16 h + 4 g .. + 3, into its planes.
template <int L>
__device__ __forceinline__ void store_weights(__bf16 *tile, int row, int h, int g, f4v x)
{
    typedef Tile<32> W;
    __bf16 *dst = tile + row * 32 + 16 * ((g >> 1) ^ W::swz(row)) + 8 * (g & 1) + 4 * h;
    bf4v o[L];
    split4<L>(x, o);
#pragma unroll
    for (int p = 0; p < L; ++p) *reinterpret_cast<bf4v *>(dst + p * W::PLANE) = o[p];
}

// Call fn with the number of planes the intermediates of this chunk take (a constant inside).
template <int LX, typename Fn>
__device__ __forceinline__ void with_planes(bool lo_on, Fn fn)
{
    if constexpr (LX == 2) {
        if (lo_on) fn(std::integral_constant<int, 2>());
        else fn(std::integral_constant<int, 1>());
    } else {
        fn(std::integral_constant<int, LX>());
    }
}

}  // namespace
}  // namespace la
