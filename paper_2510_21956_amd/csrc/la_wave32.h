// Building blocks of the bf16 kernel whose waves own 32 columns of a D x D running state and work with
// v_mfma_f32_32x32x16_bf16 on natural tiles (ks_bwd_dkv_wide).
//
// Why 32 columns.  A SIMD issues a wave's instructions one every five clocks or so, and vector
// instructions hide behind a matrix instruction only in part: one of 32 x 32 x 16 (32 clocks)
// hides some 15 clocks of them, two of 16 x 16 x 32 (16 clocks each) 9 (measured, two waves a SIMD).
// A fragment read from LDS serves twice the columns, so a chunk takes half the LDS reads
// and about two thirds of the instructions of waves with 16 columns.
//
// Lanes: c = l % 32, h = l / 32.  An operand of a product gives lane (c, h) row (or column) c and the
// contraction indices 8h .. 8h+7 of a step of 16; an accumulator gives it column c and, in element i,
// row 8 (i / 4) + 4 h + i % 4.
//
// Tiles are natural (NTile): 32 chunk rows x D columns of one tensor as it stands.  Rows as operands
// are 16-byte units.  A state comes back as an operand straight from its accumulators: its rows are
// dealt to the accumulator positions so that the eight values a lane holds of a step of 16 rows are
// those at 8h .. 8h+7: element i = 8 s + 4 q + e of block rb is row 32 rb + 16 s + 8 h + 4 q + e.
#pragma once

#include "la_planes.h"

namespace la {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f16v zero16()
{
    return f16v{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}
__device__ __forceinline__ f16v mfma32(bf8v a, bf8v b, f16v c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4v quad_of(const f16v &x, int q)
{
    return f4v{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
}
// Sum over the two halves of a wave.
__device__ __forceinline__ float both_halves(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ---- tiles -------------------------------------------------------------------------------------
// Rows of D bf16 in units of 16 bytes, XORed by a hash of the row: 16 consecutive rows put the same
// unit into 16 different places of a 256-byte window (row reads), four consecutive rows put an
// aligned 64-byte run into four different quarters of it (transposing reads).
template <int D>
struct NTile {
    static_assert(D == 32 || D == 64 || D == 128, "one, two or four rows per 256 bytes");
    static constexpr int PLANE = CR * D;
    static __device__ __forceinline__ int hash(int r)
    {
        const int low = (r >> 2) & 3;
        if (D == 128) return ((r & 3) << 2) | low;
        if (D == 64) return ((r & 2) << 1) | low;
        return low;
    }
    // offset of the four columns 4q .. 4q+3 of a row
    static __device__ __forceinline__ int quad(int row, int q)
    {
        return row * D + 8 * ((q >> 1) ^ hash(row)) + 4 * (q & 1);
    }
};

// The lane's parts of fragment addresses, elements; column steps are XORed in.
template <int D>
struct Lanes32 {
    int row;    // rows c, unit h
    int row16;  // rows l % 16, unit l / 16: products of 16 x 16 blocks
    int own;    // columns c of a 32-column block, rows 8h ..  (transposing read)
    int upd;    // the same, columns in the order of the state's rows
    __device__ __forceinline__ Lanes32(int l)
    {
        typedef NTile<D> T;
        const int c = l % 32, h = l / 32, a = l % 16, s = (l / 16) % 2, r = 8 * h + (a >> 2);
        row = c * D + 8 * (h ^ T::hash(c));
        row16 = a * D + 8 * ((l / 16) ^ T::hash(a));
        own = r * D + 8 * ((2 * s + ((a >> 1) & 1)) ^ T::hash(r)) + 4 * (a & 1);
        upd = r * D + 8 * ((2 * s + (a & 1)) ^ T::hash(r)) + 4 * ((a >> 1) & 1);
    }
};
// Rows 0 .. 31, contraction step ks (columns 16 ks ..), of a tile of L planes.
template <int D, int L = 1>
__device__ __forceinline__ void load_row_frag(bf8v (&f)[L], const __bf16 *tile, int row, int ks)
{
    const __bf16 *p = tile + (row ^ (16 * ks));
#pragma unroll
    for (int q = 0; q < L; ++q) f[q] = *reinterpret_cast<const bf8v *>(p + q * NTile<D>::PLANE);
}
// Columns 32 jb .. (lane address `col`: own or upd), contracting over chunk rows 16 kr ..  Four rows
// on, the hash differs in its lowest bit.
template <int D>
__device__ __forceinline__ bf8v load_col_frag(const __bf16 *tile, int col, int jb, int kr)
{
    return join(read_tr(tile + (col ^ (32 * jb)) + kr * 16 * D),
                read_tr(tile + (col ^ (32 * jb) ^ 8) + (kr * 16 + 4) * D));
}
// One 16 x 16 block of X_rows . Y_rows^T over D (rows 16 xb, 16 yb): accumulator rows = rows of X.
template <int D>
__device__ __forceinline__ f4v block16(const __bf16 *xt, int xb, const __bf16 *yt, int yb, int row16)
{
    constexpr int NK = D / 32;
    bf8v x[NK], y[NK];
#pragma unroll
    for (int kt = 0; kt < NK; ++kt) {
        x[kt] = *reinterpret_cast<const bf8v *>(xt + xb * 16 * D + (row16 ^ (32 * kt)));
        y[kt] = *reinterpret_cast<const bf8v *>(yt + yb * 16 * D + (row16 ^ (32 * kt)));
    }
    f4v r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < NK; ++kt) r = mfma(x[kt], y[kt], r);
    return r;
}
// A per-row factor of the chunk as planes in row order.
template <int L>
__device__ __forceinline__ void store_row_factor(__bf16 *dst, int r, float x)
{
#pragma unroll
    for (int p = 0; p < L; ++p) {
        const __bf16 v = (__bf16)x;
        dst[p * CR + r] = v;
        x -= (float)v;
    }
}
// Four weights of row `row` of a weight tile (NTile<32>), columns 16 b + 4 g .. + 3, into its planes.
template <int L>
__device__ __forceinline__ void put_weights(__bf16 *tile, int row, int b, int g, f4v x)
{
    __bf16 *dst = tile + NTile<32>::quad(row, 4 * b + g);
    bf4v o[L];
    split4<L>(x, o);
#pragma unroll
    for (int p = 0; p < L; ++p) *reinterpret_cast<bf4v *>(dst + p * NTile<32>::PLANE) = o[p];
}

// ---- products ----------------------------------------------------------------------------------
// The state in LS planes against the rows of tile y, contracting over the state's rows: accumulator
// rows = the wave's columns, columns = chunk rows.
template <int D, int LS>
__device__ __forceinline__ f16v state_rows(const f16v (&st)[D / 32], const __bf16 *y, int row)
{
    constexpr int NK = D / 16, AHEAD = 3;
    f16v hi = zero16(), lo = hi;
    bf8v f[AHEAD + 1][1];
#pragma unroll
    for (int ks = 0; ks < AHEAD && ks < NK; ++ks) load_row_frag<D>(f[ks], y, row, ks);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        const int cur = ks % (AHEAD + 1);
        if (ks + AHEAD < NK) load_row_frag<D>(f[(ks + AHEAD) % (AHEAD + 1)], y, row, ks + AHEAD);
        bf8v x[LS];
        split_frag<LS>(quad_of(st[ks / 2], 2 * (ks % 2)), quad_of(st[ks / 2], 2 * (ks % 2) + 1), x);
#pragma unroll
        for (int p = LS - 1; p >= 1; --p) lo = mfma32(x[p], f[cur][0], lo);
        hi = mfma32(x[0], f[cur][0], hi);
    }
    if constexpr (LS == 1) return hi;
    return hi + lo;
}
// st[k] += A^T B over the chunk rows: A = columns 32 k of tile `at`, B the wave's own columns (b[kr], LB
// planes).  The products meet on an accumulator of their own and are added once, rounded: an instruction
// that adds onto a long sum cuts off what lies below its last bit, and there are two a chunk.  A block's
// addition runs under the next block's instructions: + 4 % of the descending sweep (128 slices of 2048 rows) and
// - 1 % (16 of 131072) against instructions chained onto the state, + 8 % and + 1 % where each block waits for its own.
template <int D, int LB>
__device__ __forceinline__ void update_rows(f16v (&st)[D / 32], const __bf16 *at, int upd, const bf8v (&b)[2][LB])
{
    f16v t[2];
    asm volatile("" : "+v"(upd));  // addresses worked out here, not kept across the chunk loop
#pragma unroll
    for (int k = 0; k <= D / 32; ++k) {
        if (k < D / 32) {
            const bf8v a0 = load_col_frag<D>(at, upd, k, 0), a1 = load_col_frag<D>(at, upd, k, 1);
            t[k % 2] = zero16();
#pragma unroll
            for (int p = LB - 1; p >= 0; --p) t[k % 2] = mfma32(a1, b[1][p], mfma32(a0, b[0][p], t[k % 2]));
        }
        if (k > 0) {
            st[k - 1] += t[(k - 1) % 2];
            // here and not where the next chunk wants it: all blocks' products would stay in registers
            asm volatile("" : "+v"(st[k - 1]));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}
// Own columns x weight tile of LW planes, over the 32 rows of the chunk, smallest products first.
template <int LW>
__device__ __forceinline__ f16v weight_product(const bf8v (&own)[2][1], const __bf16 *wt, int row)
{
    f16v t = zero16();
    bf8v p[2][LW];
    load_row_frag<32, LW>(p[0], wt, row, 0);
    load_row_frag<32, LW>(p[1], wt, row, 1);
#pragma unroll
    for (int s = LW - 1; s >= 0; --s) t = mfma32(own[1][0], p[1][s], mfma32(own[0][0], p[0][s], t));
    return t;
}
// Sum over the chunk rows of the own columns times the row weights in planes `fac` (row order): the
// lane's column c.  Two rows an instruction on the vector ALU, the first plane's sums added up as a tree.
__device__ __forceinline__ float weighted_sum(const bf8v (&own)[2][1], const __bf16 *fac, int h)
{
    float hi[8], lo = 0.f;
#pragma unroll
    for (int p = 2; p >= 0; --p)
#pragma unroll
        for (int kr = 0; kr < 2; ++kr) {
            const bf8v w = *reinterpret_cast<const bf8v *>(fac + p * CR + 16 * kr + 8 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bf2v x = {own[kr][0][2 * e], own[kr][0][2 * e + 1]}, y = {w[2 * e], w[2 * e + 1]};
                if (p > 0) lo = __builtin_amdgcn_fdot2_f32_bf16(x, y, lo, false);
                else hi[4 * kr + e] = __builtin_amdgcn_fdot2_f32_bf16(x, y, 0.f, false);
            }
        }
    return both_halves((((hi[0] + hi[1]) + (hi[2] + hi[3])) + ((hi[4] + hi[5]) + (hi[6] + hi[7]))) + lo);
}
// Own column fragments times the row factors r, split into L planes.
template <int L>
__device__ __forceinline__ void scale_own(bf8v (&o)[2][L], const bf8v (&f)[2][1], const float *r, int h)
{
#pragma unroll
    for (int kr = 0; kr < 2; ++kr) {
        const f4v x = bf4_to_float(__builtin_shufflevector(f[kr][0], f[kr][0], 0, 1, 2, 3)),
                  y = bf4_to_float(__builtin_shufflevector(f[kr][0], f[kr][0], 4, 5, 6, 7));
        const float *rk = r + 16 * kr + 8 * h;
        split_frag<L>(x * *reinterpret_cast<const f4v *>(rk), y * *reinterpret_cast<const f4v *>(rk + 4), o[kr]);
    }
}

// ---- outputs -----------------------------------------------------------------------------------
// Accumulator rows = columns col0 .., columns = the chunk's rows, of which `rows` exist.  bf16: the
// halves of the wave exchange quads so that a lane stores eight columns.
__device__ __forceinline__ int chunk_rows(int n) { return __builtin_amdgcn_readfirstlane(n < 0 ? 0 : (n > CR ? CR : n)); }
__device__ __forceinline__ void store_cols32(__bf16 *base, int ld, int col0, int rows, int l, const f16v &x)
{
    const int n = chunk_rows(rows), c = l % 32, h = l / 32;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, n * ld * 2, kBufferFlags);
    const int off = (c * ld + col0 + 8 * h) * 2;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const u2v a = __builtin_bit_cast(u2v, to_bf4(quad_of(x, 2 * s))),
                  b = __builtin_bit_cast(u2v, to_bf4(quad_of(x, 2 * s + 1)));
        const auto p = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false),
                   q = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
        __builtin_amdgcn_raw_buffer_store_b128(u4v{p[0], q[0], p[1], q[1]}, rsrc, off + 32 * s, 0, 0);
    }
}
// The same layout, fp32.
__device__ __forceinline__ void store_cols32(float *base, int ld, int col0, int rows, int l, const f16v &x)
{
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, chunk_rows(rows) * ld * 4, kBufferFlags);
    const int off = (l % 32 * ld + col0 + 4 * (l / 32)) * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, quad_of(x, q)), rsrc, off + 32 * q, 0, 0);
}
// What they hold in fp32, in the same layout.
__device__ __forceinline__ f16v load_cols32(const float *base, int ld, int col0, int rows, int l)
{
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, chunk_rows(rows) * ld * 4, kBufferFlags);
    const int off = (l % 32 * ld + col0 + 4 * (l / 32)) * 4;
    f16v x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f4v o = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 32 * q, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * q + e] = o[e];
    }
    return x;
}
// One chunk of a gradient, 32 columns.  LD > D builds it up over two launches, the first of which leaves
// its share in `part` (fp32, rows of D); the second (`add`) has added it to x.
template <int D, int LD>
__device__ __forceinline__ void store_grad32(__bf16 *out, float *part, bool add, int col0, int rows, int l,
                                             const f16v &x)
{
    if constexpr (LD <= D) store_cols32(out, LD, col0, rows, l, x);
    else if (!add) store_cols32(part, D, col0, rows, l, x);
    else store_cols32(out, LD, col0, rows, l, x);
}

}  // namespace
}  // namespace la
