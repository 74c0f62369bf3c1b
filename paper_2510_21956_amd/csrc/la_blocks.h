// Pieces shared by the matrix-core kernel files: output stores, lane reductions, the backward
// of the row normalisation on register blocks.
#pragma once

#include <type_traits>

#include "la_common.h"

namespace la {
namespace {

typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
// Fourth word of a raw buffer descriptor on gfx9-family parts: 32-bit data format, no
// swizzle, out-of-range reads return zero.
constexpr int kBufferFlags = 0x00020000;
typedef unsigned int u2v __attribute__((ext_vector_type(2)));

// Four floats to four bf16 (round to nearest even) as two packed conversions: written on
// pairs because only the two-element form is turned into one instruction per pair.
__device__ __forceinline__ bf4v to_bf4(f4v x)
{
    const bf2v p = __builtin_convertvector((f2v{x[0], x[1]}), bf2v);
    const bf2v q = __builtin_convertvector((f2v{x[2], x[3]}), bf2v);
    return __builtin_shufflevector(p, q, 0, 1, 2, 3);
}
__device__ __forceinline__ f4v bf4_to_float(bf4v x) { return __builtin_convertvector(x, f4v); }

// x[c0 + r] of a per-row float array of N entries (c0 < N, r < 64); 0 beyond the end.
__device__ __forceinline__ float load_row_float(const float *x, long c0, int N, int r)
{
    const long rows = (N - c0 < 64) ? N - c0 : 64;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(x + c0), 0, (int)(rows * sizeof(float)), kBufferFlags);
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, 4 * r, 0, 0));
}

// Sum over each aligned group of WIDTH consecutive lanes, result in every lane of the
// group.  Up to 16 lanes this is data-parallel-primitive moves inside the vector ALU
// (swap neighbours, swap pairs, mirror the half row, mirror the row: after each step all
// lanes that already shared a partial sum still do); beyond that, lane shuffles.
template <int WIDTH>
__device__ __forceinline__ float reduce_adjacent(float s)
{
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                               0xf, 0xf, true));
    };
    if constexpr (WIDTH >= 2) s += dpp(s, std::integral_constant<int, 0xB1>{});   // quad_perm 1,0,3,2
    if constexpr (WIDTH >= 4) s += dpp(s, std::integral_constant<int, 0x4E>{});   // quad_perm 2,3,0,1
    if constexpr (WIDTH >= 8) s += dpp(s, std::integral_constant<int, 0x141>{});  // row_half_mirror
    if constexpr (WIDTH >= 16) s += dpp(s, std::integral_constant<int, 0x140>{}); // row_mirror
    if constexpr (WIDTH >= 32) s += __shfl_xor(s, 16);
    if constexpr (WIDTH >= 64) s += __shfl_xor(s, 32);
    return s;
}

// Sum over the four lane groups of a wave (lanes l, l^16, l^32, l^48).
__device__ __forceinline__ float reduce_lane_groups(float x)
{
    x += __shfl_xor(x, 32);
    x += __shfl_xor(x, 16);
    return x;
}

// 16 x 16 accumulator block: lane (c, g) of the wave, c = lane % 16 and g = lane / 16, holds rows
// 4g .. 4g+3 of column c.
struct Blk {
    f4v v;
    __device__ __forceinline__ void zero() { v = f4v{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ float get(int i) const { return v[i]; }
    __device__ __forceinline__ void set(int i, float x) { v[i] = x; }
};

// Where a branch stays one: made a selection, what a launch without `add` never loads would be waited for all
// the same.
__device__ __forceinline__ void keep_branch() { asm volatile(""); }

// Rows of a 16-row block that exist.  The clamp is a vector instruction whatever its operand; its
// result is named uniform, or every store whose descriptor it goes into becomes a loop over
// the lanes' descriptors.
__device__ __forceinline__ int valid_rows(int n)
{
    return __builtin_amdgcn_readfirstlane(n < 0 ? 0 : (n > 16 ? 16 : n));
}

// Store the wave's 16 x 16 output block.  On entry lane (c, g) holds columns col0 + 4g..4g+3
// of block row c.  Neighbouring lanes would write to different rows, which the memory
// pipeline cannot merge, so the values are first exchanged between lanes (no memory
// involved): afterwards lane l holds row l / 4, column quad l % 4, and four neighbouring
// lanes write one contiguous run of a row.  The block is addressed through a buffer
// descriptor that covers its first `rows_valid` rows (at most 16, possibly none): stores
// to rows beyond them are dropped by the address check, without a branch, and the lane's
// address is one 32-bit offset that does not change from block to block.
// With `add`, old (load_block) is added first, times old_scale[row] if given: the calls that work on a block of
// columns of wider rows build their results up over several launches.
template <typename T>
__device__ __forceinline__ void store_block(T *base, int ld, int col0, int rows_valid, int l,
                                            float x0, float x1, float x2, float x3, bool add = false,
                                            f4v old = f4v{}, const float *old_scale = nullptr)
{
    const int src = 16 * (l % 4) + l / 4;  // lane that holds (row l/4, column quad l%4)
    const int row = l / 4, cq = l % 4;
    const int nrows = valid_rows(rows_valid);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        base, 0, nrows * ld * (int)sizeof(T), kBufferFlags);
    const int off = (row * ld + col0 + 4 * cq) * (int)sizeof(T);
    if (sizeof(T) == 4 || add) {
        f4v y = {__shfl(x0, src), __shfl(x1, src), __shfl(x2, src), __shfl(x3, src)};
        if (add) {
            keep_branch();
            y += (old_scale ? old_scale[row] : 1.f) * old;
        }
        if constexpr (sizeof(T) == 4) {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, y), rsrc, off, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, to_bf4(y)), rsrc, off, 0, 0);
        }
    } else {
        bf4v p = to_bf4(f4v{x0, x1, x2, x3});
        u2v u = *reinterpret_cast<u2v *>(&p);
        const u2v v = {(unsigned)__shfl((int)u[0], src), (unsigned)__shfl((int)u[1], src)};
        __builtin_amdgcn_raw_buffer_store_b64(v, rsrc, off, 0, 0);
    }
}
// What an fp32 block holds, in the layout in which store_block adds it.  Asked for a phase ahead, before the next
// chunk's rows (loads are waited for in order): read where it is added, every block of a launch that adds waited for
// memory.  Head size 256, 64 slices of 4096 rows, a forward launch that adds 287 -> 266 us (fp32), 163 -> 136 (bf16), a
// backward launch that adds to all gradients 572 -> 520 and 291 -> 275; a step 3177 -> 3062 and 1580 -> 1458, without
// the mask 2133 -> 1980 and 1246 -> 1166.  Launches that do not add are kernels of their own: with both in one, they
// took up to 3 % longer.
__device__ __forceinline__ f4v load_block(const float *base, int ld, int col0, int rows_valid, int l)
{
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(base), 0, valid_rows(rows_valid) * ld * 4, kBufferFlags);
    return __builtin_bit_cast(
        f4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (l / 4 * ld + col0 + 4 * (l % 4)) * 4, 0, 0));
}

// One 16-row block of a bf16 gradient.  With LD > D (a block of D columns of rows LD wide) the
// gradient is the sum of two launches: the first keeps its share in `part` (fp32, rows of D: early
// rows of a masked pass are small differences of large shares) and the second (`add`) adds it and
// rounds once.  (fp32 gradients are stored by columns and added up in place.)
template <int D, int LD>
__device__ __forceinline__ void store_grad_block(__bf16 *out, float *part, bool add, int col0,
                                                 int rows_valid, int l, f4v x, f4v old)
{
    if constexpr (LD <= D)
        store_block<__bf16>(out, LD, col0, rows_valid, l, x[0], x[1], x[2], x[3]);
    else if (!add)
        store_block<float>(part, D, col0, rows_valid, l, x[0], x[1], x[2], x[3]);
    else
        store_block<__bf16>(out, LD, col0, rows_valid, l, x[0], x[1], x[2], x[3], true, old);
}

// Backward of the row normalisation (Sec. 3.3) on gradient blocks still in registers:
//   dx = (dxhat - xhat (xhat . dxhat)) / |x|     for every row of the chunk.
// Lane (c, g) holds dxhat[row 16 m + c][columns 16 w + 4 g .. + 3] of NBK row blocks in x[m] and
// the same elements of xhat in xh[m].  The row's dot product runs over all D columns, i.e.
// over the lane groups of a wave and over the waves: per-wave shares meet in dots[NW][C]
// (LDS), which costs one workgroup barrier.  Every thread of the workgroup must call this.
template <int NW, int C, int NBK>
__device__ __forceinline__ void project_blocks(float (&x)[NBK][4], const float (&xh)[NBK][4],
                                               float *dots, const float *inv, int w, int c, int g)
{
#pragma unroll
    for (int m = 0; m < NBK; ++m) {
        float s = (x[m][0] * xh[m][0] + x[m][1] * xh[m][1]) + (x[m][2] * xh[m][2] + x[m][3] * xh[m][3]);
        s = reduce_lane_groups(s);
        if (g == 0) dots[w * C + m * 16 + c] = s;
    }
    block_sync();
#pragma unroll
    for (int m = 0; m < NBK; ++m) {
        float dot = 0.f;
#pragma unroll
        for (int v = 0; v < NW; ++v) dot += dots[v * C + m * 16 + c];
        const float iv = inv[m * 16 + c];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[m][e] = (x[m][e] - xh[m][e] * dot) * iv;
    }
}

// Backward slot: [S^T (D*D) | z (D) | R (D*D) | u (D) | w (D)], all unscaled sums: S = sum k v^T,
// z = sum k, R = sum q OmegaHat^T, u = sum delta q, w = sum OmegaHat (Eq. endd without the
// factors a, b).  Readers that want R transposed take four consecutive columns of a row of it.
template <int D>
struct BwdSlot {
    static constexpr int ST = 0, Z = D * D, R = D * D + D, U = 2 * D * D + D, W = 2 * D * D + 2 * D,
                         END = 2 * D * D + 3 * D;
};

inline la_status launch_status()
{
    return hipGetLastError() == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

}  // namespace
}  // namespace la
