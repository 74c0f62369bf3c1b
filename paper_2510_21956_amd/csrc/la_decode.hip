// Incremental (decode) step: the recurrence of App. B.1 (Table 3, row 2) for the kernel
// a + b x, with the running sums of Eq. xy carried across calls in a caller-owned state.
//
// State of one (batch, head) slice, float32: [S (D*D, S[r][j] = sum k_r v_j) | z (D) | p (D) |
// count (1)], padded to a multiple of 64 floats.  A call appends T rows: each is added to the
// sums, then read out, o_t = (a p + b S^T q_t) / g_t, g_t = a count + b q_t . z (Eq. fglast, div).
//
// One workgroup per slice keeps the whole state in registers for the T rows of the call (no
// other workgroup touches that slice's state, so updating it in place is race-free).  The step
// is bound by reading and writing the state once per call, 8 D^2 bytes per slice, and with one
// row by the latency of doing so: as many lanes as the state has 16-byte units (up to 1024
// threads), each with a few of them, have the whole state in flight at once.  One row, 128
// slices, D = 128: 4.6 us (3.6 TB/s of state), 5.7 with 256 threads of single floats; 64 slices,
// D = 256: 8.6 us, 30.8 before.
#include <type_traits>

#include "la_common.h"

namespace la {
namespace {

template <int D>
struct DC {
    static constexpr int LR = D / 4;                                  // lanes that share a row
    static constexpr int NT = D * D / 16 < 64 ? 64 : (D * D / 16 > 1024 ? 1024 : D * D / 16);
    static constexpr int RG = NT / LR;                                // row groups
    static constexpr int RPT = D / RG;                                // consecutive rows per thread
    static constexpr int NW = NT / 64;
};

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m);
    return x;
}

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f4 load4(const float *p) { return *reinterpret_cast<const f4 *>(p); }
__device__ __forceinline__ f4 load4(const bf16_t *p)
{
    const u2 u = *reinterpret_cast<const u2 *>(p);
    return f4{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u),
              __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xffff0000u)};
}

// Thread t holds columns 4 (t % LR) .. + 3 of rows RPT (t / LR) .. + RPT - 1 of S; thread t < D
// also holds z[t] and p[t].
template <typename T, int D>
__global__ __launch_bounds__((DC<D>::NT)) void k_decode(const T *__restrict__ Q,
                                                       const T *__restrict__ K,
                                                       const T *__restrict__ V, T *__restrict__ O,
                                                       float *__restrict__ G,
                                                       float *__restrict__ state, int Tn,
                                                       size_t state_floats, float a, float b)
{
    constexpr int LR = DC<D>::LR, RPT = DC<D>::RPT, NW = DC<D>::NW, NT = DC<D>::NT;
    constexpr int NO = (D + NT - 1) / NT;  // output columns per thread of the final sums
    // two buffers: a row's sums are read while the next row's are written
    __shared__ __align__(16) float part[2][NW][D];
    __shared__ float partz[2][NW];
    const int bh = blockIdx.x, t = threadIdx.x, w = t / 64, j = 4 * (t % LR), r0 = RPT * (t / LR);
    float *st = state + (size_t)bh * state_floats;
    f4 S[RPT];
    float z[NO], p[NO];
#pragma unroll
    for (int i = 0; i < RPT; ++i) S[i] = load4(st + (size_t)(r0 + i) * D + j);
#pragma unroll
    for (int m = 0; m < NO; ++m) {
        const int col = t + m * NT;
        z[m] = col < D ? st[D * D + col] : 0.f;
        p[m] = col < D ? st[D * D + D + col] : 0.f;
    }
    float cnt = st[D * D + 2 * D];
    const size_t base = (size_t)bh * Tn * D;
    for (int tok = 0; tok < Tn; ++tok) {
        const T *q = Q + base + (size_t)tok * D, *k = K + base + (size_t)tok * D,
                *v = V + base + (size_t)tok * D;
        const int buf = tok & 1;
        const f4 v4 = load4(v + j);
        f4 f = {0.f, 0.f, 0.f, 0.f};
        float qz = 0.f;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {  // the new row enters the sums before it is read out
            const float ki = load_elem(k, r0 + i), qi = load_elem(q, r0 + i);
            S[i] += ki * v4;
            f += qi * S[i];
            // D = 256: 64 registers of state, so the loads of q and k stay a few rows ahead
            if (RPT > 8 && i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < NO; ++m) {
            const int col = t + m * NT;
            if (col < D) {
                z[m] += load_elem(k, col);
                p[m] += load_elem(v, col);
                qz += load_elem(q, col) * z[m];
            }
        }
        qz = wave_sum(qz);
#pragma unroll
        for (int m = LR; m < 64; m <<= 1) {  // the row groups of this wave
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] += __shfl_xor(f[e], m);
        }
        if (t % 64 < LR) *reinterpret_cast<f4 *>(&part[buf][w][j]) = f;
        if (t % 64 == 0) partz[buf][w] = qz;
        cnt += 1.f;
        block_sync();
#pragma unroll
        for (int m = 0; m < NO; ++m) {
            const int col = t + m * NT;
            if (col < D) {
                float lin = 0.f, qs = 0.f;
#pragma unroll 4
                for (int x = 0; x < NW; ++x) {
                    lin += part[buf][x][col];
                    qs += partz[buf][x];
                }
                const float gv = a * cnt + b * qs;  // g = a count + b q . z
                store_elem(O, base + (size_t)tok * D + col, (a * p[m] + b * lin) / gv);
                if (col == 0 && G) G[(size_t)bh * Tn + tok] = gv;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) *reinterpret_cast<f4 *>(st + (size_t)(r0 + i) * D + j) = S[i];
#pragma unroll
    for (int m = 0; m < NO; ++m) {
        const int col = t + m * NT;
        if (col < D) {
            st[D * D + col] = z[m];
            st[D * D + D + col] = p[m];
        }
    }
    block_sync();  // every thread has read the count
    if (t == 0) st[D * D + 2 * D] = cnt;
}

// Sum of W floats at e over the slots of a slice, in ascending order; sixteen loads in flight.
template <int W>
__device__ __forceinline__ auto sum_slots(const float *src, int e, int nseg, size_t slot_floats)
{
    typedef typename std::conditional<W == 4, f4, float>::type T;
    constexpr int BATCH = 16;
    T run{};
    for (int s0 = 0; s0 < nseg; s0 += BATCH) {
        T x[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            x[i] = s0 + i < nseg ? *reinterpret_cast<const T *>(src + (size_t)(s0 + i) * slot_floats + e) : T{};
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            if (s0 + i < nseg) run = s0 + i == 0 ? x[i] : run + x[i];
    }
    return run;
}
template <typename T>
__device__ __forceinline__ void put(float *dst, T x, int accumulate)
{
    T *d = reinterpret_cast<T *>(dst);
    *d = accumulate ? *d + x : x;
}

// Few slots a slice: this is a copy, bound by memory, 16 bytes a thread (W = 4; 1024 slices of 20 rows, D = 128, bf16,
// with the sums kernel: 37 us; 92 with 4 bytes).  Many, which only few slices have: the round trips along the slots
// bound it, so 8 groups of 32 lanes (W = 1) read a run of them each and add up through LDS.  16 bytes and runs, us, with
// the sums kernel, fp32, one slice: D = 32, 33 slots 10.6 and 10.8, 96 12.2 and 10.8, 300 27.7 and 10.8; D = 128, 33 11.5 and
// 10.9, 300 38.5 and 21.7; six slices at D = 128, 33 16.1 and 14.9, 160 42.5 and 39.1.  One thread a float and one slot
// after another, 700 slots of one slice, D = 32 38.5, D = 128 53.2; runs 12.1 and 31.3 (16 of them 10.7 and 31.8, but
// 16.3 for the 33 slots of six slices).
constexpr int kManySlots = 32, kRuns = 8;
template <int W>
constexpr int kStateThreads = W == 1 ? 32 * kRuns : 256;
// Floats that a workgroup makes, and the first one of this thread.
template <int W>
constexpr int kStateFloats = W == 1 ? 32 : 4 * 256;
template <int W>
__device__ __forceinline__ int state_float()
{
    return blockIdx.y * kStateFloats<W> + (W == 1 ? threadIdx.x % 32 : W * threadIdx.x);
}
// The sum at e over all slots where `there`; called by every thread.  W = 1: in the first 32 threads.
template <int W>
__device__ __forceinline__ auto slot_total(const float *src, int e, bool there, int nseg, size_t slot_floats)
{
    if constexpr (W == 4) {
        return there ? sum_slots<4>(src, e, nseg, slot_floats) : f4{};
    } else {
        __shared__ float sums[kRuns][32];
        const int run = threadIdx.x / 32, n = (nseg + kRuns - 1) / kRuns, first = min(run * n, nseg);
        sums[run][threadIdx.x % 32] =
            there ? sum_slots<1>(src + (size_t)first * slot_floats, e, min(n, nseg - first), slot_floats) : 0.f;
        block_sync();
        float x = 0.f;
        for (int r = 0; r < kRuns && run == 0; ++r) x += sums[r][threadIdx.x];
        return x;
    }
}

// state (+)= the sums of [S | z | p] over the slots of every slice, count (+)= N.
template <int W>
__global__ __launch_bounds__(kStateThreads<W>) void k_state_from_totals(const float *__restrict__ ws,
                                                           float *__restrict__ state, int D,
                                                           int nseg, size_t slot_floats,
                                                           size_t state_floats, int N,
                                                           int accumulate)
{
    const int bh = blockIdx.x, len = D * D + 2 * D, e = state_float<W>();
    const float *src = ws + (size_t)bh * nseg * slot_floats;
    float *dst = state + (size_t)bh * state_floats;
    const auto x = slot_total<W>(src, e, e < len, nseg, slot_floats);
    if (W == 1 && threadIdx.x >= 32) return;
    if (e < len) put(dst + e, x, accumulate);
    else if (e == len) put(dst + e, (float)N, accumulate);
}

// The same for D = 256 from the slots of the block problem (k block i, v block j) at D = 128:
// S block (i, j); z block i (taken when j = 0); p block j (when i = 0); the count once.
template <int W>
__global__ __launch_bounds__(kStateThreads<W>) void k_state_block_from_totals(const float *__restrict__ ws,
                                                                 float *__restrict__ state,
                                                                 int nseg, size_t slot_floats,
                                                                 size_t state_floats, int bi,
                                                                 int bj, int N, int accumulate)
{
    constexpr int H = 128, D = 256;
    const int bh = blockIdx.x, len = H * H + 2 * H, e = state_float<W>();
    const float *src = ws + (size_t)bh * nseg * slot_floats;
    float *dst = state + (size_t)bh * state_floats;
    int to = -1;  // nothing to write
    if (e < H * H) to = (bi * H + e / H) * D + bj * H + e % H;
    else if (e < H * H + H) to = bj == 0 ? D * D + bi * H + (e - H * H) : -1;
    else if (e < len) to = bi == 0 ? D * D + D + bj * H + (e - H * H - H) : -1;
    const auto x = slot_total<W>(src, e, to >= 0, nseg, slot_floats);
    if (W == 1 && threadIdx.x >= 32) return;
    if (to >= 0) put(dst + to, x, accumulate);
    else if (e == len && bi == 0 && bj == 0) put(dst + D * D + 2 * D, (float)N, accumulate);
}

// Stage 1 of sum(X * Y): workgroup w sums a fixed contiguous share into partials[w].
constexpr int kDotBlocks = 1024;
template <typename T>
__global__ __launch_bounds__(256) void k_dot_partial(const T *__restrict__ X,
                                                     const T *__restrict__ Y, size_t n,
                                                     float *__restrict__ partials)
{
    __shared__ float red[4];
    const size_t per = (n + gridDim.x - 1) / gridDim.x;
    const size_t lo = (size_t)blockIdx.x * per, hi = lo + per < n ? lo + per : n;
    float s = 0.f;
    for (size_t e = lo + threadIdx.x; e < hi; e += 256) s += load_elem(X, e) * load_elem(Y, e);
    s = wave_sum(s);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = s;
    block_sync();
    if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}
// Stage 2: one workgroup adds the partials in a fixed order and writes the two scaled results.
__global__ __launch_bounds__(256) void k_dot_final(const float *__restrict__ partials, int np,
                                                   float scale0, float scale1,
                                                   float *__restrict__ out)
{
    __shared__ float red[4];
    float s = 0.f;
    for (int e = threadIdx.x; e < np; e += 256) s += partials[e];
    s = wave_sum(s);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = s;
    block_sync();
    if (threadIdx.x == 0) {
        const float tot = (red[0] + red[1]) + (red[2] + red[3]);
        out[0] = scale0 * tot;
        out[1] = scale1 * tot;
    }
}

// Backward of x -> x / ||x|| for one row per 16 lanes (D <= 256: up to 16 elements a lane).
template <typename T>
__global__ __launch_bounds__(256) void k_project_rows(const T *__restrict__ X, T *__restrict__ dX,
                                                      size_t rows, int D)
{
    const size_t row = (size_t)blockIdx.x * 16 + threadIdx.x / 16;
    const int l = threadIdx.x % 16;
    if (row >= rows) return;  // whole 16-lane groups leave together
    const T *x = X + row * D;
    T *dx = dX + row * D;
    float xv[16], dv[16], ss = 0.f, dot = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int m = l + 16 * i;
        xv[i] = m < D ? load_elem(x, m) : 0.f;
        dv[i] = m < D ? load_elem(dx, m) : 0.f;
        ss += xv[i] * xv[i];
        dot += xv[i] * dv[i];
    }
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) {
        ss += __shfl_xor(ss, m);
        dot += __shfl_xor(dot, m);
    }
    const float inv = ss > 0.f ? 1.f / sqrtf(ss) : 0.f;
    const float proj = dot * inv * inv;  // (xhat . dxhat) / ||x||
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int m = l + 16 * i;
        if (m < D) store_elem(dx, m, (dv[i] - xv[i] * proj) * inv);
    }
}

template <typename T>
la_status decode_by_d(const void *Q, const void *K, const void *V, void *O, float *G, float *state,
                      int BH, int Tn, int D, size_t sf, float a, float b, hipStream_t st)
{
    const T *q = (const T *)Q, *k = (const T *)K, *v = (const T *)V;
    T *o = (T *)O;
#define LA_DECODE_CASE(DD)                                                                       \
    case DD:                                                                                     \
        k_decode<T, DD><<<dim3(BH), dim3(DC<DD>::NT), 0, st>>>(q, k, v, o, G, state, Tn, sf, a, b); \
        break;
    switch (D) {
        LA_DECODE_CASE(16)
        LA_DECODE_CASE(32)
        LA_DECODE_CASE(64)
        LA_DECODE_CASE(128)
        LA_DECODE_CASE(256)
        default: return LA_ERR_UNSUPPORTED;
    }
#undef LA_DECODE_CASE
    return hipGetLastError() == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

}  // namespace

int reduce_dot_partials() { return kDotBlocks; }

la_status reduce_dot(const void *X, const void *Y, size_t n, la_dtype dt, float scale0, float scale1,
                     float *partials, float *out, hipStream_t st)
{
    if (dt == LA_F32)
        k_dot_partial<float><<<dim3(kDotBlocks), dim3(256), 0, st>>>((const float *)X,
                                                                     (const float *)Y, n, partials);
    else
        k_dot_partial<bf16_t><<<dim3(kDotBlocks), dim3(256), 0, st>>>((const bf16_t *)X,
                                                                      (const bf16_t *)Y, n, partials);
    k_dot_final<<<dim3(1), dim3(256), 0, st>>>(partials, kDotBlocks, scale0, scale1, out);
    return hipGetLastError() == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

la_status project_rows(const void *X, void *dX, size_t rows, int D, la_dtype dt, hipStream_t st)
{
    const dim3 grid((unsigned)((rows + 15) / 16)), block(256);
    if (dt == LA_F32)
        k_project_rows<float><<<grid, block, 0, st>>>((const float *)X, (float *)dX, rows, D);
    else
        k_project_rows<bf16_t><<<grid, block, 0, st>>>((const bf16_t *)X, (bf16_t *)dX, rows, D);
    return hipGetLastError() == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

size_t decode_state_floats(int D) { return ((size_t)D * D + 2 * (size_t)D + 1 + 63) / 64 * 64; }

la_status decode_step(const void *Q, const void *K, const void *V, void *O, float *G, float *state,
                      int BH, int Tn, int D, float a, float b, la_dtype dt, hipStream_t st)
{
    const size_t sf = decode_state_floats(D);
    if (dt == LA_F32) return decode_by_d<float>(Q, K, V, O, G, state, BH, Tn, D, sf, a, b, st);
    return decode_by_d<bf16_t>(Q, K, V, O, G, state, BH, Tn, D, sf, a, b, st);
}

// Workgroups for len floats and the count.
template <int W>
static int state_blocks(int len) { return (len + 1 + kStateFloats<W> - 1) / kStateFloats<W>; }

la_status state_from_totals(const float *ws, float *state, int BH, int D, int nseg,
                            size_t slot_floats, int N, int accumulate, hipStream_t st)
{
    const int len = D * D + 2 * D;
    const bool many = nseg > kManySlots;
    (many ? k_state_from_totals<1> : k_state_from_totals<4>)<<<
        dim3(BH, many ? state_blocks<1>(len) : state_blocks<4>(len)),
        dim3(many ? kStateThreads<1> : kStateThreads<4>), 0, st>>>(
        ws, state, D, nseg, slot_floats, decode_state_floats(D), N, accumulate);
    return hipGetLastError() == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

la_status state_block_from_totals(const float *ws, float *state, int BH, int nseg,
                                  size_t slot_floats, int bi, int bj, int N, int accumulate,
                                  hipStream_t st)
{
    const int len = 128 * 128 + 2 * 128;
    const bool many = nseg > kManySlots;
    (many ? k_state_block_from_totals<1> : k_state_block_from_totals<4>)<<<
        dim3(BH, many ? state_blocks<1>(len) : state_blocks<4>(len)),
        dim3(many ? kStateThreads<1> : kStateThreads<4>), 0, st>>>(
        ws, state, nseg, slot_floats, decode_state_floats(256), bi, bj, N, accumulate);
    return hipGetLastError() == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

}  // namespace la
