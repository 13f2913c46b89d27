// Shared inner loop of the vectorised SpMM kernels: a group of G lanes
// holds a batch of (column, value) pairs, one per lane, and gathers the
// corresponding X rows B at a time, each lane loading NQ float4 at columns
// c0 + 4*G*q (so one load instruction reads G*16 contiguous bytes of a row).
// Any width of at least 4 columns and any 4-byte aligned operands are taken
// this way: quads need no 16-byte alignment, and a width that is no multiple
// of 4 ends in a quad that overlaps the one before it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

namespace gs {

// Column words with a reference class: bits 27..30 hold the class of the
// column (bit length of its entry count, at most 15), bits 0..26 the column.
constexpr int kColClassShift = 27;
constexpr int kColMask = (1 << kColClassShift) - 1;

// Four floats at any 4-byte aligned address: one 16-byte load or store (the
// memory pipeline needs dword alignment only; an access that straddles a
// 128-byte line costs that line's second request).
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double d4 __attribute__((ext_vector_type(4), aligned(8)));

// Accumulator quads: fp32, or fp64 where the products are summed exactly.
template <class A> struct Quad;
template <> struct Quad<float> {
    typedef f4u type;
};
template <> struct Quad<double> {
    typedef d4 type;
};

// Lane t's value of entry j0 + J of the group's batch.  A group of a whole wave
// holds 64 entries and reads one into a scalar register; groups of 16 and 32
// lanes hold the same batch of 16 entries in every DPP row of 16 lanes, so one
// row_newbcast serves them; smaller groups hold a batch of G entries (j0 is 0
// for all but whole waves).  No LDS round trip, unlike a shuffle.
template <int J, int G> __device__ __forceinline__ int bcast_entry(int v, int j0 = 0)
{
    if constexpr (G == 64) {
        return __builtin_amdgcn_readlane(v, j0 + J);
    } else if constexpr (G == 4) {
        return __builtin_amdgcn_update_dpp(0, v, J * 0x55, 0xf, 0xf, true);  // quad_perm: lane J of each quad
    } else if constexpr (G == 8) {
        const int lo = __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xf, 0xf, true);
        return __builtin_amdgcn_update_dpp(lo, v, 0x150 + 8 + J, 0xf, 0xc, true);  // banks 2, 3: the upper group
    } else {
        return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xf, 0xf, true);  // row_newbcast:J
    }
}

// Entries per register of a group of G lanes, and per batch of NB registers
// (NB = 2 for groups of 32 lanes only).
template <int G> constexpr int kEntryReg = G == 64 ? 64 : G < 16 ? G : 16;
template <int G, int NB> constexpr int kEntryBatch = NB * kEntryReg<G>;

// Column quads of a lane: quad q starts at column c0 + 4 G q, the last one
// of a width that is no multiple of 4 moved back to end at column F (the
// lanes that overlap then compute and store the same sums twice), quads past
// the width folded onto it and not stored.
template <int NQ, int G, bool FULL> struct Quads {
    static constexpr bool kFull = FULL;
    int c0;               // (F is at most 2^24)
    int col[FULL ? 1 : NQ];
    bool live[FULL ? 1 : NQ];
    __device__ __forceinline__ Quads(int64_t cbase, int lane, int64_t F)
    {
        c0 = (int)cbase + 4 * lane;
        if constexpr (!FULL) {
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                const int c = c0 + 4 * G * q;
                live[q] = c < (int)F;
                col[q] = c < (int)F - 4 ? c : (int)F - 4;
            }
        }
    }
    // column of quad q = base(q) + step(q), step a compile-time constant
    __device__ __forceinline__ int base(int q) const { return FULL ? c0 : col[FULL ? 0 : q]; }
    __device__ __forceinline__ int step(int q) const { return FULL ? 4 * G * q : 0; }
    __device__ __forceinline__ bool ok(int q) const { return FULL || live[FULL ? 0 : q]; }
};

// How the X row of an entry is addressed: the column becomes its row's offset
// in the lane that loads the entry, so that only offsets are broadcast.
//   kOff32: byte offset in 32 bits (X spans less than 4 GiB)
//   kOff64: byte offset in 64 bits
enum { kOff32 = 0, kOff64 = 1 };

template <int OFF> struct RowRef {
    uint32_t lo = 0, hi = 0;
    __device__ __forceinline__ void set(int col, int64_t ldx)
    {
        if constexpr (OFF == kOff32) {
            lo = (uint32_t)col * (uint32_t)(ldx * 4);
        } else {
            const uint64_t o = (uint64_t)(uint32_t)col * (uint64_t)ldx * 4u;
            lo = (uint32_t)o;
            hi = (uint32_t)(o >> 32);
        }
    }
};

// Address of quad q of the lane in the X row at (hi, lo).
template <int OFF, class Q>
__device__ __forceinline__ const float *x_at(const float *X, uint32_t lo, uint32_t hi, const Q &cols, int q)
{
    const char *b = reinterpret_cast<const char *>(X);
    if constexpr (OFF == kOff32)
        return reinterpret_cast<const float *>(b + (uint64_t)(lo + 4u * (uint32_t)cols.base(q))) + cols.step(q);
    else
        return reinterpret_cast<const float *>(b + (((uint64_t)hi << 32) | lo)) + (int64_t)cols.base(q) + cols.step(q);
}

// Entries J0 .. J0+B-1 of the group's batch (ref, v: one entry per lane and
// register): B X rows requested back to back, then B multiply-adds into acc:
// one chain (NA = 1), or a chain for every four entries, which joins two sums in
// turn (NA = 2; ODD: the first of them the second sum).  MASKED: entries past the
// t-th gather nothing (a dead gather costs as much as a live one) and add
// -0 * 0 = -0, which leaves every sum as it is.  CLS: entries whose lane set
// `cold` are gathered non-temporally.
template <int J0, int B, int NQ, int G, bool MASKED, int OFF, bool CLS, int NA, bool ODD, class Q, class A>
__device__ __forceinline__ void gather_step(const RowRef<OFF> *ref, const float *v, const int *cold, int t,
                                            const float *X, const Q &cols, A *acc, int j0 = 0)
{
    f4u x[B][NQ];
    float vv[B];
    uint32_t lo[B], hi[B];
    int c[B];
    [&]<int... U>(std::integer_sequence<int, U...>) {
        (
            [&] {
                constexpr int E = (J0 + U) % kEntryReg<G>, R = (J0 + U) / kEntryReg<G>;
                lo[U] = (uint32_t)bcast_entry<E, G>((int)ref[R].lo, j0);
                hi[U] = 0;
                if constexpr (OFF == kOff64) hi[U] = (uint32_t)bcast_entry<E, G>((int)ref[R].hi, j0);
                vv[U] = __int_as_float(bcast_entry<E, G>(__float_as_int(v[R]), j0));
                c[U] = 0;
                if constexpr (CLS) c[U] = bcast_entry<E, G>(cold[R], j0);
            }(),
            ...);
    }(std::make_integer_sequence<int, B>{});
#pragma unroll
    for (int u = 0; u < B; u++)
#pragma unroll
        for (int q = 0; q < NQ; q++)
            x[u][q] = MASKED ? f4u{0.f, 0.f, 0.f, 0.f} : __builtin_nondeterministic_value(x[u][q]);
    // (lanes past the width load nothing: dead lanes cost data return, 12% at
    // F = 156)
    auto load = [&](int q) {
#pragma unroll
        for (int u = 0; u < B; u++) {
            if (MASKED && j0 + J0 + u >= t) continue;
            const f4u *p = reinterpret_cast<const f4u *>(x_at<OFF>(X, lo[u], hi[u], cols, q));
            if (CLS && c[u]) {
                // (the empty asm statements keep the compiler from merging the two branches' loads
                // into one that has lost the non-temporal hint)
                asm volatile("");
                x[u][q] = __builtin_nontemporal_load(p);
                asm volatile("");
            } else {
                x[u][q] = *p;
            }
        }
    };
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        if constexpr (Q::kFull)
            load(q);
        else if (cols.ok(q))
            load(q);
    }
    if constexpr (NA == 1) {
#pragma unroll
        for (int u = 0; u < B; u++)
#pragma unroll
            for (int q = 0; q < NQ; q++)
#pragma unroll
                for (int i = 0; i < 4; i++)
                    acc[4 * q + i] = __builtin_elementwise_fma((A)vv[u], (A)x[u][q][i], acc[4 * q + i]);
    } else {
        static_assert(NA == 2 && B % 4 == 0 && J0 % 4 == 0, "whole chains of four");
#pragma unroll
        for (int u = 0; u < B; u += 4)
#pragma unroll
            for (int q = 0; q < NQ; q++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const A a = (A)vv[u] * (A)x[u][q][i];
                    const A b = __builtin_elementwise_fma((A)vv[u + 1], (A)x[u + 1][q][i], a);
                    const A c = __builtin_elementwise_fma((A)vv[u + 2], (A)x[u + 2][q][i], b);
                    acc[(((J0 + u) / 4 + ODD) % 2 * NQ + q) * 4 + i] +=
                        __builtin_elementwise_fma((A)vv[u + 3], (A)x[u + 3][q][i], c);
                }
        // (keeps the compiler from merging the ends of steps that add to
        // different sums, which would put the sums into scratch memory)
        asm volatile("" ::"n"(((J0 * 64 + B) * 2 + MASKED) * 2 + ODD));
    }
}

// Adds the NA sums of N elements each, pairwise, into the first.
template <int NA, int N, class A> __device__ __forceinline__ void add_sums(A *acc)
{
#pragma unroll
    for (int w = 1; w < NA; w <<= 1)
#pragma unroll
        for (int k = 0; k < NA; k += 2 * w)
#pragma unroll
            for (int i = 0; i < N; i++) acc[k * N + i] += acc[(k + w) * N + i];
}

// The first t (1 .. kEntryBatch<G, NB>) entries of the group's batch, U at a
// time, a last half batch where that still holds whole chains.
template <int J0, int U, int NQ, int G, int NB, int OFF, bool CLS, int NA, class Q, class A>
__device__ __forceinline__ void gather_entries_of(const RowRef<OFF> *ref, const float *v, const int *cold, int t,
                                                  const float *X, const Q &cols, A *acc)
{
    constexpr int H = U / 2 >= (NA == 2 ? 4 : 1) ? U / 2 : U;
    if constexpr (G == 64) {
        constexpr bool PAIR = NA == 2 && U == 4;  // two steps, one for each sum
        const int n = __builtin_amdgcn_readfirstlane(t);  // one row to the wave
        int j = 0;
        if constexpr (PAIR) {
            for (; j + 2 * U <= n; j += 2 * U) {
                gather_step<0, U, NQ, G, false, OFF, CLS, NA, false>(ref, v, cold, n, X, cols, acc, j);
                gather_step<0, U, NQ, G, false, OFF, CLS, NA, true>(ref, v, cold, n, X, cols, acc, j + U);
            }
            if (j + U < n) {
                gather_step<0, U, NQ, G, false, OFF, CLS, NA, false>(ref, v, cold, n, X, cols, acc, j);
                gather_step<0, U, NQ, G, true, OFF, CLS, NA, true>(ref, v, cold, n, X, cols, acc, j + U);
                return;
            }
        } else {
            for (; j + U <= n; j += U)
                gather_step<0, U, NQ, G, false, OFF, CLS, NA, false>(ref, v, cold, n, X, cols, acc, j);
        }
        if (H < U && j < n && n - j <= H)
            gather_step<0, H, NQ, G, true, OFF, CLS, NA, false>(ref, v, cold, n, X, cols, acc, j);
        else if (j < n)
            gather_step<0, U, NQ, G, true, OFF, CLS, NA, false>(ref, v, cold, n, X, cols, acc, j);
    } else if constexpr (J0 < kEntryBatch<G, NB>) {
        if (t >= J0 + U) {
            gather_step<J0, U, NQ, G, false, OFF, CLS, NA, false>(ref, v, cold, t, X, cols, acc);
            gather_entries_of<J0 + U, U, NQ, G, NB, OFF, CLS, NA>(ref, v, cold, t, X, cols, acc);
        } else if (t > J0) {
            if (H < U && t - J0 <= H)
                gather_step<J0, H, NQ, G, true, OFF, CLS, NA, false>(ref, v, cold, t, X, cols, acc);
            else
                gather_step<J0, U, NQ, G, true, OFF, CLS, NA, false>(ref, v, cold, t, X, cols, acc);
        }
        if constexpr (NA == 2 && J0 == 0 && kEntryBatch<G, NB> == 4) {  // a batch is one chain: the other sum is next
#pragma unroll
            for (int i = 0; i < 4 * NQ; i++) {
                const A a = acc[i];
                acc[i] = acc[4 * NQ + i];
                acc[4 * NQ + i] = a;
            }
        }
    }
}

// Stores the lane's quads of acc (rounded to fp32) at the row pointer p,
// streaming: Y is not read again by this kernel, so it does not displace the
// gathered X rows.
template <int NQ, class Q, class A>
__device__ __forceinline__ void store_quads_stream(float *p, const Q &cols, const A *acc)
{
#pragma unroll
    for (int q = 0; q < NQ; q++)
        if (cols.ok(q)) {
            const f4u r = {(float)acc[4 * q], (float)acc[4 * q + 1], (float)acc[4 * q + 2], (float)acc[4 * q + 3]};
            __builtin_nontemporal_store(r, reinterpret_cast<f4u *>(p + cols.base(q) + cols.step(q)));
        }
}

// The lane's quads of acc at p, unrounded (partial sums).
template <int NQ, class Q, class A>
__device__ __forceinline__ void store_quads(A *p, const Q &cols, const A *acc)
{
#pragma unroll
    for (int q = 0; q < NQ; q++)
        if (cols.ok(q))
            *reinterpret_cast<typename Quad<A>::type *>(p + cols.base(q) + cols.step(q)) = {
                acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
}

// One batch of B entries j .. j+B-1 of the group's current index batch:
// B X-row loads issued back to back, then B fused multiply-adds.  MASKED
// batches may run past the last entry m: those slots gather nothing (on a
// 512 x 512 mesh one dead gather a row made the DIA kernel 7% slower) and add
// -0 * 0 = -0, which leaves every sum as it is.  Entry u of the batch goes to
// the sums u % NA.
template <int B, int NQ, int G, bool MASKED, int NA, bool FENCE = false, class Q>
__device__ __forceinline__ void gather_batch(int cj, float vj, int j, int m, const float *__restrict__ X, int64_t ldx,
                                             const Q &cols, float *acc)
{
    f4u x[B][NQ];
    float v[B];
#pragma unroll
    for (int u = 0; u < B; u++) {
        const int cu = __shfl(cj, j + u, G);
        v[u] = __shfl(vj, j + u, G);
        const float *xp = X + (int64_t)cu * ldx;
        if (MASKED) {
#pragma unroll
            for (int q = 0; q < NQ; q++) x[u][q] = f4u{0.f, 0.f, 0.f, 0.f};
            if (j + u >= m) v[u] = -0.0f;
        }
        if (!MASKED) {
#pragma unroll
            for (int q = 0; q < NQ; q++) x[u][q] = __builtin_nondeterministic_value(x[u][q]);
        }
        if (!MASKED || j + u < m) {
#pragma unroll
            for (int q = 0; q < NQ; q++)
                if (Q::kFull || cols.ok(q))
                    x[u][q] = *reinterpret_cast<const f4u *>(xp + cols.base(q) + cols.step(q));
        }
    }
    // FENCE: every load of the batch is issued before the first use.  Where
    // the scheduler aims at a higher occupancy it may otherwise sink each
    // load next to its use, one round trip per X row (seen in the ELL kernel
    // with chain folds: 50 VGPRs and twice the time on a power-law matrix).
    if constexpr (FENCE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < B; u++)
#pragma unroll
        for (int q = 0; q < NQ; q++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                float &a = acc[(u % NA * NQ + q) * 4 + i];
                a = __builtin_fmaf(v[u], x[u][q][i], a);
            }
}

// The first m entries of the group's index batch, U at a time (U a multiple of
// NA), a last half batch where it still holds every sum.
template <int U, int NQ, int G, int NA, bool FENCE, class Q>
__device__ __forceinline__ void gather_batches(int cj, float vj, int m, const float *__restrict__ X, int64_t ldx,
                                               const Q &cols, float *acc)
{
    static_assert(U % NA == 0, "entry j belongs to the sums j % NA");
    constexpr int H = U / 2 >= NA && U > 1 ? U / 2 : U;
    int j = 0;
    for (; j + U <= m; j += U) gather_batch<U, NQ, G, false, NA, FENCE>(cj, vj, j, m, X, ldx, cols, acc);
    if (j >= m) return;
    if (H < U && m - j <= H)
        gather_batch<H, NQ, G, true, NA, FENCE>(cj, vj, j, m, X, ldx, cols, acc);
    else
        gather_batch<U, NQ, G, true, NA, FENCE>(cj, vj, j, m, X, ldx, cols, acc);
}

// One batch of B entries j .. j+B-1 of the group's index batch in a row
// tile whose X rows [w0, w1) are staged in LDS (xs, G*NQ float4 per row, the
// lane's float4 at lane + G*q): in-window rows are read from LDS, the others
// from global memory.  Slots past m gather a valid row and are dropped by a
// select.
template <int B, int NQ, int G, class Q>
__device__ __forceinline__ void window_batch(int cj, float vj, int j, int m, const float4 *xs, int64_t w0,
                                             int64_t w1, int lane, const float *__restrict__ X, int64_t ldx,
                                             const Q &cols, float *acc)
{
    constexpr int RW = G * NQ;
    f4u x[B][NQ];
    float v[B];
#pragma unroll
    for (int u = 0; u < B; u++) {
        const int cu = __shfl(cj, j + u, G);
        v[u] = __shfl(vj, j + u, G);
        if (cu >= w0 && cu < w1) {
            const float4 *xr = xs + (int64_t)(cu - w0) * RW + lane;
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                const float4 r = xr[q * G];
                x[u][q] = f4u{r.x, r.y, r.z, r.w};
            }
        } else {
            const float *xp = X + (int64_t)cu * ldx;
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                x[u][q] = __builtin_nondeterministic_value(x[u][q]);
                if (Q::kFull || cols.ok(q))
                    x[u][q] = *reinterpret_cast<const f4u *>(xp + cols.base(q) + cols.step(q));
            }
        }
    }
#pragma unroll
    for (int u = 0; u < B; u++) {
        const bool live = j + u < m;
#pragma unroll
        for (int q = 0; q < NQ; q++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float a = __builtin_fmaf(v[u], x[u][q][i], acc[4 * q + i]);
                acc[4 * q + i] = live ? a : acc[4 * q + i];
            }
    }
}

// Copies X rows [w0, w0 + W) of the column slice at cbase into LDS, RW quads
// per row, the quads placed as Quads places them.
template <int RW, int NT>
__device__ __forceinline__ void stage_window(float4 *xs, int W, int64_t w0, const float *__restrict__ X, int64_t ldx,
                                             int64_t cbase, int64_t F)
{
    for (int idx = threadIdx.x; idx < W * RW; idx += NT) {
        const int wr = idx / RW, j = idx - wr * RW;
        const int64_t c = cbase + 4 * j;
        const f4u v = *reinterpret_cast<const f4u *>(X + (w0 + wr) * ldx + (c < F - 4 ? c : F - 4));
        xs[idx] = make_float4(v[0], v[1], v[2], v[3]);
    }
}

}  // namespace gs
