// gfx950 kernels for one operation per pass: the amplitude-pair update of
// Eq. 1 (Sec. II.B.1) for state vectors, the 4-element group update that
// fuses the two passes of Eq. 2 for density matrices, the channel updates,
// probability reductions and measurement collapse.
//
// Layout: interleaved complex (double2 / float2), qubit q = bit q of the
// index.  Every kernel loops over 64-bit indices with a grid capped at 16
// blocks per CU, or 64 for passes over 512 MiB and more (stream_shape); the
// streaming kernels take kPer amplitudes per thread per step (see qs_device.h).
#include <algorithm>
#include <complex>
#include <vector>

#include "qs_device.h"

namespace qs {

BitInsert make_insert(const int* positions, int count, uint64_t ones)
{
    BitInsert b{0, ones};
    for (int k = 0; k < count; ++k) b.at |= 1ull << positions[k];
    return b;
}

namespace {

// ---------------------------------------------------------------------------
// Initialisation: every amplitude 0 except `index`, which is (re, im).
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_init_basis(typename C2<T>::type* __restrict__ amp,
                                                       uint64_t len, uint64_t index, T re, T im)
{
    using V = typename C2<T>::type;
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i >= len) continue;
            V v;  // plain stores: measured faster than non-temporal ones for write-only streams
            v.x = (i == index) ? re : T(0);
            v.y = (i == index) ? im : T(0);
            amp[i] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// Eq. 1 pair update for targets whose pair partner lies in another wavefront
// row (t >= 6): each lane owns a pair (a, a + 2^t); 64 consecutive lanes
// touch two contiguous 1 KiB (c128) runs.  `ins` inserts a 0 at t and a 1
// at every control of at least kLineBits; lower controls are the bits of
// `lowmask`, tested per pair.
template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_gate_pair(typename C2<T>::type* __restrict__ amp,
                                                      uint64_t npairs, uint64_t tb, BitInsert ins,
                                                      uint64_t lowmask, Mat2<T> u)
{
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * P;
    const StepItems<P> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    const bool ok = (et & lowmask) == lowmask;  // bits within a line are the thread's own
    for (uint64_t s = blockIdx.x; step_base(s, ps) < npairs; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins) | ins.ones;
        V x[P], y[P];
        bool on[P];
        // all low halves, then all high halves: each run of loads alternates
        // between the step's two half-runs
#pragma unroll
        for (int j = 0; j < P; ++j) {
            on[j] = step_item(c, j, ps) < npairs;
            x[j].x = x[j].y = y[j].x = y[j].y = T(0);
            if (on[j]) x[j] = ldnt(amp + (et + (ec + at(j))));
        }
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (on[j]) y[j] = ldnt(amp + (et + (ec + at(j) + tb)));
#pragma unroll
        for (int j = 0; j < P; ++j) {
            // controls below the line size are tested per pair: unselected
            // pairs are written back unchanged, so every store is a full line
            V nx = x[j], ny = y[j];
            apply2<T, V>(u.m, nx, ny);
            // component-wise selects: a select of whole vector structs puts
            // the arrays in scratch memory
            x[j].x = ok ? nx.x : x[j].x;
            x[j].y = ok ? nx.y : x[j].y;
            y[j].x = ok ? ny.x : y[j].x;
            y[j].y = ok ? ny.y : y[j].y;
        }
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (on[j]) stnt(amp + (et + (ec + at(j))), x[j]);
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (on[j]) stnt(amp + (et + (ec + at(j) + tb)), y[j]);
    }
}

// Cross-lane exchange with lane ^ 2^TT inside a wavefront of 64 lanes:
// DPP quad permutes for 1 and 2, ds_swizzle bit mode for 4, 8, 16 and a
// backwards permute for 32.  All lanes must be active.
template <int TT>
__device__ __forceinline__ int lane_xor(int v, int lane)
{
    if constexpr (TT == 0) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
    else if constexpr (TT == 1) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
    else if constexpr (TT == 2) return __builtin_amdgcn_ds_swizzle(v, 0x101F);
    else if constexpr (TT == 3) return __builtin_amdgcn_ds_swizzle(v, 0x201F);
    else if constexpr (TT == 4) return __builtin_amdgcn_ds_swizzle(v, 0x401F);
    else return __builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, v);
}

template <int TT>
__device__ __forceinline__ double xchg(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = lane_xor<TT>((int)(b & 0xffffffffll), lane);
    const int hi = lane_xor<TT>((int)(b >> 32), lane);
    return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

template <int TT>
__device__ __forceinline__ float xchg(float v, int lane)
{
    return __int_as_float(lane_xor<TT>(__float_as_int(v), lane));
}

// Eq. 1 for targets t < 6: each lane loads ONE amplitude of a contiguous
// 64-amplitude chunk, fetches its pair partner from lane ^ 2^t in registers
// and writes its own new value, so loads and stores stay fully contiguous.
// Controls at bits >= 6 are folded into the chunk index (`hi`); controls at
// bits < 6 become a lane mask.
template <typename T, int TT, int U>
__global__ __launch_bounds__(kBlock) void k_gate_low(typename C2<T>::type* __restrict__ amp,
                                                     uint64_t nchunks, BitInsert hi,
                                                     uint32_t lowmask, Mat2<T> u)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    const int lane = threadIdx.x & 63;
    const bool up = (lane >> TT) & 1;
    const bool ok = ((uint32_t)lane & lowmask) == lowmask;
    // A lane whose controls at or above the 128-byte line are not all set
    // holds a whole line the gate leaves unchanged: it loads and stores
    // nothing.  Its pair partner (lane ^ 2^TT; the target is never a
    // control) has the same control bits, so no active lane reads it.
    constexpr uint32_t kLine = sizeof(T) == 8 ? 3 : 4;
    const uint32_t linemask = lowmask & ~((1u << kLine) - 1);
    const bool act = ((uint32_t)lane & linemask) == linemask;
    // new = s * self + p * partner
    const T sr = up ? u.m[6] : u.m[0], si = up ? u.m[7] : u.m[1];
    const T pr = up ? u.m[4] : u.m[2], pi = up ? u.m[5] : u.m[3];
    // chunks play the role of items: a workgroup step of PS = 4 * kPer
    // chunks is two half-runs PS apart, alternated as in step_item (with
    // the 4 waves in place of the threads)
    const uint64_t w = (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t ps = (uint64_t)(kBlock / 64) * U;
    const StepItems<U> at(ps, kBlock / 64, hi);
    for (uint64_t s = blockIdx.x; step_base(s, ps) < nchunks; s += gridDim.x) {
        const uint64_t c0 = step_base(s, ps) + w;
        const uint64_t ec = deposit(c0, hi) | hi.ones;
        V v[U];
        bool on[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            on[j] = c0 + (uint64_t)(j & 1) * ps + (uint64_t)(j >> 1) * (kBlock / 64) < nchunks;  // uniform over the wave
            v[j].x = T(0);
            v[j].y = T(0);
            if (act && on[j]) v[j] = ldnt(amp + (((ec + at(j)) << 6) + (uint64_t)lane));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            // the chunk test is uniform over the wave, so every lane joins the exchange
            V p;
            p.x = xchg<TT>(v[j].x, lane);
            p.y = xchg<TT>(v[j].y, lane);
            const V r = cmac2<T, V>(sr, si, v[j], pr, pi, p);
            // active lanes whose controls below the line are not all set
            // store their value unchanged, so that every store covers whole
            // lines
            V o;
            o.x = ok ? r.x : v[j].x;
            o.y = ok ? r.y : v[j].y;
            if (act && on[j]) stnt(amp + (((ec + at(j)) << 6) + (uint64_t)lane), o);
        }
    }
}

// Multi-controlled NOT: swap each pair whose controls are set (controls
// below kLineBits tested per pair, as in k_gate_pair).
template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_not(typename C2<T>::type* __restrict__ amp,
                                                uint64_t npairs, uint64_t tb, BitInsert ins, uint64_t lowmask)
{
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * P;
    const StepItems<P> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    const bool ok = (et & lowmask) == lowmask;  // bits within a line are the thread's own
    for (uint64_t s = blockIdx.x; step_base(s, ps) < npairs; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins) | ins.ones;
        V x[P], y[P];
        bool on[P];
        // all low halves, then all high halves: each run of loads alternates
        // between the step's two half-runs
#pragma unroll
        for (int j = 0; j < P; ++j) {
            on[j] = step_item(c, j, ps) < npairs;
            x[j].x = x[j].y = y[j].x = y[j].y = T(0);
            if (on[j]) x[j] = ldnt(amp + (et + (ec + at(j))));
        }
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (on[j]) y[j] = ldnt(amp + (et + (ec + at(j) + tb)));
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const T x0 = x[j].x, x1 = x[j].y;
            x[j].x = ok ? y[j].x : x0;
            x[j].y = ok ? y[j].y : x1;
            y[j].x = ok ? x0 : y[j].x;
            y[j].y = ok ? x1 : y[j].y;
        }
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (on[j]) stnt(amp + (et + (ec + at(j))), x[j]);
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (on[j]) stnt(amp + (et + (ec + at(j) + tb)), y[j]);
    }
}

// Diagonal phase on the amplitudes whose `ins.ones` bits are all set,
// except those that also have every bit of `skip` set (skip != 0).
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_phase(typename C2<T>::type* __restrict__ amp,
                                                  uint64_t count, BitInsert ins, uint64_t lowmask,
                                                  uint64_t skip, T fr, T fi)
{
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * U;
    const StepItems<U> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    // bits within a line are the thread's own: its other values are written
    // back unchanged so that every store is a full line, and so are excepted
    // ones; only where no bit of `skip` lies within a line are those not touched
    const bool ok = (et & lowmask) == lowmask;
    constexpr uint64_t kIn = (1ull << kLineBits<T>) - 1;
    const uint64_t sin = skip & kIn, sline = skip & ~kIn;
    const uint64_t none = skip && !sin ? 0 : ~0ull;              // all ones: no line is left out
    const uint64_t kept = sin && (et & sin) == sin ? 0 : ~0ull;  // all ones: this thread's values all turn
    for (uint64_t s = blockIdx.x; step_base(s, ps) < count; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins) | ins.ones;
        bool on[U], hit[U];
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t e = et + (ec + at(j));
            on[j] = step_item(c, j, ps) < count && (e & sline) != (sline | none);
            hit[j] = ok && (e & sline) != (sline | kept);
            v[j].x = v[j].y = T(0);
            if (on[j]) v[j] = ldnt(amp + e);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const V m = cmul<T, V>(fr, fi, v[j]);
            v[j].x = hit[j] ? m.x : v[j].x;
            v[j].y = hit[j] ? m.y : v[j].y;
        }
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (on[j]) stnt(amp + (et + (ec + at(j))), v[j]);
    }
}

// Phase of a density matrix on qubits some of which lie within a line, rows
// and columns in one pass: rows with all bits of `rmask` set gain (fr, fi), columns with
// all bits of `cmask` set its conjugate, entries with both nothing.  Two
// passes of k_phase read and write most lines twice (CZ on qubits 0 and 1 of
// 13: complex128 512 us, 365 so; complex64 455, 162).
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_dm_phase(typename C2<T>::type* __restrict__ rho, uint64_t len,
                                                     uint64_t rmask, uint64_t cmask, T fr, T fi)
{
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * U;
    constexpr uint64_t kIn = (1ull << kLineBits<T>) - 1;
    const bool rin = ((threadIdx.x & rmask) & kIn) == (rmask & kIn), cin = ((threadIdx.x & cmask) & kIn) == (cmask & kIn);
    const uint64_t rline = rmask & ~kIn, cline = cmask & ~kIn;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        bool r[U], k[U];
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t e = step_item(c, j, ps);
            r[j] = e < len && (e & rline) == rline;
            k[j] = e < len && (e & cline) == cline;
            v[j].x = v[j].y = T(0);
            if (r[j] || k[j]) v[j] = ldnt(rho + e);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const bool row = r[j] && rin, col = k[j] && cin;
            const V m = cmul<T, V>(fr, row ? fi : -fi, v[j]);
            v[j].x = row != col ? m.x : v[j].x;
            v[j].y = row != col ? m.y : v[j].y;
        }
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (r[j] || k[j]) stnt(rho + step_item(c, j, ps), v[j]);
    }
}

template <typename T> constexpr int kHalfBits = kLineBits<T> - 1;

// Density matrix, Eq. 2 fused into one pass.  A group is the four entries
// (rho[r][c]) with row bit t = r and column bit t + N = c; the gate is
// rho -> (R ? U : I) rho (C ? U^dagger : I), R and C: all bits of rmask, cmask
// set.  Columns multiplied by U^dagger is conj(U) on the column qubit.
// `rline`, `cline`: the parts of rmask and cmask at or above half a line; a
// lane whose half holds no selected entry touches nothing, the others store
// whole halves.  13 qubits, control 2 (the upper half of each line, complex128),
// gate on qubit 12: 350 us by whole lines, 315 so; control 3 in complex64 177, 158.
template <typename T, int G>
__global__ __launch_bounds__(kBlock) void k_dm_gate(typename C2<T>::type* __restrict__ rho,
                                                    uint64_t ngroups, uint64_t tb, uint64_t cb,
                                                    BitInsert ins, uint64_t rmask, uint64_t cmask,
                                                    Mat2<T> u)
{
    using V = typename C2<T>::type;
    T uc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) uc[k] = (k & 1) ? -u.m[k] : u.m[k];
    const uint64_t rline = rmask & ~((1ull << kHalfBits<T>) - 1), cline = cmask & ~((1ull << kHalfBits<T>) - 1);
    const uint64_t ps = (uint64_t)kBlock * G;
    const StepItems<G> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    for (uint64_t s = blockIdx.x; step_base(s, ps) < ngroups; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins);
        uint64_t b[G];
        bool act[G];
        V m00[G], m10[G], m01[G], m11[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            b[j] = et + (ec + at(j));
            act[j] = step_item(c, j, ps) < ngroups && ((b[j] & rline) == rline || (b[j] & cline) == cline);
            if (act[j]) {
                m00[j] = ldnt(rho + b[j]);
                m10[j] = ldnt(rho + b[j] + tb);
                m01[j] = ldnt(rho + b[j] + cb);
                m11[j] = ldnt(rho + b[j] + tb + cb);
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (!act[j]) continue;
            if ((b[j] & rmask) == rmask) {  // U on the row index, for each column
                apply2<T, V>(u.m, m00[j], m10[j]);
                apply2<T, V>(u.m, m01[j], m11[j]);
            }
            if ((b[j] & cmask) == cmask) {  // conj(U) on the column index, for each row
                apply2<T, V>(uc, m00[j], m01[j]);
                apply2<T, V>(uc, m10[j], m11[j]);
            }
            stnt(rho + b[j], m00[j]);
            stnt(rho + b[j] + tb, m10[j]);
            stnt(rho + b[j] + cb, m01[j]);
            stnt(rho + b[j] + tb + cb, m11[j]);
        }
    }
}

// The same for a target within a line: a lane holds the two entries (column
// bit 0 and 1) of its own row bit and gets the other row's from the lane that
// holds them, so that every access covers whole lines.  One 4-group per
// thread touched each line twice, half of it at a time.  13 qubits, target 0:
// complex128 637 us before, 350 now; complex64 247, 173 (6.2 TB/s).
template <typename T, int G>
__global__ __launch_bounds__(kBlock) void k_dm_gate_low(typename C2<T>::type* __restrict__ rho, uint64_t nitems,
                                                        uint64_t tb, uint64_t cb, BitInsert ins, uint64_t rmask,
                                                        uint64_t cmask, Mat2<T> u)
{
    using V = typename C2<T>::type;
    const bool up = (threadIdx.x & tb) != 0;
    const int src = (int)(((threadIdx.x & 63) ^ tb) << 2);
    const T sr = up ? u.m[6] : u.m[0], si = up ? u.m[7] : u.m[1];
    const T pr = up ? u.m[4] : u.m[2], pi = up ? u.m[5] : u.m[3];
    T uc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) uc[k] = (k & 1) ? -u.m[k] : u.m[k];
    const uint64_t rline = rmask & ~((1ull << kHalfBits<T>) - 1), cline = cmask & ~((1ull << kHalfBits<T>) - 1);
    const uint64_t ps = (uint64_t)kBlock * G;
    const StepItems<G> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    for (uint64_t s = blockIdx.x; step_base(s, ps) < nitems; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins);
        uint64_t b[G];
        bool act[G];
        V v0[G], v1[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            b[j] = et + (ec + at(j));
            act[j] = step_item(c, j, ps) < nitems && ((b[j] & rline) == rline || (b[j] & cline) == cline);
            v0[j].x = v0[j].y = v1[j].x = v1[j].y = T(0);
            if (act[j]) {
                v0[j] = ldnt(rho + b[j]);
                v1[j] = ldnt(rho + b[j] + cb);
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            V p0, p1;  // all lanes take part; a lane and its partner are both active or both not
            p0.x = lane_across(v0[j].x, src);
            p0.y = lane_across(v0[j].y, src);
            p1.x = lane_across(v1[j].x, src);
            p1.y = lane_across(v1[j].y, src);
            if (!act[j]) continue;
            const bool r = (b[j] & rmask) == rmask, k = (b[j] & cmask) == cmask;
            // U on the row index (its first term is the row with bit 0)
            const V n0 = up ? cmac2<T, V>(pr, pi, p0, sr, si, v0[j]) : cmac2<T, V>(sr, si, v0[j], pr, pi, p0);
            const V n1 = up ? cmac2<T, V>(pr, pi, p1, sr, si, v1[j]) : cmac2<T, V>(sr, si, v1[j], pr, pi, p1);
            V a, d;
            a.x = r ? n0.x : v0[j].x;
            a.y = r ? n0.y : v0[j].y;
            d.x = r ? n1.x : v1[j].x;
            d.y = r ? n1.y : v1[j].y;
            V o0 = a, o1 = d;
            apply2<T, V>(uc, o0, o1);
            a.x = k ? o0.x : a.x;
            a.y = k ? o0.y : a.y;
            d.x = k ? o1.x : d.x;
            d.y = k ? o1.y : d.y;
            stnt(rho + b[j], a);
            stnt(rho + b[j] + cb, d);
        }
    }
}

// Channel closed forms on each 4-group (arithmetic in double).
//   dephasing p:     off-diagonals * (1 - 2p)
//   depolarising p:  r00 <- (1-2p/3) r00 + (2p/3) r11, r11 symmetric,
//                    off-diagonals * (1 - 4p/3)
//   damping g:       r00 <- r00 + g r11, r11 <- (1-g) r11,
//                    off-diagonals * sqrt(1-g)
// a, b: diagonal mixing (r00' = a r00 + b r11 ... per channel), f: off-diagonal factor.
template <typename T, int CH, int G>
__global__ __launch_bounds__(kBlock) void k_dm_channel(typename C2<T>::type* __restrict__ rho,
                                                       uint64_t ngroups, uint64_t tb, uint64_t cb,
                                                       BitInsert ins, double p0, double p1, double f)
{
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * G;
    const StepItems<G> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    for (uint64_t s = blockIdx.x; step_base(s, ps) < ngroups; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins);
        uint64_t b[G];
        V m00[G], m10[G], m01[G], m11[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            b[j] = et + (ec + at(j));
            if (step_item(c, j, ps) >= ngroups) continue;
            m10[j] = ldnt(rho + b[j] + tb);
            m01[j] = ldnt(rho + b[j] + cb);
            if constexpr (CH != QS_DEPHASING) {
                m00[j] = ldnt(rho + b[j]);
                m11[j] = ldnt(rho + b[j] + tb + cb);
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (step_item(c, j, ps) >= ngroups) continue;
            V n10, n01;
            n10.x = (T)(f * (double)m10[j].x);
            n10.y = (T)(f * (double)m10[j].y);
            n01.x = (T)(f * (double)m01[j].x);
            n01.y = (T)(f * (double)m01[j].y);
            stnt(rho + b[j] + tb, n10);
            stnt(rho + b[j] + cb, n01);
            if constexpr (CH != QS_DEPHASING) {
                const double a0 = m00[j].x, a1 = m00[j].y, d0 = m11[j].x, d1 = m11[j].y;
                V n00, n11;
                if constexpr (CH == QS_DEPOLARISING) {  // p0 = 1 - 2p/3, p1 = 2p/3
                    n00.x = (T)(p0 * a0 + p1 * d0);
                    n00.y = (T)(p0 * a1 + p1 * d1);
                    n11.x = (T)(p0 * d0 + p1 * a0);
                    n11.y = (T)(p0 * d1 + p1 * a1);
                } else {  // damping: p0 = gamma, p1 = 1 - gamma
                    n00.x = (T)(a0 + p0 * d0);
                    n00.y = (T)(a1 + p0 * d1);
                    n11.x = (T)(p1 * d0);
                    n11.y = (T)(p1 * d1);
                }
                stnt(rho + b[j], n00);
                stnt(rho + b[j] + tb + cb, n11);
            }
        }
    }
}

// The same for a target within a line (see k_dm_gate_low): a lane holds one
// diagonal and one off-diagonal entry of its group, and the other diagonal
// entry comes from the partner lane.  Depolarising on qubit 0 of 13: complex128
// 710 us with one group per thread, 343 so; complex64 305, 168.  Dephasing
// rewrites whole lines here, half of them unchanged: 575 and 355 us.
template <typename T, int CH, int G>
__global__ __launch_bounds__(kBlock) void k_dm_channel_low(typename C2<T>::type* __restrict__ rho, uint64_t nitems,
                                                           uint64_t tb, uint64_t cb, BitInsert ins, double p0,
                                                           double p1, double f)
{
    using V = typename C2<T>::type;
    const bool up = (threadIdx.x & tb) != 0;
    const int src = (int)(((threadIdx.x & 63) ^ tb) << 2);
    const uint64_t ps = (uint64_t)kBlock * G;
    const StepItems<G> at(ps, kBlock, ins);
    const uint64_t et = deposit(threadIdx.x, ins);
    for (uint64_t s = blockIdx.x; step_base(s, ps) < nitems; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        const uint64_t ec = deposit(c, ins);
        uint64_t b[G];
        bool on[G];
        V v0[G], v1[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            b[j] = et + (ec + at(j));
            on[j] = step_item(c, j, ps) < nitems;
            v0[j].x = v0[j].y = v1[j].x = v1[j].y = T(0);
            if (on[j]) {
                v0[j] = ldnt(rho + b[j]);
                v1[j] = ldnt(rho + b[j] + cb);
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            // the diagonal entry is the one whose column bit is the lane's row bit
            V d, n, m;
            d.x = up ? v1[j].x : v0[j].x;
            d.y = up ? v1[j].y : v0[j].y;
            m.x = up ? v0[j].x : v1[j].x;
            m.y = up ? v0[j].y : v1[j].y;
            n = d;
            if constexpr (CH != QS_DEPHASING) {
                const double q0 = lane_across(d.x, src), q1 = lane_across(d.y, src);
                const double d0 = d.x, d1 = d.y;
                if constexpr (CH == QS_DEPOLARISING) {  // p0 = 1 - 2p/3, p1 = 2p/3
                    n.x = (T)(p0 * d0 + p1 * q0);
                    n.y = (T)(p0 * d1 + p1 * q1);
                } else {  // damping: p0 = gamma, p1 = 1 - gamma
                    n.x = up ? (T)(p1 * d0) : (T)(d0 + p0 * q0);
                    n.y = up ? (T)(p1 * d1) : (T)(d1 + p0 * q1);
                }
            }
            m.x = (T)(f * (double)m.x);
            m.y = (T)(f * (double)m.y);
            v0[j].x = up ? m.x : n.x;
            v0[j].y = up ? m.y : n.y;
            v1[j].x = up ? n.x : m.x;
            v1[j].y = up ? n.y : m.y;
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (!on[j]) continue;
            stnt(rho + b[j], v0[j]);
            stnt(rho + b[j] + cb, v1[j]);
        }
    }
}

// ---------------------------------------------------------------------------
// Reductions: per-thread Neumaier sums in double, merged across the wave
// with cross-lane shuffles and across the block through LDS; one partial
// per block, folded by k_reduce_final.  A block that is alone writes the two
// results itself.  `out` may be pinned host memory: the sums are there when
// the stream has been waited for, with no copy behind the kernels.
__device__ __forceinline__ NSum wave_merge(NSum a)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        NSum o;
        o.s = __shfl_xor(a.s, off, 64);
        o.c = __shfl_xor(a.c, off, 64);
        a = nmerge(a, o);
    }
    return a;
}

__device__ __forceinline__ void block_store2(NSum s0, NSum s1, double* partials, double* out)
{
    __shared__ double sh[4][kBlock / 64];
    s0 = wave_merge(s0);
    s1 = wave_merge(s1);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[0][w] = s0.s;
        sh[1][w] = s0.c;
        sh[2][w] = s1.s;
        sh[3][w] = s1.c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        NSum a = {sh[0][0], sh[1][0]}, b = {sh[2][0], sh[3][0]};
        for (int k = 1; k < kBlock / 64; ++k) {
            a = nmerge(a, NSum{sh[0][k], sh[1][k]});
            b = nmerge(b, NSum{sh[2][k], sh[3][k]});
        }
        if (gridDim.x == 1) {
            out[0] = a.s + a.c;
            out[1] = b.s + b.c;
            return;
        }
        partials[4 * blockIdx.x + 0] = a.s;
        partials[4 * blockIdx.x + 1] = a.c;
        partials[4 * blockIdx.x + 2] = b.s;
        partials[4 * blockIdx.x + 3] = b.c;
    }
}

// Sum |alpha_i|^2 split by bit q of i (q < 0: everything in the first sum).
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_prob_sv(const typename C2<T>::type* __restrict__ amp,
                                                    uint64_t len, int q, double* partials,
                                                    double* out)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    NSum s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            v[j] = ldnt(amp + (i < len ? i : len - 1));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            const double p = i < len ? (double)v[j].x * (double)v[j].x + (double)v[j].y * (double)v[j].y : 0.0;
            const bool one = (q >= 0) && ((i >> q) & 1);
            nadd(s0, one ? 0.0 : p);
            nadd(s1, one ? p : 0.0);
        }
    }
    block_store2(s0, s1, partials, out);
}

// Sum |alpha_i|^2 over the indices i whose bit q equals o, reading only
// those: item k stands for k with bit o inserted at position q.  With q at
// or above the line bits every 128-byte line lies in one half, so half the
// state is read.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_prob_half_sv(const typename C2<T>::type* __restrict__ amp,
                                                         uint64_t half, int q, int o, double* partials,
                                                         double* out)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    NSum s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    const uint64_t ps = (uint64_t)kBlock * U;
    const uint64_t low = (1ull << q) - 1, bit = (uint64_t)o << q;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < half; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t k0 = step_item(c, j, ps);
            const uint64_t k = k0 < half ? k0 : half - 1;
            v[j] = ldnt(amp + (((k & ~low) << 1) | bit | (k & low)));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const double p = step_item(c, j, ps) < half
                                 ? (double)v[j].x * (double)v[j].x + (double)v[j].y * (double)v[j].y
                                 : 0.0;
            nadd(s0, p);
        }
    }
    block_store2(s0, s1, partials, out);
}

// Sum Re rho[j][j] split by bit q of j (the diagonal is entry j (2^N + 1)).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_prob_dm(const typename C2<T>::type* __restrict__ rho,
                                                    uint64_t dim, int q, double* partials,
                                                    double* out)
{
    NSum s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t j = (uint64_t)blockIdx.x * kBlock + threadIdx.x; j < dim; j += stride) {
        const double p = (double)rho[j * (dim + 1)].x;
        const bool one = (q >= 0) && ((j >> q) & 1);
        nadd(s0, one ? 0.0 : p);
        nadd(s1, one ? p : 0.0);
    }
    block_store2(s0, s1, partials, out);
}

// out[j] = sum over rows i of part[i * cols + j], in row order (one thread
// per column, compensated): the fused readouts' per-workgroup sums.
__global__ __launch_bounds__(64) void k_sum_columns(const double* __restrict__ part, int rows, int cols,
                                                    double* __restrict__ out)
{
    const int j = blockIdx.x * 64 + threadIdx.x;
    if (j >= cols) return;
    NSum a = {0.0, 0.0};
    for (int i = 0; i < rows; ++i) nadd(a, part[(size_t)i * cols + j]);
    out[j] = a.s + a.c;
}

__global__ __launch_bounds__(kBlock) void k_reduce_final(const double* __restrict__ partials,
                                                         int nblocks, double* out)
{
    NSum s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    for (int b = threadIdx.x; b < nblocks; b += kBlock) {
        s0 = nmerge(s0, NSum{partials[4 * b + 0], partials[4 * b + 1]});
        s1 = nmerge(s1, NSum{partials[4 * b + 2], partials[4 * b + 3]});
    }
    __shared__ double tmp[4 * 4];
    s0 = wave_merge(s0);
    s1 = wave_merge(s1);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        tmp[4 * w + 0] = s0.s;
        tmp[4 * w + 1] = s0.c;
        tmp[4 * w + 2] = s1.s;
        tmp[4 * w + 3] = s1.c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        NSum a = {tmp[0], tmp[1]}, b = {tmp[2], tmp[3]};
        for (int k = 1; k < kBlock / 64; ++k) {
            a = nmerge(a, NSum{tmp[4 * k + 0], tmp[4 * k + 1]});
            b = nmerge(b, NSum{tmp[4 * k + 2], tmp[4 * k + 3]});
        }
        out[0] = a.s + a.c;
        out[1] = b.s + b.c;
    }
}

// Collapse: keep amplitudes with bit q == outcome (scaled in double), zero
// the rest without reading them.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_collapse_sv(typename C2<T>::type* __restrict__ amp,
                                                        uint64_t len, int q, int outcome, double scale)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            v[j].x = T(0);
            v[j].y = T(0);
            if (i < len && (int)((i >> q) & 1) == outcome) v[j] = ldnt(amp + i);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i >= len) continue;
            V r;
            r.x = (T)(scale * (double)v[j].x);
            r.y = (T)(scale * (double)v[j].y);
            stnt(amp + i, r);
        }
    }
}

// Density-matrix collapse: keep rho[j][k] when bit q of j and of k both
// equal the outcome (bits q and q+N of the vector index), scaled by 1/p.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_collapse_dm(typename C2<T>::type* __restrict__ rho,
                                                        uint64_t len, int q, int N, int outcome,
                                                        double scale)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            v[j].x = T(0);
            v[j].y = T(0);
            const bool keep = (int)((i >> q) & 1) == outcome && (int)((i >> (q + N)) & 1) == outcome;
            if (i < len && keep) v[j] = ldnt(rho + i);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i >= len) continue;
            V r;
            r.x = (T)(scale * (double)v[j].x);
            r.y = (T)(scale * (double)v[j].y);
            stnt(rho + i, r);
        }
    }
}

// ---------------------------------------------------------------------------
// Measure-all.  The items j < count of a subspace sit at index
// pattern + (j << shift), with the outcomes so far in `st` (null: none yet);
// item j falls in bin j mod 2^mbits; mbits is 10, or less and count = 2^mbits.
// Each block writes 2^mbits Neumaier partials (sum, compensation) of
// |alpha|^2, or of a density matrix's diagonal (DM: entry i at i (dim + 1)).
// Steps are multiples of 1024 items, so with the alternating step order the
// thread's j-th element lies in bin ((j >> 1) & 3) * kBlock + tid of 1024:
// four bins per thread, no exchange between threads.
template <typename T, int U, bool DM>
__global__ __launch_bounds__(kBlock) void k_hist(const typename C2<T>::type* __restrict__ amp, uint64_t count,
                                                 int shift, uint64_t dim, const MeasureState* __restrict__ st,
                                                 int mbits, double* __restrict__ partials)
{
    using V = typename C2<T>::type;
    const uint64_t fixed = st ? st->pattern : 0;
    static_assert((kBlock * U / 2) % 1024 == 0, "steps must be whole multiples of 1024 bins");
    NSum acc[4] = {};
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < count; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t item = step_item(c, j, ps);
            const uint64_t i = fixed + ((item < count ? item : count - 1) << shift);
            v[j] = ldnt(amp + (DM ? i * (dim + 1) : i));
        }
        // all loads before the sums: left alone the compiler keeps one or two in flight, 1.54 ms for 28 qubits, not 0.61
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const double p = DM ? (double)v[j].x : (double)v[j].x * (double)v[j].x + (double)v[j].y * (double)v[j].y;
            nadd(acc[(j >> 1) & 3], step_item(c, j, ps) < count ? p : 0.0);
        }
    }
    const int nb = 1 << mbits;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int b = k * kBlock + threadIdx.x;
        if (b < nb) {
            partials[2 * ((uint64_t)blockIdx.x * nb + b)] = acc[k].s;
            partials[2 * ((uint64_t)blockIdx.x * nb + b) + 1] = acc[k].c;
        }
    }
}

// Folds the blocks' partials of each bin, 16 bins of 16 slices of the rows per
// block; out[2b], out[2b+1] = (sum, compensation).  256 rows of 1024 bins in 6
// us, 67 by one thread per bin.
__global__ __launch_bounds__(kBlock) void k_hist_final(const double* __restrict__ partials, int nblocks,
                                                       int nb, double* __restrict__ out)
{
    const int lb = threadIdx.x & 15, slice = threadIdx.x >> 4;
    const int b = blockIdx.x * 16 + lb;
    __shared__ NSum sh[16][16];
    NSum a = {0.0, 0.0};
    if (b < nb)
        for (int k = slice; k < nblocks; k += 16)
            a = nmerge(a, NSum{partials[2 * ((uint64_t)k * nb + b)], partials[2 * ((uint64_t)k * nb + b) + 1]});
    sh[slice][lb] = a;
    __syncthreads();
    if (slice != 0 || b >= nb) return;
    for (int k = 1; k < 16; ++k) a = nmerge(a, sh[k][lb]);
    out[2 * b] = a.s;
    out[2 * b + 1] = a.c;
}

// Outcomes of the 2^mbits-bin group of qubits from `shift` on, one after the
// other (see launch_measure_stage), by one block from `rows` rows of bin
// sums.  The bins are folded in halves, so that level k holds the sums over
// all bins that agree in their k low bits, and a qubit's two weights are two
// entries of its level.  `last` also forms the measured entry.  Results go to
// pinned host memory: on the host the walk cost a copy and a wait per group,
// of 13 qubits two of them and about 40 us.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_measure_walk(const double* __restrict__ bins, int rows, int mbits,
                                                         int shift, Draws draws, bool last, bool dm, int n,
                                                         const typename C2<T>::type* __restrict__ amp,
                                                         MeasureState* __restrict__ st, double* __restrict__ res)
{
    __shared__ NSum t[2048];  // level k at 2^k
    const int nb = 1 << mbits;
    for (int b = threadIdx.x; b < nb; b += kBlock) {
        NSum a = {0.0, 0.0};
        for (int r = 0; r < rows; ++r)
            a = nmerge(a, NSum{bins[2 * ((uint64_t)r * nb + b)], bins[2 * ((uint64_t)r * nb + b) + 1]});
        t[nb + b] = a;
    }
    for (int k = mbits - 1; k >= 1; --k) {
        __syncthreads();
        const int h = 1 << k;
        for (int b = threadIdx.x; b < h; b += kBlock) t[h + b] = nmerge(t[2 * h + b], t[3 * h + b]);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double g = shift ? st->g : 1.0;
    uint64_t pattern = shift ? st->pattern : 0;
    int err = shift ? st->err : 0;
    for (int k = 0, sub = 0; k < mbits && !err; ++k) {
        const NSum w0 = t[(2 << k) + sub], w1 = t[(2 << k) + (sub | (1 << k))];
        double p0 = (w0.s + w0.c) * g;
        if (p0 < 0.0) p0 = 0.0;
        if (p0 > 1.0) p0 = 1.0;
        const int o = draws.u[shift + k] < p0 ? 0 : 1;
        const double p = (o ? w1.s + w1.c : w0.s + w0.c) * g;
        if (!(p > 0.0)) {
            err = 1;
            break;
        }
        res[1 + shift + k] = p;
        res[1 + kMaxMeasured + shift + k] = o;
        g /= p;
        pattern |= (uint64_t)o << (shift + k);
        sub |= o << k;
    }
    if (last && !err) {  // the kept entry, scaled in double precision
        const uint64_t pos = dm ? pattern + (pattern << n) : pattern;
        const double scale = dm ? g : sqrt(g);
        st->re = (double)amp[pos].x * scale;
        st->im = (double)amp[pos].y * scale;
        st->pos = pos;
    }
    st->g = g;
    st->pattern = pattern;
    st->err = err;
    if (last) res[0] = err;
}

// The basis entry that k_measure_walk has formed, everything else zero; after
// an error the state is left as it is.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_measure_basis(typename C2<T>::type* __restrict__ amp, uint64_t len,
                                                          const MeasureState* __restrict__ st)
{
    using V = typename C2<T>::type;
    if (st->err) return;
    const uint64_t pos = st->pos;
    const T re = (T)st->re, im = (T)st->im;
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i >= len) continue;
            V v;
            v.x = i == pos ? re : T(0);
            v.y = i == pos ? im : T(0);
            amp[i] = v;
        }
    }
}

// dst <- src, from 256 MiB on; smaller states take the runtime's copy.  28
// qubits complex128, 8.6 GB moved: 1.44 ms, 1.98 by the runtime's copy; plain
// stores 1.54.  256 MiB 95 us and 100; 128 MiB 46 and 37; 16 MiB 6.9 and 4.5.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_copy(typename C2<T>::type* __restrict__ dst,
                                                 const typename C2<T>::type* __restrict__ src, uint64_t len)
{
    using V = typename C2<T>::type;
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i < len) v[j] = ldnt(src + i);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i < len) stnt(dst + i, v[j]);
        }
    }
}

// ---------------------------------------------------------------------------
// k-qubit groups.  Eq. 1 and the Eq. 2 identity hold for gates on several
// qubits (Sec. II.B.1): a group is the D = 2^k amplitudes that agree on
// every bit outside the target set, member r at base + the sum of the target
// bits whose bit of r is set; the group is replaced by m times it (m: D x D
// complex, row-major, interleaved).  Targets and member bits are in ascending
// order of the qubits.  Controls below the line size are the bits of
// `lowmask`, tested per group: unselected groups are written back unchanged.
//
// k <= 3, no target within a line: one thread holds P groups, all D members
// of each, and the matrix is read with scalar loads.
template <typename T, int K>
struct MatK {
    T m[2 << (2 * K)];
};

template <int K>
struct GroupBits {
    uint64_t tbit[K];
};

template <int K>
__device__ __forceinline__ uint64_t group_off(const GroupBits<K>& gb, int r)
{
    uint64_t o = 0;
#pragma unroll
    for (int j = 0; j < K; ++j)
        if ((r >> j) & 1) o += gb.tbit[j];
    return o;
}

template <typename T, int K, int P>
__global__ __launch_bounds__(kBlock) void k_group_gate(typename C2<T>::type* __restrict__ amp,
                                                       uint64_t ngroups, BitInsert ins, GroupBits<K> gb,
                                                       uint64_t lowmask, MatK<T, K> mk)
{
    using V = typename C2<T>::type;
    constexpr int D = 1 << K;
    const uint64_t tb = deposit(threadIdx.x, ins);
    for (uint64_t g0 = (uint64_t)blockIdx.x * kBlock * P; g0 < ngroups; g0 += (uint64_t)gridDim.x * kBlock * P) {
        uint64_t b[P];
        bool on[P];
        V x[P][D];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            b[p] = tb + (deposit(g0 + (uint64_t)p * kBlock, ins) | ins.ones);
            on[p] = g0 + (uint64_t)p * kBlock + threadIdx.x < ngroups;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                x[p][j].x = x[p][j].y = T(0);
                if (on[p]) x[p][j] = ldnt(amp + b[p] + group_off<K>(gb, j));
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (!on[p]) continue;
            const bool ok = (b[p] & lowmask) == lowmask;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const T* row = mk.m + 2 * D * i;
                // one product or multiply-add per statement: every term is a
                // fused multiply-add
                T re = row[0] * x[p][0].x;
                T im = row[0] * x[p][0].y;
                re = -row[1] * x[p][0].y + re;
                im = row[1] * x[p][0].x + im;
#pragma unroll
                for (int j = 1; j < D; ++j) {
                    re = row[2 * j] * x[p][j].x + re;
                    re = -row[2 * j + 1] * x[p][j].y + re;
                    im = row[2 * j] * x[p][j].y + im;
                    im = row[2 * j + 1] * x[p][j].x + im;
                }
                V y;
                y.x = ok ? re : x[p][i].x;
                y.y = ok ? im : x[p][i].y;
                stnt(amp + b[p] + group_off<K>(gb, i), y);
            }
        }
    }
}

// k <= 3 with L targets within a line: those select the lane, the K - L others
// the register, and a lane gets the members of the other lanes of its group by
// cross-lane reads.  Loads and stores stay whole lines; with one group per
// thread each load of a wave touched 64 lines (k = 3 on qubits 0, 1, 2 of 25
// in complex128: 1,535 us against 190 on high qubits; 192 so).  `ins` inserts a
// 0 at the targets of at least a line and a 1 at the high controls.
template <typename T, int K, int L, int P>
__global__ __launch_bounds__(kBlock) void k_group_lane(typename C2<T>::type* __restrict__ amp, uint64_t nitems,
                                                       BitInsert ins, GroupBits<K> gb, uint64_t lowmask,
                                                       MatK<T, K> mk)
{
    using V = typename C2<T>::type;
    constexpr int D = 1 << K, X = 1 << L, R = 1 << (K - L);
    static_assert(P % 2 == 0, "the step order alternates two half-runs");
    const int lane = threadIdx.x & 63;
    uint32_t own = 0;  // this lane's low member bits
    int src[X];        // byte index of the lane that differs in the member bits of x
#pragma unroll
    for (int j = 0; j < L; ++j) own |= ((uint32_t)lane & (uint32_t)gb.tbit[j]) ? 1u << j : 0u;
#pragma unroll
    for (int x = 0; x < X; ++x) {
        uint32_t mask = 0;
#pragma unroll
        for (int j = 0; j < L; ++j)
            if ((x >> j) & 1) mask |= (uint32_t)gb.tbit[j];
        src[x] = (int)(((uint32_t)lane ^ mask) << 2);
    }
    // c[r][x][s]: entry (own + r X, (own ^ x) + s X), read by each lane from
    // the kernel's arguments (selected from scalar registers, an 8 x 8 matrix
    // did not fit them: complex128, 25 qubits, targets 0, 1, 2: 293 us, 225 so)
    T cr[R][X][R], ci[R][X][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int x = 0; x < X; ++x)
#pragma unroll
            for (int s = 0; s < R; ++s) {
                const uint32_t e = 2 * ((own + r * X) * D + ((own ^ x) + s * X));
                cr[r][x][s] = mk.m[e];
                ci[r][x][s] = mk.m[e + 1];
            }
    }
    uint64_t hoff[R];
#pragma unroll
    for (int r = 0; r < R; ++r) hoff[r] = group_off<K>(gb, r * X);
    const uint64_t tb = deposit(threadIdx.x, ins);
    const uint64_t ps = (uint64_t)kBlock * P;
    const StepItems<P> at(ps, kBlock, ins);
    for (uint64_t st = blockIdx.x; step_base(st, ps) < nitems; st += gridDim.x) {
        const uint64_t c = step_base(st, ps);
        const uint64_t ec = deposit(c, ins) | ins.ones;
        V v[P][R];
        bool on[P];
        uint64_t e[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            on[p] = step_item(c, p, ps) < nitems;
            e[p] = tb + (ec + at(p));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[p][r].x = v[p][r].y = T(0);
                if (on[p]) v[p][r] = ldnt(amp + e[p] + hoff[r]);
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            V y[R], z[R];  // products with the real and with the imaginary parts of m: two short sums
#pragma unroll
            for (int r = 0; r < R; ++r) y[r].x = y[r].y = z[r].x = z[r].y = T(0);
#pragma unroll
            for (int x = 0; x < X; ++x)
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    // every lane of a wave takes part, also those past the end
                    const T ax = x ? lane_across(v[p][s].x, src[x]) : v[p][s].x;
                    const T ay = x ? lane_across(v[p][s].y, src[x]) : v[p][s].y;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        y[r].x = cr[r][x][s] * ax + y[r].x;
                        z[r].x = ci[r][x][s] * ay + z[r].x;
                        y[r].y = cr[r][x][s] * ay + y[r].y;
                        z[r].y = ci[r][x][s] * ax + z[r].y;
                    }
                }
            if (!on[p]) continue;
            const bool ok = (e[p] & lowmask) == lowmask;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                V o;
                o.x = ok ? y[r].x - z[r].x : v[p][r].x;
                o.y = ok ? y[r].y + z[r].y : v[p][r].y;
                stnt(amp + e[p] + hoff[r], o);
            }
        }
    }
}

// k = 4 and 5 on the matrix cores: a wave takes 16 groups at a time as the
// columns of a D x 16 matrix.  Lane (g, q) = (lane & 15, lane >> 4) holds the
// members 4 s + q of group g, which is both the B operand of step s and, with
// the rows of m in the order below, the place where the products come out, so
// amplitudes go from memory to the matrix cores and back without passing
// through LDS.  m stays in registers for the whole launch (Re and Im apart).
// The two lowest targets select q, so that a load of a wave covers
// consecutive amplitudes as far as the targets allow; where lines are shared
// between the loads of a wave (targets within a line) the caches hold them:
// plain loads there, non-temporal ones else.
//
// One thread per group held 2^k amplitudes and waited for the matrix row by
// row: k = 5 on 25 qubits in complex128 took 620 us on high qubits and 1,414
// us on qubits 0..4, so 207 and 217; memory alone needs about 180 us, the
// multiply-adds 110.
typedef double Acc64 __attribute__((ext_vector_type(4)));
typedef float Acc32 __attribute__((ext_vector_type(4)));
template <typename T> struct MfmaAcc;
template <> struct MfmaAcc<double> { using type = Acc64; };
template <> struct MfmaAcc<float> { using type = Acc32; };

__device__ __forceinline__ Acc64 mfma(double a, double b, Acc64 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Acc32 mfma(float a, float b, Acc32 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <typename T, int K, bool NT>
__global__ __launch_bounds__(kBlock, 2) void k_group_mfma(typename C2<T>::type* __restrict__ amp, uint64_t ngroups,
                                                          BitInsert ins, GroupBits<K> gb, uint64_t lowmask,
                                                          const T* __restrict__ m)
{
    using V = typename C2<T>::type;
    using Acc = typename MfmaAcc<T>::type;
    constexpr int D = 1 << K, S = D / 4, B = D / 16;
    const int lane = threadIdx.x & 63, g = lane & 15, q = lane >> 4;
    // Operand rows: result element r of lane (g, q) in block b is row 4 q + r
    // of the block in single precision and row q + 4 r in double; it has to be
    // member 4 (r + 4 b) + q.
    T ur[B][S], ui[B][S];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int row = sizeof(T) == 8 ? 16 * b + g : 16 * b + 4 * (g & 3) + (g >> 2);
            const T* e = m + 2 * (row * D + 4 * s + q);
            ur[b][s] = e[0];
            ui[b][s] = e[1];
        }
    uint64_t off[S];
#pragma unroll
    for (int s = 0; s < S; ++s) off[s] = group_off<K>(gb, 4 * s);
    const bool on = (uint64_t)g < ngroups;  // a register of fewer than 16 groups is one set
    const uint64_t le = deposit(on ? g : 0, ins) + ((q & 1) ? gb.tbit[0] : 0) + ((q & 2) ? gb.tbit[1] : 0);
    const uint64_t nsets = (ngroups + 15) / 16, nw = (uint64_t)gridDim.x * (kBlock / 64);
    uint64_t set = (uint64_t)blockIdx.x * (kBlock / 64) + (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (set >= nsets) return;
    auto load = [&](const V* p) { return NT ? ldnt(p) : *p; };
    uint64_t e = le + (deposit(set * 16, ins) | ins.ones);
    V x[S];
#pragma unroll
    for (int s = 0; s < S; ++s) x[s] = load(amp + e + off[s]);
    for (;;) {
        // the next set's amplitudes, in flight during the products
        const uint64_t next = set + nw;
        uint64_t ne = e;
        V nx[S];
        if (next < nsets) ne = le + (deposit(next * 16, ins) | ins.ones);
#pragma unroll
        for (int s = 0; s < S; ++s) nx[s] = x[s];
        if (next < nsets) {
#pragma unroll
            for (int s = 0; s < S; ++s) nx[s] = load(amp + ne + off[s]);
        }
        // the two products of each part apart: half as long a chain of sums
        // (smaller rounding errors) and independent accumulators
        Acc re[B], im[B], re2[B], im2[B];
#pragma unroll
        for (int b = 0; b < B; ++b) re[b] = im[b] = re2[b] = im2[b] = Acc{T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int b = 0; b < B; ++b) {
                re[b] = mfma(ur[b][s], x[s].x, re[b]);
                im[b] = mfma(ur[b][s], x[s].y, im[b]);
                re2[b] = mfma(ui[b][s], x[s].y, re2[b]);
                im2[b] = mfma(ui[b][s], x[s].x, im2[b]);
            }
        const bool ok = (e & lowmask) == lowmask;
        if (on) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                V y;
                y.x = ok ? re[s >> 2][s & 3] - re2[s >> 2][s & 3] : x[s].x;
                y.y = ok ? im[s >> 2][s & 3] + im2[s >> 2][s & 3] : x[s].y;
                if (NT) stnt(amp + e + off[s], y);
                else amp[e + off[s]] = y;
            }
        }
        if (next >= nsets) return;
        set = next;
        e = ne;
#pragma unroll
        for (int s = 0; s < S; ++s) x[s] = nx[s];
    }
}

// U on two qubits of a density matrix: U on the row bits, then conj(U) on the
// column bits, in one pass.  Lanes and members as in k_group_mfma: q are the row
// bits and s the column bits, so the rows are a product of the matrix cores with
// U on the diagonal blocks (the zeros add nothing), and the columns one within
// the lane.  As one 16 x 16 product conj(U) (x) U every entry was rounded once
// more and the sums were four times as long: error of a random U on 7 qubits
// 1.67e-16 in complex128 and 8.55e-8 in complex64, 1.28e-16 and 7.81e-8 so (two
// passes: 1.39e-16 and 8.37e-8).  Both row bits select lanes, so a load covers
// whole lines wherever the targets lie, and is non-temporal.  Bound by HBM: 13
// qubits 370 to 393 us in complex128 (5.5 to 5.8 TB/s), 186 to 189 in complex64;
// the 16 x 16 product took 386 to 418 and 202 to 215.
template <typename T>
__global__ __launch_bounds__(kBlock, 2) void k_dm_two(typename C2<T>::type* __restrict__ rho, uint64_t ngroups,
                                                      BitInsert ins, GroupBits<4> gb, MatK<T, 2> u)
{
    using V = typename C2<T>::type;
    using Acc = typename MfmaAcc<T>::type;
    const int lane = threadIdx.x & 63, g = lane & 15, q = lane >> 4;
    T ur[4], ui[4];
    const int row = sizeof(T) == 8 ? g : 4 * (g & 3) + (g >> 2);
    const T er = u.m[2 * (4 * (row & 3) + q)], ei = u.m[2 * (4 * (row & 3) + q) + 1];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        ur[s] = row >> 2 == s ? er : T(0);
        ui[s] = row >> 2 == s ? ei : T(0);
    }
    uint64_t off[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) off[s] = group_off<4>(gb, 4 * s);
    const bool on = (uint64_t)g < ngroups;  // a register of fewer than 16 groups is one set
    const uint64_t le = deposit(on ? g : 0, ins) + ((q & 1) ? gb.tbit[0] : 0) + ((q & 2) ? gb.tbit[1] : 0);
    const uint64_t nsets = (ngroups + 15) / 16, nw = (uint64_t)gridDim.x * (kBlock / 64);
    uint64_t set = (uint64_t)blockIdx.x * (kBlock / 64) + (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (set >= nsets) return;
    uint64_t e = le + deposit(set * 16, ins);
    V x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = ldnt(rho + e + off[s]);
    for (;;) {
        // the next set's entries, in flight during the products
        const uint64_t next = set + nw;
        uint64_t ne = e;
        V nx[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) nx[s] = x[s];
        if (next < nsets) {
            ne = le + deposit(next * 16, ins);
#pragma unroll
            for (int s = 0; s < 4; ++s) nx[s] = ldnt(rho + ne + off[s]);
        }
        Acc re = {T(0), T(0), T(0), T(0)}, im = re, re2 = re, im2 = re;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            re = mfma(ur[s], x[s].x, re);
            im = mfma(ur[s], x[s].y, im);
            re2 = mfma(ui[s], x[s].y, re2);
            im2 = mfma(ui[s], x[s].x, im2);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            x[s].x = re[s] - re2[s];
            x[s].y = im[s] + im2[s];
        }
        V y[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // products with the real and with the imaginary parts of conj(U)
            const T* w = u.m + 8 * c;
            T yx = w[0] * x[0].x, yy = w[0] * x[0].y, zx = w[1] * x[0].y, zy = w[1] * x[0].x;
#pragma unroll
            for (int s = 1; s < 4; ++s) {
                yx = w[2 * s] * x[s].x + yx;
                yy = w[2 * s] * x[s].y + yy;
                zx = w[2 * s + 1] * x[s].y + zx;
                zy = w[2 * s + 1] * x[s].x + zy;
            }
            y[c].x = yx + zx;
            y[c].y = yy - zy;
        }
        __builtin_amdgcn_sched_barrier(0);  // the four stores of a set together
        if (on) {
#pragma unroll
            for (int c = 0; c < 4; ++c) stnt(rho + e + off[c], y[c]);
        }
        if (next >= nsets) return;
        set = next;
        e = ne;
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = nx[s];
    }
}

// ---------------------------------------------------------------------------
// Every amplitude set to (re, im).  Write-only.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_init_fill(typename C2<T>::type* __restrict__ amp, uint64_t len,
                                                      T re, T im)
{
    using V = typename C2<T>::type;
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    const uint64_t ps = (uint64_t)kBlock * U;
    V v;
    v.x = re;
    v.y = im;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i < len) amp[i] = v;
        }
    }
}

// rho[j][k] = psi_j conj(psi_k) at vector index j + 2^N k (Eq. 2 layout).
// Write-only on rho; psi (2^N amplitudes) is read through the caches.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_dm_from_pure(typename C2<T>::type* __restrict__ rho,
                                                         const typename C2<T>::type* __restrict__ psi, int N)
{
    using V = typename C2<T>::type;
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    const uint64_t len = 1ull << (2 * N), low = (1ull << N) - 1;
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i = step_item(c, j, ps);
            if (i >= len) continue;
            const V a = psi[i & low], b = psi[i >> N];
            V v;  // a conj(b)
            v.x = a.x * b.x + a.y * b.y;
            v.y = a.y * b.x - a.x * b.y;
            stnt(rho + i, v);
        }
    }
}

// sum_i conj(a_i) b_i: real part in the first compensated sum, imaginary
// part in the second (products formed in double).
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_inner_sv(const typename C2<T>::type* __restrict__ a,
                                                     const typename C2<T>::type* __restrict__ b, uint64_t len,
                                                     double* partials, double* out)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    NSum s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V x[U], y[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i0 = step_item(c, j, ps);
            const uint64_t i = i0 < len ? i0 : len - 1;
            x[j] = ldnt(a + i);
            y[j] = ldnt(b + i);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const bool in = step_item(c, j, ps) < len;
            const double xr = x[j].x, xi = x[j].y, yr = y[j].x, yi = y[j].y;
            nadd(s0, in ? xr * yr + xi * yi : 0.0);
            nadd(s1, in ? xr * yi - xi * yr : 0.0);
        }
    }
    block_store2(s0, s1, partials, out);
}

// <psi| rho |psi> = sum_{j,k} conj(psi_j) rho[j][k] psi_k over the Eq. 2
// vector (entry j + 2^N k): real part in the first sum, imaginary part (zero
// for a Hermitian rho, up to rounding) in the second.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_fid_dm(const typename C2<T>::type* __restrict__ rho,
                                                   const typename C2<T>::type* __restrict__ psi, int N,
                                                   double* partials, double* out)
{
    static_assert(U % 2 == 0, "the step order alternates two half-runs");
    using V = typename C2<T>::type;
    NSum s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    const uint64_t len = 1ull << (2 * N), low = (1ull << N) - 1;
    const uint64_t ps = (uint64_t)kBlock * U;
    for (uint64_t s = blockIdx.x; step_base(s, ps) < len; s += gridDim.x) {
        const uint64_t c = step_base(s, ps);
        V r[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i0 = step_item(c, j, ps);
            r[j] = ldnt(rho + (i0 < len ? i0 : len - 1));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t i0 = step_item(c, j, ps);
            const uint64_t i = i0 < len ? i0 : len - 1;
            const V pj = psi[i & low], pk = psi[i >> N];
            // t = conj(psi_j) rho psi_k, in double
            const double ar = pj.x, ai = -(double)pj.y, rr = r[j].x, ri = r[j].y, br = pk.x, bi = pk.y;
            const double ur = ar * rr - ai * ri, ui = ar * ri + ai * rr;
            const bool in = i0 < len;
            nadd(s0, in ? ur * br - ui * bi : 0.0);
            nadd(s1, in ? ur * bi + ui * br : 0.0);
        }
    }
    block_store2(s0, s1, partials, out);
}

}  // namespace

// ===========================================================================
// Launchers

// Controls (and phase bits) below kLineBits select within a 128-byte line:
// the pair, group and phase kernels walk those bits too and test them per
// item, so that loads and stores stay contiguous.

// Small registers take kSmallPer items (amplitudes, pairs or 4-groups) per
// thread per step instead of 256 bytes' worth, so that the grid still
// spreads over the CUs (below 512 blocks with the large steps).  The step
// order needs an even count.
constexpr int kSmallPer = 2;

inline bool wide(uint64_t items, int per) { return items >= (uint64_t)512 * kBlock * per; }

// Grid and LDS reserve of a streaming pass over `items` items that touches
// `amps` amplitudes.  From 512 MiB on, which is past the 256 MiB last-level cache,
// the pass runs at the HBM's rate, and that falls when many workgroups read
// and write far apart: a reserve of 64 KB of LDS, never touched, keeps two
// workgroups on a CU, and more of them in the grid let the dispatcher even
// out the CUs.  complex128, 29 qubits: gate on qubit 17 5.4 TB/s with six
// workgroups on a CU, 5.7 with four, 6.0 with two; T gate 5.3 to 5.9;
// complex64, 30 qubits, CNOT 5.6 to 6.2.  A pass that touches only the
// amplitudes whose `ones` bits are set stays at 16 blocks per CU where one of
// these is the address bit of 2 KB: blocks that take one step each, in the
// order of their addresses, keep half the memory channels busy.  complex128,
// 27 qubits, control 7, gate on qubit 14 473 us with the larger grid, 378 so,
// targets 14 and 15 585 and 402; control 8 and 6 365 and 370, 3% slower so.
//
// Of the passes that touch less, from 128 MiB on only those gain that walk
// pairs or a strided part of the state (`mid`): complex128, gate on qubit 6 of
// 23 and 24 51 and 100 us, 47 and 91 so; CNOT of 24 94 and 87; dephasing of
// qubit 2 of 12 95 and 89; targets 4 and 5 of 25, control 7, 162 and 144;
// complex64, 25 qubits, gate on qubit 6 95 and 89; 24 qubits, CNOT 48.5, with
// four workgroups 46.4, with two 49.  The others want the waves: complex64,
// 128 MiB, gate on qubit 4 43 us, 47 with two; complex128, 24 qubits, gate on
// qubit 4 86 and 90, targets 0, 1, 2 91 and 106; phase on qubit 5 of a 12-qubit
// density matrix 61 and 64; dephasing of qubit 5 of 13, complex64, 100 and 140.
// Four as well where `ones` holds the address bit of 4 KB: complex128, 25
// qubits, phase on qubits 8 and 15 56 us, 70 with two.
struct StreamShape {
    dim3 grid;
    unsigned lds;
};
template <typename T>
static StreamShape stream_shape(uint64_t items, int per, uint64_t amps, uint64_t ones = 0, bool mid = false,
                                unsigned lds = 64u << 10)
{
    const uint64_t bytes = amps * 2 * sizeof(T), fixed = ones * 2 * sizeof(T);
    if (bytes < (512ull << 20)) {
        const bool few = mid && bytes >= (128ull << 20);
        const bool four = (fixed & 4096) || (sizeof(T) == 4 && bytes < (256ull << 20));
        return {dim3(grid_for(items, per)), !few ? 0u : four ? 40000u : 64u << 10};
    }
    const uint64_t blocks = items / ((uint64_t)kBlock * per);
    return {dim3((unsigned)std::min(blocks, fixed & 2048 ? kMaxGrid : 4 * kMaxGrid)), lds};
}

template <typename T>
hipError_t launch_init_basis(const Launch& L, void* amp, uint64_t len, uint64_t index, double re, double im)
{
    using V = typename C2<T>::type;
    if (wide(len, kPer<T>))
        hipLaunchKernelGGL((k_init_basis<T, kPer<T>>), dim3(grid_for(len, kPer<T>)), dim3(kBlock), 0, L.stream,
                           (V*)amp, len, index, (T)re, (T)im);
    else
        hipLaunchKernelGGL((k_init_basis<T, kSmallPer>), dim3(grid_for(len, kSmallPer)), dim3(kBlock), 0,
                           L.stream, (V*)amp, len, index, (T)re, (T)im);
    return hipGetLastError();
}

template <typename T, int U, bool DM>
static int hist_rows(const Launch& L, const void* amp, uint64_t count, int shift, uint64_t dim, const MeasureState* st,
                     int mb, double* partials)
{
    const int grid = std::min(grid_for(count, U), kHistBlocks);
    hipLaunchKernelGGL((k_hist<T, U, DM>), dim3(grid), dim3(kBlock), 0, L.stream, (const typename C2<T>::type*)amp, count,
                       shift, dim, st, mb, partials);
    return grid;
}

template <typename T>
hipError_t launch_measure_stage(const Launch& L, const void* amp, int n, bool dm, int shift, const Draws& draws,
                                double* buf, double* res)
{
    using V = typename C2<T>::type;
    double* bins = buf + 2 * 1024 * (size_t)kHistBlocks;
    MeasureState* st = (MeasureState*)(bins + 2 * 1024);
    const uint64_t count = 1ull << (n - shift), dim = 1ull << n;
    const int mb = std::min(10, n - shift);
    const MeasureState* before = shift ? st : nullptr;
    // small registers, and diagonals: the least that a step holds, for more blocks
    int rows = dm                     ? hist_rows<T, 8, true>(L, amp, count, shift, dim, before, mb, buf)
               : wide(count, kPer<T>) ? hist_rows<T, kPer<T>, false>(L, amp, count, shift, dim, before, mb, buf)
                                      : hist_rows<T, 8, false>(L, amp, count, shift, dim, before, mb, buf);
    const double* w = buf;
    // few rows are folded by the walk's own block, which saves a launch
    if (rows > 8) {
        hipLaunchKernelGGL(k_hist_final, dim3(((1 << mb) + 15) / 16), dim3(kBlock), 0, L.stream, buf, rows, 1 << mb, bins);
        w = bins;
        rows = 1;
    }
    hipLaunchKernelGGL(k_measure_walk<T>, dim3(1), dim3(kBlock), 0, L.stream, w, rows, mb, shift, draws,
                       shift + mb == n, dm, n, (const V*)amp, st, res);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_measure_basis(const Launch& L, void* amp, uint64_t len, const double* buf)
{
    using V = typename C2<T>::type;
    const MeasureState* st = (const MeasureState*)(buf + 2 * 1024 * (size_t)kHistBlocks + 2 * 1024);
    if (wide(len, kPer<T>))
        hipLaunchKernelGGL((k_measure_basis<T, kPer<T>>), dim3(grid_for(len, kPer<T>)), dim3(kBlock), 0, L.stream,
                           (V*)amp, len, st);
    else
        hipLaunchKernelGGL((k_measure_basis<T, kSmallPer>), dim3(grid_for(len, kSmallPer)), dim3(kBlock), 0, L.stream,
                           (V*)amp, len, st);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_copy(const Launch& L, void* dst, const void* src, uint64_t len)
{
    using V = typename C2<T>::type;
    if (len * 2 * sizeof(T) < (256ull << 20))
        return hipMemcpyAsync(dst, src, len * 2 * sizeof(T), hipMemcpyDeviceToDevice, L.stream);
    const StreamShape sh = stream_shape<T>(len, kPer<T>, len);
    hipLaunchKernelGGL((k_copy<T, kPer<T>>), sh.grid, dim3(kBlock), sh.lds, L.stream, (V*)dst, (const V*)src, len);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_gate(const Launch& L, void* amp, int nbits, int t, const int* ctrls, int nc,
                       const Mat2<T>& u, int* klass)
{
    using V = typename C2<T>::type;
    if (t < 6 && nbits >= 6) {
        // chunk index = amplitude index >> 6; controls >= 6 are inserted as ones
        int hp[64];
        int nh = 0;
        uint64_t ones = 0;
        uint32_t lowmask = 0;
        for (int k = 0; k < nc; ++k) {
            if (ctrls[k] >= 6) {
                hp[nh++] = ctrls[k] - 6;
                ones |= 1ull << (ctrls[k] - 6);
            } else {
                lowmask |= 1u << ctrls[k];
            }
        }
        const BitInsert hi = make_insert(hp, nh, ones);
        const uint64_t nchunks = 1ull << (nbits - 6 - nh);
        // one wave-row of 64 lanes per chunk, U chunks per wave per step
        const bool big = wide(nchunks * 64, kPer<T>);
        const StreamShape sh = stream_shape<T>(nchunks * 64, big ? kPer<T> : kSmallPer, nchunks * 64, ones << 6);
        switch (t) {
#define QS_LOW(TT) case TT:                                                                              \
    if (big)                                                                                             \
        hipLaunchKernelGGL((k_gate_low<T, TT, kPer<T>>), sh.grid, dim3(kBlock), sh.lds, L.stream, (V*)amp, \
                           nchunks, hi, lowmask, u);                                                     \
    else                                                                                                 \
        hipLaunchKernelGGL((k_gate_low<T, TT, kSmallPer>), sh.grid, dim3(kBlock), 0, L.stream, (V*)amp, \
                           nchunks, hi, lowmask, u);                                                     \
    break;
            QS_LOW(0) QS_LOW(1) QS_LOW(2) QS_LOW(3) QS_LOW(4) QS_LOW(5)
#undef QS_LOW
        }
        if (klass) *klass = QS_K_GATE_LOW;
        return hipGetLastError();
    }
    int pos[64];
    int np = 0;
    uint64_t ones = 0, lowmask = 0;
    for (int k = 0; k < nc; ++k) {
        if (ctrls[k] < kLineBits<T>) {
            lowmask |= 1ull << ctrls[k];
            continue;
        }
        pos[np++] = ctrls[k];
        ones |= 1ull << ctrls[k];
    }
    pos[np] = t;
    const BitInsert ins = make_insert(pos, np + 1, ones);
    const uint64_t npairs = 1ull << (nbits - 1 - np);
    const StreamShape sh = stream_shape<T>(npairs, kPer<T> / 2, 2 * npairs, ones, true);
    if (wide(npairs, kPer<T> / 2))
        hipLaunchKernelGGL((k_gate_pair<T, kPer<T> / 2>), sh.grid, dim3(kBlock), sh.lds, L.stream,
                           (V*)amp, npairs, 1ull << t, ins, lowmask, u);
    else
        hipLaunchKernelGGL((k_gate_pair<T, kSmallPer>), dim3(grid_for(npairs, kSmallPer)), dim3(kBlock), 0,
                           L.stream, (V*)amp, npairs, 1ull << t, ins, lowmask, u);
    if (klass) *klass = QS_K_GATE;
    return hipGetLastError();
}

template <typename T>
hipError_t launch_not(const Launch& L, void* amp, int nbits, int t, const int* ctrls, int nc)
{
    if (t < 6 && nbits >= 6) {
        // the in-wave exchange path of dense gates keeps every access a full
        // line; X costs a few multiply-adds there
        Mat2<T> x;
        for (int k = 0; k < 8; ++k) x.m[k] = (k == 2 || k == 4) ? T(1) : T(0);
        return launch_gate<T>(L, amp, nbits, t, ctrls, nc, x, nullptr);
    }
    using V = typename C2<T>::type;
    int pos[64];
    int np = 0;
    uint64_t ones = 0, lowmask = 0;
    for (int k = 0; k < nc; ++k) {
        if (ctrls[k] < kLineBits<T>) {
            lowmask |= 1ull << ctrls[k];
            continue;
        }
        pos[np++] = ctrls[k];
        ones |= 1ull << ctrls[k];
    }
    pos[np] = t;
    const BitInsert ins = make_insert(pos, np + 1, ones);
    const uint64_t npairs = 1ull << (nbits - 1 - np);
    const StreamShape sh = stream_shape<T>(npairs, kPer<T> / 2, 2 * npairs, ones, true);
    if (wide(npairs, kPer<T> / 2))
        hipLaunchKernelGGL((k_not<T, kPer<T> / 2>), sh.grid, dim3(kBlock), sh.lds, L.stream,
                           (V*)amp, npairs, 1ull << t, ins, lowmask);
    else
        hipLaunchKernelGGL((k_not<T, kSmallPer>), dim3(grid_for(npairs, kSmallPer)), dim3(kBlock), 0, L.stream,
                           (V*)amp, npairs, 1ull << t, ins, lowmask);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_phase(const Launch& L, void* amp, int nbits, uint64_t mask, uint64_t skip,
                        double fre, double fim)
{
    using V = typename C2<T>::type;
    int pos[64];
    int np = 0;
    const uint64_t lowmask = mask & ((1ull << kLineBits<T>) - 1);
    for (int q = kLineBits<T>; q < nbits; ++q)
        if ((mask >> q) & 1) pos[np++] = q;
    const BitInsert ins = make_insert(pos, np, mask & ~lowmask);
    const uint64_t count = 1ull << (nbits - np);
    const StreamShape sh = stream_shape<T>(count, kPer<T>, count, mask, !skip);
    if (wide(count, kPer<T>))
        hipLaunchKernelGGL((k_phase<T, kPer<T>>), sh.grid, dim3(kBlock), sh.lds, L.stream,
                           (V*)amp, count, ins, lowmask, skip, (T)fre, (T)fim);
    else
        hipLaunchKernelGGL((k_phase<T, kSmallPer>), dim3(grid_for(count, kSmallPer)), dim3(kBlock), 0, L.stream,
                           (V*)amp, count, ins, lowmask, skip, (T)fre, (T)fim);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_dm_phase(const Launch& L, void* rho, int N, uint64_t rmask, double fre, double fim)
{
    using V = typename C2<T>::type;
    // qubits within a line: one pass over everything, while the lines that a
    // pass for the rows and one for the columns would leave out are few, or the
    // second launch costs more than the walk over them.  Two passes against
    // one, 13 qubits, complex128 / complex64: qubits 0 and 1 401 us, 362 / 221,
    // 161; 2 and 4 269, 214 / 140, 120; 0, 1 and 12 235, 253 / 118, 118; 2, 4
    // and 5 161, 143 / 82, 106; 2 to 5 82, 128 / 72, 103; 11 qubits, 2 to 5
    // 8.9, 12.5 (64 MiB) / 8.8, 7.0 (32 MiB).
    const uint64_t len = 1ull << (2 * N);
    const int inside = __builtin_popcountll(rmask & ((1ull << kLineBits<T>) - 1));
    const int above = __builtin_popcountll(rmask >> kLineBits<T>);
    if (inside && (above == 0 || (above == 1 && inside == 1) || len * 2 * sizeof(T) <= (32ull << 20))) {
        // complex64 too: its 32 index tests per step cost more than the fewer steps save
        constexpr int U = kPer<double>;
        const bool big = wide(len, U);
        const StreamShape sh = stream_shape<T>(len, big ? U : kSmallPer, len);
        if (big)
            hipLaunchKernelGGL((k_dm_phase<T, U>), sh.grid, dim3(kBlock), sh.lds, L.stream, (V*)rho, len, rmask,
                               rmask << N, (T)fre, (T)fim);
        else
            hipLaunchKernelGGL((k_dm_phase<T, kSmallPer>), sh.grid, dim3(kBlock), 0, L.stream, (V*)rho, len, rmask,
                               rmask << N, (T)fre, (T)fim);
        return hipGetLastError();
    }
    // rows with all bits set gain the phase, columns its conjugate; entries
    // with both keep their value
    const hipError_t e = launch_phase<T>(L, rho, 2 * N, rmask, rmask << N, fre, fim);
    return e != hipSuccess ? e : launch_phase<T>(L, rho, 2 * N, rmask << N, rmask, fre, -fim);
}

template <typename T>
hipError_t launch_dm_gate(const Launch& L, void* rho, int N, int t, const int* ctrls, int nc,
                          const Mat2<T>& u)
{
    using V = typename C2<T>::type;
    const int pos[2] = {t + N, t};
    const bool low = t < kLineBits<T>;
    const BitInsert ins = make_insert(pos, low ? 1 : 2, 0);
    uint64_t rmask = 0;
    for (int k = 0; k < nc; ++k) rmask |= 1ull << ctrls[k];
    // items: 4-groups, or for a low target the pairs (column bit 0, 1) of a row
    const uint64_t items = 1ull << (2 * N - (low ? 1 : 2));
    const uint64_t tb = 1ull << t, cb = 1ull << (t + N);
    constexpr int G = kPer<T> / 4, G2 = kPer<T> / 2;
    const bool big = wide(items, low ? G2 : G);
    const StreamShape sh = stream_shape<T>(items, !big ? kSmallPer : low ? G2 : G,
                                             (nc ? 3ull : 4ull) << (2 * N - 2), 0, sizeof(T) == 8);
#define QS_DM(K)                                                                                              \
    hipLaunchKernelGGL(K, sh.grid, dim3(kBlock), sh.lds, L.stream, (V*)rho, items, tb, cb, ins, rmask, rmask << N, u)
    if (low) {
        if (big) QS_DM((k_dm_gate_low<T, G2>));
        else QS_DM((k_dm_gate_low<T, kSmallPer>));
    } else {
        if (big) QS_DM((k_dm_gate<T, G>));
        else QS_DM((k_dm_gate<T, kSmallPer>));
    }
#undef QS_DM
    return hipGetLastError();
}

template <typename T, int CH>
static hipError_t dm_channel(const Launch& L, void* rho, int N, int t, double p0, double p1, double f)
{
    using V = typename C2<T>::type;
    const int pos[2] = {t + N, t};
    // dephasing on the top qubit within a line leaves one half of each line
    // alone, which pays in the cache: complex64, qubit 3 of 12 48 us by whole
    // lines, 43 so; of 13 173 and 174; complex128, qubit 2 of 12 89 and 90
    const bool halves = CH == QS_DEPHASING && sizeof(T) == 4 && t == kHalfBits<T> && N <= 12;
    const bool low = t < kLineBits<T> && !halves;
    const BitInsert ins = make_insert(pos, low ? 1 : 2, 0);
    const uint64_t items = 1ull << (2 * N - (low ? 1 : 2));
    const uint64_t tb = 1ull << t, cb = 1ull << (t + N);
    constexpr int G = kPer<T> / 4, G2 = kPer<T> / 2;
    // a group of a dephasing holds two entries, not four: twice the groups before
    // the large steps (complex64, 11 qubits, qubit 5: 6.8 us with them, 5.8 without)
    const bool big = wide(items, low ? G2 : CH == QS_DEPHASING ? 2 * G : G);
    const StreamShape sh = stream_shape<T>(items, !big ? kSmallPer : low ? G2 : G,
                                             (CH == QS_DEPHASING && !low ? 1ull : 2ull) << (2 * N - 1),
                                             0, sizeof(T) == 8);
#define QS_CH(K) hipLaunchKernelGGL(K, sh.grid, dim3(kBlock), sh.lds, L.stream, (V*)rho, items, tb, cb, ins, p0, p1, f)
    if (low) {
        if (big) QS_CH((k_dm_channel_low<T, CH, G2>));
        else QS_CH((k_dm_channel_low<T, CH, kSmallPer>));
    } else {
        if (big) QS_CH((k_dm_channel<T, CH, G>));
        else QS_CH((k_dm_channel<T, CH, kSmallPer>));
    }
#undef QS_CH
    return hipGetLastError();
}

template <typename T>
hipError_t launch_dm_channel(const Launch& L, void* rho, int N, int t, int channel, double p)
{
    switch (channel) {
    case QS_DEPHASING: return dm_channel<T, QS_DEPHASING>(L, rho, N, t, 0.0, 0.0, 1.0 - 2.0 * p);
    case QS_DEPOLARISING:
        return dm_channel<T, QS_DEPOLARISING>(L, rho, N, t, 1.0 - 2.0 * p / 3.0, 2.0 * p / 3.0, 1.0 - 4.0 * p / 3.0);
    default: return dm_channel<T, QS_DAMPING>(L, rho, N, t, p, 1.0 - p, sqrt(1.0 - p));
    }
}

// Up to this many items one block does the whole sum, and there is one launch
// instead of two.  These are two steps of kAlonePer loads per thread, since the
// step order leaves out every other half-run, and half of the loads lie past
// the end: they repeat the last item, from the cache.  Beyond, many
// blocks and a fold are faster: 13 qubits complex64 3.3 us and 2.4 against
// 9.1 by one block.
constexpr int kAlonePer = 8;
constexpr uint64_t kAlone = kAlonePer * kBlock;

// The step of a sum over `items` items, `per` for large ones, and its grid.
struct SumShape {
    int per, grid;
};
static SumShape sum_shape(uint64_t items, int per)
{
    if (items <= kAlone) return {kAlonePer, 1};
    const int p = wide(items, per) ? per : kSmallPer;
    return {p, std::min(grid_for(items, p), kReduceBlocks)};
}

static hipError_t reduce_final(const Launch& L, const double* partials, int grid, double* dev_out)
{
    if (grid > 1) hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(kBlock), 0, L.stream, partials, grid, dev_out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_prob_sv(const Launch& L, const void* amp, int nbits, int q, double* partials,
                          double* dev_out)
{
    using V = typename C2<T>::type;
    const uint64_t len = 1ull << nbits;
    const SumShape sh = sum_shape(len, kPer<T>);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(sh.grid), dim3(kBlock), 0, L.stream, (const V*)amp, len, q, partials, dev_out);
    };
    if (sh.per == kAlonePer) run(k_prob_sv<T, kAlonePer>);
    else if (sh.per == kSmallPer) run(k_prob_sv<T, kSmallPer>);
    else run(k_prob_sv<T, kPer<T>>);
    return reduce_final(L, partials, sh.grid, dev_out);
}

template <typename T>
hipError_t launch_prob_half_sv(const Launch& L, const void* amp, int nbits, int q, int outcome, double* partials,
                               double* dev_out)
{
    using V = typename C2<T>::type;
    const uint64_t half = 1ull << (nbits - 1);
    const SumShape sh = sum_shape(half, kPer<T>);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(sh.grid), dim3(kBlock), 0, L.stream, (const V*)amp, half, q, outcome, partials, dev_out);
    };
    if (sh.per == kAlonePer) run(k_prob_half_sv<T, kAlonePer>);
    else if (sh.per == kSmallPer) run(k_prob_half_sv<T, kSmallPer>);
    else run(k_prob_half_sv<T, kPer<T>>);
    return reduce_final(L, partials, sh.grid, dev_out);
}

template <typename T>
hipError_t launch_prob_dm(const Launch& L, const void* rho, int N, int q, double* partials,
                          double* dev_out)
{
    using V = typename C2<T>::type;
    const uint64_t dim = 1ull << N;
    const int grid = std::min(grid_for(dim, 1), kReduceBlocks);
    hipLaunchKernelGGL(k_prob_dm<T>, dim3(grid), dim3(kBlock), 0, L.stream, (const V*)rho, dim, q,
                       partials, dev_out);
    return reduce_final(L, partials, grid, dev_out);
}

template <typename T>
hipError_t launch_collapse_sv(const Launch& L, void* amp, int nbits, int q, int outcome, double scale)
{
    using V = typename C2<T>::type;
    const uint64_t len = 1ull << nbits;
    const StreamShape sh = stream_shape<T>(len, kPer<T>, len);
    if (wide(len, kPer<T>))
        hipLaunchKernelGGL((k_collapse_sv<T, kPer<T>>), sh.grid, dim3(kBlock), sh.lds, L.stream,
                           (V*)amp, len, q, outcome, scale);
    else
        hipLaunchKernelGGL((k_collapse_sv<T, kSmallPer>), dim3(grid_for(len, kSmallPer)), dim3(kBlock), 0, L.stream,
                           (V*)amp, len, q, outcome, scale);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_collapse_dm(const Launch& L, void* rho, int N, int q, int outcome, double scale)
{
    using V = typename C2<T>::type;
    const uint64_t len = 1ull << (2 * N);
    const StreamShape sh = stream_shape<T>(len, kPer<T>, len);
    if (wide(len, kPer<T>))
        hipLaunchKernelGGL((k_collapse_dm<T, kPer<T>>), sh.grid, dim3(kBlock), sh.lds, L.stream,
                           (V*)rho, len, q, N, outcome, scale);
    else
        hipLaunchKernelGGL((k_collapse_dm<T, kSmallPer>), dim3(grid_for(len, kSmallPer)), dim3(kBlock), 0, L.stream,
                           (V*)rho, len, q, N, outcome, scale);
    return hipGetLastError();
}

// The group kernels keep half as much in flight per lane as the others, and
// twice the workgroups on a CU: complex128, 25 qubits, targets 10 and 20:
// 204 us with five, 214 with two; 0, 1, 2: 192 and 225.  With the smaller grid
// of a control at the address bit of 2 KB, all that fit (complex64, 27 qubits,
// targets 4 and 5, control 8: 224 us, 242 with five).  From 2 GiB on two, but
// where targets lie within a line: 28 qubits, complex64, targets 17, 25 and 27
// 853 us with five, 737 with two, 18 and 19 767 and 700; 26 qubits 189 and 192,
// 174 and 175; 0, 1 and 2 of 28 747 and 814.
template <typename T>
static unsigned group_lds(uint64_t ones, uint64_t amps = 0)
{
    return (ones * 2 * sizeof(T)) & 2048 ? 0 : amps * 2 * sizeof(T) >= (2ull << 30) ? 64u << 10 : 32000;
}

// Sorts the targets, with the bits of the matrix index in the same order.
template <typename T>
static void sort_targets(const int* targets, int k, const std::complex<double>* m, int* st, T* sm)
{
    const int d = 1 << k;
    int order[5];
    for (int j = 0; j < k; ++j) order[j] = j;
    std::sort(order, order + k, [&](int a, int b) { return targets[a] < targets[b]; });
    int from[32];  // matrix index of member r
    for (int r = 0; r < d; ++r) {
        from[r] = 0;
        for (int j = 0; j < k; ++j)
            if ((r >> j) & 1) from[r] |= 1 << order[j];
    }
    for (int j = 0; j < k; ++j) st[j] = targets[order[j]];
    for (int r = 0; r < d; ++r)
        for (int c = 0; c < d; ++c) {
            sm[2 * (r * d + c)] = (T)m[from[r] * d + from[c]].real();
            sm[2 * (r * d + c) + 1] = (T)m[from[r] * d + from[c]].imag();
        }
}

template <typename T, int K, int L>
static hipError_t group_lane(const Launch& L0, void* amp, int nbits, const int* st, const int* pos, int np, uint64_t ones,
                             uint64_t lowmask, const GroupBits<K>& gb, const MatK<T, K>& mk)
{
    using V = typename C2<T>::type;
    // 128 bytes per lane in flight, less where the 8 x 8 rows fill the registers
    constexpr int P = std::max(2, (sizeof(T) == 8 ? (K == 3 && L == 3 ? 4 : 8) : 16) >> (K - L));
    int ip[64];
    int ni = 0;
    for (int j = L; j < K; ++j) ip[ni++] = st[j];
    for (int j = 0; j < np; ++j) ip[ni++] = pos[j];
    const uint64_t nitems = 1ull << (nbits - ni);
    const BitInsert ins = make_insert(ip, ni, ones);
    const StreamShape sh = stream_shape<T>(nitems, P, nitems << (K - L), ones, K == 2 && sizeof(T) == 8,
                                           group_lds<T>(ones));
    if (wide(nitems, P))
        hipLaunchKernelGGL((k_group_lane<T, K, L, P>), sh.grid, dim3(kBlock), sh.lds, L0.stream, (V*)amp,
                           nitems, ins, gb, lowmask, mk);
    else
        hipLaunchKernelGGL((k_group_lane<T, K, L, kSmallPer>), dim3(grid_for(nitems, kSmallPer)), dim3(kBlock), 0,
                           L0.stream, (V*)amp, nitems, ins, gb, lowmask, mk);
    return hipGetLastError();
}

template <typename T, int K>
static hipError_t group_small(const Launch& L, void* amp, int nbits, const int* targets, const int* ctrls, int nc,
                              const std::complex<double>* m)
{
    using V = typename C2<T>::type;
    int st[5], pos[64];
    MatK<T, K> mk;
    sort_targets<T>(targets, K, m, st, mk.m);
    int np = 0, nlow = 0;
    uint64_t ones = 0, lowmask = 0;
    for (int j = 0; j < nc; ++j) {
        if (ctrls[j] < kLineBits<T>) {
            lowmask |= 1ull << ctrls[j];
            continue;
        }
        pos[np++] = ctrls[j];
        ones |= 1ull << ctrls[j];
    }
    GroupBits<K> gb;
    for (int j = 0; j < K; ++j) {
        gb.tbit[j] = 1ull << st[j];
        nlow += st[j] < kLineBits<T>;
    }
    // cross-lane reads need every lane of a group's 2^nlow active: the item
    // count is a power of two of at least that
    switch (nlow) {
    case 1: return group_lane<T, K, 1>(L, amp, nbits, st, pos, np, ones, lowmask, gb, mk);
    case 2: return group_lane<T, K, 2>(L, amp, nbits, st, pos, np, ones, lowmask, gb, mk);
    case 3:
        if constexpr (K == 3) return group_lane<T, K, 3>(L, amp, nbits, st, pos, np, ones, lowmask, gb, mk);
        break;
    default: break;
    }
    for (int j = 0; j < K; ++j) pos[np++] = st[j];
    const BitInsert ins = make_insert(pos, np, ones);
    const uint64_t ngroups = 1ull << (nbits - np);
    constexpr int P = std::max(1, (sizeof(T) == 8 ? 8 : 16) >> K);
    const StreamShape sh = stream_shape<T>(ngroups, P, ngroups << K, ones, K == 2 && sizeof(T) == 8,
                                           group_lds<T>(ones, ngroups << K));
    if (wide(ngroups, P))
        hipLaunchKernelGGL((k_group_gate<T, K, P>), sh.grid, dim3(kBlock), sh.lds, L.stream, (V*)amp,
                           ngroups, ins, gb, lowmask, mk);
    else
        hipLaunchKernelGGL((k_group_gate<T, K, 1>), dim3(grid_for(ngroups, 1)), dim3(kBlock), 0, L.stream, (V*)amp,
                           ngroups, ins, gb, lowmask, mk);
    return hipGetLastError();
}

// Two blocks per CU: as fast as more in complex128, faster in complex64 (k = 5
// on 25 qubits 118 us; with four 150).
constexpr uint64_t kMfmaGrid = 256 * 2;

template <typename T, int K>
static hipError_t group_mfma(const Launch& L, void* amp, int nbits, const int* targets, const int* ctrls, int nc,
                             const std::complex<double>* m, T* dev_m)
{
    using V = typename C2<T>::type;
    constexpr int D = 1 << K;
    int st[5], pos[64];
    std::vector<T> sm(2 * D * D);
    sort_targets<T>(targets, K, m, st, sm.data());
    // from pageable memory the copy has left `sm` when the call returns
    const hipError_t e = hipMemcpyAsync(dev_m, sm.data(), sm.size() * sizeof(T), hipMemcpyHostToDevice, L.stream);
    if (e != hipSuccess) return e;
    int np = 0;
    uint64_t ones = 0, lowmask = 0;
    GroupBits<K> gb;
    for (int j = 0; j < K; ++j) {
        gb.tbit[j] = 1ull << st[j];
        pos[np++] = st[j];
    }
    for (int j = 0; j < nc; ++j) {
        if (ctrls[j] < kLineBits<T>) {
            lowmask |= 1ull << ctrls[j];
            continue;
        }
        pos[np++] = ctrls[j];
        ones |= 1ull << ctrls[j];
    }
    const BitInsert ins = make_insert(pos, np, ones);
    const uint64_t ngroups = 1ull << (nbits - np);
    const uint64_t blocks = (ngroups + 63) / 64;  // four waves of 16 groups
    const dim3 grid((unsigned)std::min(blocks, kMfmaGrid));
    if (st[0] < kLineBits<T>)
        hipLaunchKernelGGL((k_group_mfma<T, K, false>), grid, dim3(kBlock), 0, L.stream, (V*)amp, ngroups, ins, gb, lowmask,
                           dev_m);
    else
        hipLaunchKernelGGL((k_group_mfma<T, K, true>), grid, dim3(kBlock), 0, L.stream, (V*)amp, ngroups, ins, gb, lowmask,
                           dev_m);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_dm_two(const Launch& L, void* rho, int N, const int* targets, const std::complex<double>* m)
{
    using V = typename C2<T>::type;
    int st[2];
    MatK<T, 2> u;
    sort_targets<T>(targets, 2, m, st, u.m);
    const int pos[4] = {st[0], st[1], st[0] + N, st[1] + N};
    GroupBits<4> gb;
    for (int j = 0; j < 4; ++j) gb.tbit[j] = 1ull << pos[j];
    const BitInsert ins = make_insert(pos, 4, 0);
    const uint64_t ngroups = 1ull << (2 * N - 4);
    const dim3 grid((unsigned)std::min<uint64_t>((ngroups + 63) / 64, kMfmaGrid));
    hipLaunchKernelGGL(k_dm_two<T>, grid, dim3(kBlock), 0, L.stream, (V*)rho, ngroups, ins, gb, u);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_group_gate(const Launch& L, void* amp, int nbits, const int* targets, int k, const int* ctrls,
                             int nc, const std::complex<double>* m, T* dev_m)
{
    switch (k) {
    case 1: {
        Mat2<T> u;
        for (int i = 0; i < 4; ++i) {
            u.m[2 * i] = (T)m[i].real();
            u.m[2 * i + 1] = (T)m[i].imag();
        }
        return launch_gate<T>(L, amp, nbits, targets[0], ctrls, nc, u, nullptr);
    }
    case 2: return group_small<T, 2>(L, amp, nbits, targets, ctrls, nc, m);
    case 3: return group_small<T, 3>(L, amp, nbits, targets, ctrls, nc, m);
    case 4: return group_mfma<T, 4>(L, amp, nbits, targets, ctrls, nc, m, dev_m);
    case 5: return group_mfma<T, 5>(L, amp, nbits, targets, ctrls, nc, m, dev_m);
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_init_fill(const Launch& L, void* amp, uint64_t len, double re, double im)
{
    using V = typename C2<T>::type;
    if (wide(len, kPer<T>))
        hipLaunchKernelGGL((k_init_fill<T, kPer<T>>), dim3(grid_for(len, kPer<T>)), dim3(kBlock), 0, L.stream,
                           (V*)amp, len, (T)re, (T)im);
    else
        hipLaunchKernelGGL((k_init_fill<T, kSmallPer>), dim3(grid_for(len, kSmallPer)), dim3(kBlock), 0,
                           L.stream, (V*)amp, len, (T)re, (T)im);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_dm_from_pure(const Launch& L, void* rho, int N, const void* psi)
{
    using V = typename C2<T>::type;
    const uint64_t len = 1ull << (2 * N);
    if (wide(len, kPer<T>))
        hipLaunchKernelGGL((k_dm_from_pure<T, kPer<T>>), dim3(grid_for(len, kPer<T>)), dim3(kBlock), 0,
                           L.stream, (V*)rho, (const V*)psi, N);
    else
        hipLaunchKernelGGL((k_dm_from_pure<T, kSmallPer>), dim3(grid_for(len, kSmallPer)), dim3(kBlock), 0,
                           L.stream, (V*)rho, (const V*)psi, N);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_inner_sv(const Launch& L, const void* a, const void* b, int nbits, double* partials,
                           double* dev_out)
{
    using V = typename C2<T>::type;
    const uint64_t len = 1ull << nbits;
    constexpr int U = kPer<T> / 2;  // two streams per step
    const SumShape sh = sum_shape(len, U);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(sh.grid), dim3(kBlock), 0, L.stream, (const V*)a, (const V*)b, len, partials, dev_out);
    };
    if (sh.per == kAlonePer) run(k_inner_sv<T, kAlonePer>);
    else if (sh.per == kSmallPer) run(k_inner_sv<T, kSmallPer>);
    else run(k_inner_sv<T, U>);
    return reduce_final(L, partials, sh.grid, dev_out);
}

template <typename T>
hipError_t launch_fid_dm(const Launch& L, const void* rho, int N, const void* psi, double* partials,
                         double* dev_out)
{
    using V = typename C2<T>::type;
    const uint64_t len = 1ull << (2 * N);
    const SumShape sh = sum_shape(len, kPer<T>);
    const auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(sh.grid), dim3(kBlock), 0, L.stream, (const V*)rho, (const V*)psi, N, partials, dev_out);
    };
    if (sh.per == kAlonePer) run(k_fid_dm<T, kAlonePer>);
    else if (sh.per == kSmallPer) run(k_fid_dm<T, kSmallPer>);
    else run(k_fid_dm<T, kPer<T>>);
    return reduce_final(L, partials, sh.grid, dev_out);
}

#define QS_INSTANTIATE(T)                                                                              \
    template hipError_t launch_init_basis<T>(const Launch&, void*, uint64_t, uint64_t, double, double); \
    template hipError_t launch_measure_stage<T>(const Launch&, const void*, int, bool, int, const Draws&, double*, \
                                                double*);                                              \
    template hipError_t launch_measure_basis<T>(const Launch&, void*, uint64_t, const double*);        \
    template hipError_t launch_copy<T>(const Launch&, void*, const void*, uint64_t);                   \
    template hipError_t launch_gate<T>(const Launch&, void*, int, int, const int*, int, const Mat2<T>&, \
                                       int*);                                                          \
    template hipError_t launch_not<T>(const Launch&, void*, int, int, const int*, int);                \
    template hipError_t launch_phase<T>(const Launch&, void*, int, uint64_t, uint64_t, double, double); \
    template hipError_t launch_dm_phase<T>(const Launch&, void*, int, uint64_t, double, double);       \
    template hipError_t launch_dm_gate<T>(const Launch&, void*, int, int, const int*, int,             \
                                          const Mat2<T>&);                                             \
    template hipError_t launch_dm_channel<T>(const Launch&, void*, int, int, int, double);             \
    template hipError_t launch_prob_sv<T>(const Launch&, const void*, int, int, double*, double*);     \
    template hipError_t launch_prob_half_sv<T>(const Launch&, const void*, int, int, int, double*, double*); \
    template hipError_t launch_prob_dm<T>(const Launch&, const void*, int, int, double*, double*);     \
    template hipError_t launch_collapse_sv<T>(const Launch&, void*, int, int, int, double);            \
    template hipError_t launch_collapse_dm<T>(const Launch&, void*, int, int, int, double); \
    template hipError_t launch_dm_two<T>(const Launch&, void*, int, const int*, const std::complex<double>*); \
    template hipError_t launch_group_gate<T>(const Launch&, void*, int, const int*, int, const int*, int, \
                                             const std::complex<double>*, T*);                         \
    template hipError_t launch_init_fill<T>(const Launch&, void*, uint64_t, double, double);           \
    template hipError_t launch_dm_from_pure<T>(const Launch&, void*, int, const void*);                \
    template hipError_t launch_inner_sv<T>(const Launch&, const void*, const void*, int, double*, double*); \
    template hipError_t launch_fid_dm<T>(const Launch&, const void*, int, const void*, double*, double*);

QS_INSTANTIATE(double)
QS_INSTANTIATE(float)

hipError_t launch_sum_columns(const Launch& L, const double* part, int rows, int cols, double* out)
{
    if (rows < 1 || cols < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_sum_columns, dim3((cols + 63) / 64), dim3(64), 0, L.stream, part, rows, cols, out);
    return hipGetLastError();
}

}  // namespace qs
