// Gate fusion for state vectors: a run of gates whose targets lie in a set S
// of K qubits is applied to every 2^K-amplitude tile (all amplitudes that
// agree on the qubits outside S) in one read and one write of HBM -- the
// GPU form of the cache blocking / gate fusion described in Sec. II.B.
//
// Tile layout.  A workgroup of 2^TB threads holds a tile of 2^K = 2^(TB+RB)
// amplitudes in registers, 2^RB per thread.  At any moment each local qubit
// of the tile is either a "thread bit" (selects the thread) or a "register
// bit" (selects the register inside the thread).  A gate whose target is a
// register bit is applied by every thread to its own registers; controls and
// diagonal phases may sit anywhere, since a thread knows the value of its
// thread bits and of the qubits outside S (fixed per tile).  When the next
// gates target thread bits, the tile is re-laid out through LDS (one write
// and one read of 2^K amplitudes) so that those qubits become register
// bits.  Lanes 0..63 always cover global qubits 0..5 when the tile is read
// from or written to HBM, so every global access is a contiguous 64-element
// run per wavefront.
//
// LDS addresses are a linear map over GF(2) of the local index (an XOR
// swizzle chosen per re-layout so that the 8 lanes of a 128-byte LDS cycle
// hit distinct banks in both the writing and the reading layout).  Each
// layout is handed to the kernel as the images of single thread / register
// bits, so the kernel only XORs precomputed values.
#include <string.h>

#include <algorithm>
#include <complex>
#include <memory>
#include <vector>

#include "qs_device.h"
#include "qs_host.h"
#include "qs_plan.h"

namespace qs {
namespace {

constexpr int kTBMax = 10;
constexpr int kRBMax = 5;

// One register layout of a pass, 32 words: every wave loads it as one word
// per lane and reads the words back with v_readlane.
struct alignas(16) FPhase {
    uint32_t wthr[kTBMax], wreg[kRBMax];  // LDS images of the layout being left
    uint32_t rthr[kTBMax], rreg[kRBMax];  // LDS images of the layout entered
    uint32_t op_begin, op_end;
};
static_assert(sizeof(FPhase) == 32 * sizeof(uint32_t), "a phase is one word for each of 32 lanes");

struct FPass {
    int nphases;
    int final_transpose;  // 1: re-lay out to the store layout before storing
    uint64_t ld_thr[kTBMax], ld_reg[kRBMax];  // HBM offsets of the load layout
    uint64_t st_thr[kTBMax], st_reg[kRBMax];  // HBM offsets of the store layout
    BitInsert outside;                        // inserts zeros at the tile's qubits
    uint32_t first_op[kPhMax + 1];            // of each phase among the FOps, and the end of the last
    FPhase ph[kPhMax + 1];                    // the phases, then (final_transpose) the store layout
};

// Host form of an op.
struct FOp {
    int kind;        // op code, below
    int rb;          // target register bit (dense / not / core)
    uint32_t rmask;  // register bits that must be 1
    uint32_t tmask;  // thread-index bits that must be 1
    uint64_t gmask;  // global qubits outside the tile that must be 1
    double m[8];     // dense matrix, phase factor in m[0], m[1], or core coefficient k in m[0], m[1]
    uint32_t aux;    // 4x4 ops: entry of the 4x4 matrix table
    bool cx;         // kNot with a register control: the phase of both bits follows
    bool lane;       // kPhase: a phase of lanes in the planned layout (phase_case)
};

// Device form: one or more FOps that a wave runs under one dispatch, in the
// order cores, NOT, phase, signs (bundle() below).
//   code  class bits | tmask << 16
//   sub   one bit of the class's list (NOT, 4x4, other)
//   multi bits 0..4 in-place cores on register bits 0..4, 5..9 exchanged cores, 10..14 rmask,
//         15..19 signs of single bits, 20..29 signs of pairs
//   ph    the phase's register bits: 0..4 single bits, 5..14 pairs, kPhAny rmask, kPhAll none
//   m     the core coefficient of register bit b at 2 b; at 10 a phase factor; the matrix of kOther
//         at 0; the table entry of a 4x4 in the bits of m[10]
template <typename T>
struct alignas(16) FRec {
    uint32_t code, sub, multi, ph;
    uint64_t gmask;
    T m[12];
};

// Device form of one FOp, for passes that run op by op.
template <typename T>
struct alignas(16) FOne {
    uint32_t kind, rmask, tmask, aux;
    uint64_t gmask;
    uint32_t cx, pad;
    T m[8];
};

// Op kinds: class << 5 | sub.  Register-bit pairs (b1 < b2) are numbered in
// lexical order.
//   kCoreA, sub rb     unit-diagonal core, amplitudes in place: (a, b) <- (a + k b, b - conj(k) a)
//   kCoreB, sub rb     core with the pair exchanged: (a, b) <- (k a + b, a - conj(k) b)
//   kNot, sub 6 rb + c NOT on rb where register bit c is 1 (c = 5: everywhere)
//   kNotM, sub rb      NOT with any register and thread-bit controls
//   kPhase, sub        phase m[0] + i m[1]: sub 0 no register bit, 1 + b where bit b is 1,
//                      6 + pair where both are 1, 16 any rmask; thread-bit controls in tmask
//   kSign, sub         the phase of an angle of pi or -pi: a sign, subs as kPhase up to 15
//   kDense4, sub pair  4x4 on register bits, matrix in the 4x4 table
//   kOther, sub rb     dense 2x2 with any controls; sub 8 + rb: a diagonal one;
//                      sub 16: nothing (a gate whose effect is deferred)
// A kNot with `cx` has c < 5 and is followed by the phase m[0] + i m[1] where
// both bits of rmask are 1.
enum : int {
    kCoreA = 0, kCoreB = 32, kNot = 64, kNotM = 96, kPhase = 128, kSign = 160, kDense4 = 192, kOther = 224,
    kDiag = kOther + 8, kNop = kOther + 16,
    // of FOne, where NOTs with one register control are kNotM and phases and signs kPhase
    kOneDense = 256,  // + rb, + 5 with register controls, + 10 with thread-bit controls
    kOneDiag = 288    // + rb
};
// Class bits of the device code.
enum : uint32_t {
    kcCore = 1, kcNot = 2, kcPhase = 4, kcSign = 8, kcRare = 16, kcNotM = 32, kcDense4 = 64, kcOther = 128, kcLane = 256,
    kcBack = 512  // its signs are of -pi, not pi
};
// sin of the double next to pi: what exp(i pi) and exp(-i pi) have beside -1.
// That is a whole unit in the last place of complex128, and the same way for
// every CZ of a circuit: left out, 16 layers with a CZ ladder on 12 qubits are
// off by 5.4e-15 instead of 2.4e-15, 400 CZs by 1.4e-14 instead of 1.8e-15.
// A sign of complex128 therefore brings its turn, i k sin pi for k half turns;
// complex64 does not see it.
constexpr double kSinPi = 1.2246467991473532e-16;

constexpr uint32_t kPhAny = 1u << 15, kPhAll = 1u << 16;

constexpr int kPairB1[10] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3};
constexpr int kPairB2[10] = {1, 2, 3, 4, 2, 3, 4, 3, 4, 4};

inline int pair_of(int b1, int b2)
{
    if (b1 > b2) std::swap(b1, b2);
    int p = 0;
    while (!(kPairB1[p] == b1 && kPairB2[p] == b2)) ++p;
    return p;
}

__device__ __forceinline__ uint32_t lane_get(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ float lane_get(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_get(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = lane_get((uint32_t)b, l), hi = lane_get((uint32_t)((unsigned long long)b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ float flip_sign(float v, uint32_t s) { return __uint_as_float(__float_as_uint(v) ^ s); }
__device__ __forceinline__ double flip_sign(double v, uint32_t s)
{
    return __longlong_as_double(__double_as_longlong(v) ^ (long long)((unsigned long long)s << 32));
}

// Up to 64 op records of a phase, one per lane.
template <typename T, int RB>
struct OpLanes {
    uint32_t code, sub, multi, ph;
    uint64_t gmask;
    T m[2 * RB], f0, f1;
};

template <typename T, int RB>
__device__ __forceinline__ OpLanes<T, RB> load_ops(const FRec<T>* __restrict__ recs, uint32_t begin, uint32_t end,
                                                   uint32_t lane)
{
    OpLanes<T, RB> o;
    const uint32_t i = begin + lane;
    const FRec<T>* R = recs + (i < end ? i : begin);
    o.code = R->code;
    o.sub = R->sub;
    o.multi = R->multi;
    o.ph = R->ph;
    o.gmask = R->gmask;
#pragma unroll
    for (int k = 0; k < 2 * RB; ++k) o.m[k] = R->m[k];
    o.f0 = R->m[10];
    o.f1 = R->m[11];
    return o;
}

// --- in-register ops: straight-line code over compile-time register indices ---

// Dense 2x2 on register bit RBIT for the pairs whose register index has every
// bit of rmask set (uniform branches) on the lanes that `sel` selects.
template <typename T, int RB, int RBIT>
__device__ __forceinline__ void dense_case(typename C2<T>::type (&v)[1 << RB], const T (&mm)[8], uint32_t rmask,
                                           bool sel)
{
    using V = typename C2<T>::type;
    T m[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) m[k] = sel ? mm[k] : (k == 0 || k == 6) ? T(1) : T(0);
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if (r0 & (1 << RBIT)) continue;
        if (((uint32_t)r0 & rmask) == rmask) apply2<T, V>(m, v[r0], v[r0 | (1 << RBIT)]);
    }
}

template <typename T, int RB, int RBIT>
__device__ __forceinline__ void diag_case(typename C2<T>::type (&v)[1 << RB], const T (&mm)[8], uint32_t rmask,
                                          bool sel)
{
    const T d0r = sel ? mm[0] : T(1), d0i = sel ? mm[1] : T(0), d1r = sel ? mm[6] : T(1), d1i = sel ? mm[7] : T(0);
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if (r0 & (1 << RBIT)) continue;
        if (((uint32_t)r0 & rmask) != rmask) continue;
        const int r1 = r0 | (1 << RBIT);
        const T ax = v[r0].x, ay = v[r0].y, bx = v[r1].x, by = v[r1].y;
        v[r0].x = fma(d0r, ax, -(d0i * ay));
        v[r0].y = fma(d0r, ay, d0i * ax);
        v[r1].x = fma(d1r, bx, -(d1i * by));
        v[r1].y = fma(d1r, by, d1i * bx);
    }
}

// NOT on RBIT where register bit C is 1 (C == 5: everywhere): moves only.
template <typename T, int RB, int RBIT, int C>
__device__ __forceinline__ void not_case(typename C2<T>::type (&v)[1 << RB])
{
    using V = typename C2<T>::type;
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if (r0 & (1 << RBIT)) continue;
        if (C < 5 && !((r0 >> C) & 1)) continue;
        const int r1 = r0 | (1 << RBIT);
        // float pairs move as one (component by component twice the moves: 200
        // NOTs on 26 qubits 1.77 ms, 1.60 so); double pairs cost k_fused 12
        // registers and a wave that way
        if constexpr (sizeof(T) == 4) {
            const V t = v[r0];
            v[r0] = v[r1];
            v[r1] = t;
        } else {
            const T ax = v[r0].x, ay = v[r0].y, bx = v[r1].x, by = v[r1].y;
            v[r0].x = bx;
            v[r0].y = by;
            v[r1].x = ax;
            v[r1].y = ay;
        }
    }
}

template <typename T, int RB, int RBIT>
__device__ __forceinline__ void notm_case(typename C2<T>::type (&v)[1 << RB], uint32_t rmask, bool sel)
{
    using V = typename C2<T>::type;
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if (r0 & (1 << RBIT)) continue;
        const int r1 = r0 | (1 << RBIT);
        if (((uint32_t)r0 & rmask) != rmask) continue;  // uniform over the wave
        const V a = v[r0], b = v[r1];
        v[r0].x = sel ? b.x : a.x;
        v[r0].y = sel ? b.y : a.y;
        v[r1].x = sel ? a.x : b.x;
        v[r1].y = sel ? a.y : b.y;
    }
}

// Multiply the registers whose index has every bit of MASK set by (fr, fi).
// The two products of the imaginary part round differently with their order;
// LANE has the one that phases of lanes use.  Each kind keeps its order, so
// that the sums of a complex64 batch do not change with its layout.
template <typename T, int RB, uint32_t MASK, bool LANE = false>
__device__ __forceinline__ void phase_case(typename C2<T>::type (&v)[1 << RB], T fr, T fi, uint32_t rmask = 0)
{
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r)
        if (((uint32_t)r & MASK) == MASK && ((uint32_t)r & rmask) == rmask) {
            const T x = v[r].x, y = v[r].y;
            v[r].x = fma(fr, x, -(fi * y));
            v[r].y = LANE ? fma(fi, x, fr * y) : fma(fr, y, fi * x);
        }
}

// Exchange the signs that `s` has set in the registers whose index has every
// bit of MASK set and, in complex128, multiply them by 1 - i r (r^2 far below
// an ulp).
template <typename T, int RB, uint32_t MASK>
__device__ __forceinline__ void sign_case(typename C2<T>::type (&v)[1 << RB], uint32_t s, T r)
{
#pragma unroll
    for (int k = 0; k < (1 << RB); ++k)
        if (((uint32_t)k & MASK) == MASK) {
            const T x = flip_sign(v[k].x, s), y = flip_sign(v[k].y, s);
            v[k].x = sizeof(T) == 8 ? fma(r, y, x) : x;
            v[k].y = sizeof(T) == 8 ? fma(-r, x, y) : y;
        }
}

// In-place form: the new b takes a fresh register, the new a is accumulated
// where a was (for EXCH, where b was).
template <typename T, int RB, int RBIT, bool EXCH>
__device__ __forceinline__ void core_case(typename C2<T>::type (&v)[1 << RB], T kr, T ki)
{
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if (r0 & (1 << RBIT)) continue;
        // with the pair exchanged, (k a + b, a - conj(k) b) is the plain core of (b, a)
        const int ra = EXCH ? r0 | (1 << RBIT) : r0, rb = EXCH ? r0 : r0 | (1 << RBIT);
        T ax = v[ra].x, ay = v[ra].y, bx = v[rb].x, by = v[rb].y;
        T nx = -kr * ax + bx;
        T ny = -kr * ay + by;
        nx = -ki * ay + nx;
        ny = ki * ax + ny;
        ax = kr * bx + ax;
        ay = kr * by + ay;
        ax = -ki * by + ax;
        ay = ki * bx + ay;
        v[r0].x = ax;
        v[r0].y = ay;
        v[r0 | (1 << RBIT)].x = nx;
        v[r0 | (1 << RBIT)].y = ny;
    }
}

// 4x4 complex matrix on every register quad, index bit(B1) + 2 bit(B2); lane
// e of `mv` holds value e of the row-major interleaved matrix.
template <typename T, int RB, int B1, int B2>
__device__ __forceinline__ void dense4_case(typename C2<T>::type (&v)[1 << RB], T mv)
{
    using V = typename C2<T>::type;
    // Row by row, 8 values at a time, for all quads before the next row: the
    // whole complex128 matrix is 64 scalar registers, and was spilled lane by
    // lane (density matrix of 13 qubits, complex128, eight noisy layers with
    // 104 of these: 11.7 ms, 10.1 so).
    V y[1 << RB];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        T m[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) m[k] = lane_get(mv, 8 * i + k);
#pragma unroll
        for (int r0 = 0; r0 < (1 << RB); ++r0) {
            if ((r0 >> B1) & 1 || (r0 >> B2) & 1) continue;
            const int r[4] = {r0, r0 | (1 << B1), r0 | (1 << B2), r0 | (1 << B1) | (1 << B2)};
            // one product or multiply-add per statement
            T re = m[0] * v[r0].x;
            T im = m[0] * v[r0].y;
            re = -m[1] * v[r0].y + re;
            im = m[1] * v[r0].x + im;
#pragma unroll
            for (int j = 1; j < 4; ++j) {
                re = m[2 * j] * v[r[j]].x + re;
                re = -m[2 * j + 1] * v[r[j]].y + re;
                im = m[2 * j] * v[r[j]].y + im;
                im = m[2 * j + 1] * v[r[j]].x + im;
            }
            y[r[i]].x = re;
            y[r[i]].y = im;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) v[r] = y[r];
}

__device__ __forceinline__ uint32_t table_entry(float m) { return __float_as_uint(m); }
__device__ __forceinline__ uint32_t table_entry(double m) { return (uint32_t)__double_as_longlong(m); }

// One record.  Its classes and subs are single bits, tested one after the
// other without else branches, each on a value the compiler cannot relate to
// the last test: such a chain keeps the amplitudes in the same registers
// throughout, while a switch over the ops becomes a net of branches that
// copies all of them (2,200 moves in the kernel, about 800 cycles per op).
#define QS_IF(word, mask) \
    asm volatile("" : "+s"(word)); \
    if (__builtin_expect(((word) & (mask)) != 0, 0))

template <typename T, int RB>
__device__ __forceinline__ void apply_op(typename C2<T>::type (&v)[1 << RB], const OpLanes<T, RB>& o, int i, uint32_t code,
                                         T m4, const FRec<T>* __restrict__ rec, uint32_t tid)
{
    uint32_t multi = lane_get(o.multi, i), sub = lane_get(o.sub, i);
    QS_IF(code, kcCore) {
#define QS_C(B)                                                                                                      \
    if constexpr (RB > B) {                                                                                          \
        QS_IF(multi, 1u << B) core_case<T, RB, B, false>(v, lane_get(o.m[2 * B], i), lane_get(o.m[2 * B + 1], i));   \
        QS_IF(multi, 32u << B) core_case<T, RB, B, true>(v, lane_get(o.m[2 * B], i), lane_get(o.m[2 * B + 1], i));   \
    }
        QS_C(0) QS_C(1) QS_C(2) QS_C(3) QS_C(4)
#undef QS_C
    }
    QS_IF(code, kcNot) {
#define QS_N(B, C) \
    if constexpr ((C == 5 || RB > C) && B != C) { QS_IF(sub, 1u << (6 * B + C)) not_case<T, RB, B, C>(v); }
#define QS_NB(B)                                                                 \
    if constexpr (RB > B) {                                                      \
        QS_IF(sub, 63u << (6 * B)) {                                             \
            QS_N(B, 0) QS_N(B, 1) QS_N(B, 2) QS_N(B, 3) QS_N(B, 4) QS_N(B, 5)    \
        }                                                                        \
    }
        QS_NB(0) QS_NB(1) QS_NB(2) QS_NB(3) QS_NB(4)
#undef QS_NB
#undef QS_N
    }
    QS_IF(code, kcPhase) {
        const uint32_t tmask = code >> 16, rmask = (multi >> 10) & 31u;
        const bool sel = (tid & tmask) == tmask;
        const T m0 = lane_get(o.f0, i), m1 = lane_get(o.f1, i);
        const T fr = sel ? m0 : T(1), fi = sel ? m1 : T(0);
        uint32_t ph = lane_get(o.ph, i);
        QS_IF(ph, 31u) {
#define QS_P(B) if constexpr (RB > B) { QS_IF(ph, 1u << B) phase_case<T, RB, 1u << B>(v, fr, fi); }
            QS_P(0) QS_P(1) QS_P(2) QS_P(3) QS_P(4)
#undef QS_P
        }
        QS_IF(ph, 1023u << 5) {
#define QS_P(P)                                                                                    \
    if constexpr (RB > kPairB2[P]) {                                                               \
        QS_IF(ph, 32u << P) phase_case<T, RB, (1u << kPairB1[P]) | (1u << kPairB2[P])>(v, fr, fi); \
    }
            QS_P(0) QS_P(1) QS_P(2) QS_P(3) QS_P(4) QS_P(5) QS_P(6) QS_P(7) QS_P(8) QS_P(9)
#undef QS_P
        }
        QS_IF(ph, kPhAll) phase_case<T, RB, 0>(v, fr, fi);
        QS_IF(ph, kPhAny) phase_case<T, RB, 0, true>(v, fr, fi, rmask);  // uniform branches
    }
    QS_IF(code, kcSign) {
        const uint32_t tmask = code >> 16;
        const bool sel = (tid & tmask) == tmask;
        const uint32_t s = sel ? 0x80000000u : 0u;
        const T r = (T)(!sel ? 0.0 : (code & kcBack) ? -kSinPi : kSinPi);
        QS_IF(multi, 31u << 15) {
#define QS_P(B) if constexpr (RB > B) { QS_IF(multi, (1u << 15) << B) sign_case<T, RB, 1u << B>(v, s, r); }
            QS_P(0) QS_P(1) QS_P(2) QS_P(3) QS_P(4)
#undef QS_P
        }
        QS_IF(multi, 1023u << 20) {
#define QS_P(P)                                                                                        \
    if constexpr (RB > kPairB2[P]) {                                                                   \
        QS_IF(multi, (1u << 20) << P)                                                                  \
            sign_case<T, RB, (1u << kPairB1[P]) | (1u << kPairB2[P])>(v, s, r);                        \
    }
            QS_P(0) QS_P(1) QS_P(2) QS_P(3) QS_P(4) QS_P(5) QS_P(6) QS_P(7) QS_P(8) QS_P(9)
#undef QS_P
        }
    }
    QS_IF(code, kcRare) {
        const uint32_t rmask = (multi >> 10) & 31u, tmask = code >> 16;
        const bool sel = (tid & tmask) == tmask;
        QS_IF(code, kcDense4) {
#define QS_D4(P) \
    if constexpr (RB > kPairB2[P]) { QS_IF(sub, 1u << P) dense4_case<T, RB, kPairB1[P], kPairB2[P]>(v, m4); }
            QS_D4(0) QS_D4(1) QS_D4(2) QS_D4(3) QS_D4(4) QS_D4(5) QS_D4(6) QS_D4(7) QS_D4(8) QS_D4(9)
#undef QS_D4
        }
        QS_IF(code, kcNotM) {
#define QS_C(B) if constexpr (RB > B) { QS_IF(sub, 1u << B) notm_case<T, RB, B>(v, rmask, sel); }
            QS_C(0) QS_C(1) QS_C(2) QS_C(3) QS_C(4)
#undef QS_C
        }
        QS_IF(code, kcOther) {
            T m[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) m[k] = rec->m[k];
#define QS_O(B)                                                                          \
    if constexpr (RB > B) {                                                              \
        QS_IF(sub, 1u << B) dense_case<T, RB, B>(v, m, rmask, sel);                      \
        QS_IF(sub, 256u << B) diag_case<T, RB, B>(v, m, rmask, sel);                     \
    }
            QS_O(0) QS_O(1) QS_O(2) QS_O(3) QS_O(4)
#undef QS_O
        }
    }
}

#undef QS_IF

// XOR of img[b] over the set bits b of x (x < 2^NB).
template <int NB, typename U>
__device__ __forceinline__ U span(uint32_t x, const U* img)
{
    U s = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if ((x >> b) & 1) s ^= img[b];
    return s;
}

template <int NB, typename U>
__device__ __forceinline__ U span_sum(uint32_t x, const U* img)
{
    U s = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if ((x >> b) & 1) s += img[b];
    return s;
}

// Orders the workgroup's LDS accesses (only those: global loads stay in
// flight).  A one-wave workgroup needs no barrier.
template <int TB>
__device__ __forceinline__ void lds_barrier()
{
    if constexpr (TB > 6) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Write the tile in the layout being left, read it in the one entered; word(e)
// is word e of the FPhase.
template <typename T, int TB, int RB, typename W>
__device__ __forceinline__ void relayout(typename C2<T>::type (&v)[1 << RB],
                                         typename C2<T>::type* lds, W word, uint32_t tid)
{
    uint32_t tw = 0, tr = 0, wreg[RB], rreg[RB];
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const uint32_t on = 0u - ((tid >> b) & 1u);
        tw ^= on & word(b);
        tr ^= on & word(kTBMax + kRBMax + b);
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        wreg[b] = word(kTBMax + b);
        rreg[b] = word(2 * kTBMax + kRBMax + b);
    }
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) lds[tw ^ span<RB, uint32_t>((uint32_t)r, wreg)] = v[r];
    lds_barrier<TB>();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) v[r] = lds[tr ^ span<RB, uint32_t>((uint32_t)r, rreg)];
    lds_barrier<TB>();
}

// One tile of a planned pass: load, apply every phase's ops with the
// re-layouts between them, store.  `base` = tile index with zeros at the
// tile's qubits.
//
// What bounds it is the op stream, not the arithmetic (a core on 16 complex128
// registers is 64 multiply-adds, 256 cycles): read through the scalar cache
// record by record, each op waited for two dependent loads and took about
// 2,400 cycles.  So a wave loads up to 64 records of a phase at once, one
// per lane, a phase ahead of their use, drops those whose outside controls
// are 0 in this tile with one ballot, and gets each op's few words with
// v_readlane.
template <typename T, int TB, int RB>
__device__ __forceinline__ void process_tile(typename C2<T>::type* __restrict__ amp, const FPass* __restrict__ P,
                                             const FRec<T>* __restrict__ recs, const T* __restrict__ m4tab,
                                             uint64_t tile, typename C2<T>::type* lds, uint32_t tid,
                                             bool zero_init = false)
{
    using V = typename C2<T>::type;
    constexpr int E = 1 << RB;
    // 1024 complex128 threads have 128 registers each: no room for a second set of records
    constexpr bool kAhead = TB < 10 || sizeof(T) == 4;
    // a 4x4 matrix loaded while the one before it is applied takes two more, which would cost the fourth wave here
    constexpr bool kAhead4 = RB != 3 || sizeof(T) == 4;
    const uint32_t lane = tid & 63u;
    const int nph = P->nphases;
    uint32_t pw = ((const uint32_t*)&P->ph[0])[lane & 31u];
    uint32_t ob = lane_get(pw, 30), oe = lane_get(pw, 31);
    OpLanes<T, RB> cur = load_ops<T, RB>(recs, ob, oe, lane);
    const uint64_t ld_t = span_sum<TB, uint64_t>(tid, P->ld_thr);
    const uint64_t st_t = span_sum<TB, uint64_t>(tid, P->st_thr);
    const uint64_t base = expand(tile, P->outside);
    V v[E];
    if (zero_init) {  // the tile of |0..0>: nothing to read
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const uint64_t a = base + ld_t + span_sum<RB, uint64_t>((uint32_t)r, P->ld_reg);
            v[r].x = (a == 0) ? T(1) : T(0);
            v[r].y = T(0);
        }
    } else {
#pragma unroll
        for (int r = 0; r < E; ++r) v[r] = amp[base + ld_t + span_sum<RB, uint64_t>((uint32_t)r, P->ld_reg)];
    }
    const int nlay = nph + P->final_transpose;
    for (int ph = 0; ph < nlay; ++ph) {
        // the next phase's words and records, in flight during this one's ops
        const uint32_t npw = ((const uint32_t*)&P->ph[ph + 1 < nlay ? ph + 1 : ph])[lane & 31u];
        if (ph > 0) relayout<T, TB, RB>(v, lds, [&](int e) { return lane_get(pw, e); }, tid);
        const uint32_t nob = lane_get(npw, 30), noe = lane_get(npw, 31);
        OpLanes<T, RB> nxt;
        if constexpr (kAhead) nxt = load_ops<T, RB>(recs, nob, noe, lane);
        for (uint32_t c = ob;;) {
            uint64_t act = __ballot(c + lane < oe && (base & cur.gmask) == cur.gmask);
            // signs on thread and outside bits alone
            uint64_t lanes = act & __ballot((cur.code & kcLane) != 0);
            act ^= lanes;
            if (lanes) {
                uint32_t s = 0;
                int turns = 0;  // complex128
                while (lanes) {
                    const uint32_t code = lane_get(cur.code, __builtin_ctzll(lanes)), tmask = code >> 16;
                    lanes &= lanes - 1;
                    const bool sel = (tid & tmask) == tmask;
                    s ^= sel ? 0x80000000u : 0u;
                    turns += !sel ? 0 : (code & kcBack) ? -1 : 1;
                }
                sign_case<T, RB, 0>(v, s, (T)(kSinPi * turns));
            }
            // the next 4x4 matrix, one value per lane, loaded ahead
            uint64_t d4 = act & __ballot((cur.code & kcDense4) != 0);
            const uint32_t entry = table_entry(cur.f0);
            T m4 = T(0), m4n = T(0);
            if (d4) m4n = m4tab[32 * (uint64_t)lane_get(entry, __builtin_ctzll(d4)) + (lane & 31u)];
            while (act) {
                const int i = __builtin_ctzll(act);
                act &= act - 1;
                const uint32_t code = lane_get(cur.code, i);
                const bool is4 = (code & kcDense4) != 0;
                if constexpr (kAhead4) {
                    if (__builtin_expect(is4, 0)) {
                        m4 = m4n;
                        d4 &= d4 - 1;
                        if (d4) m4n = m4tab[32 * (uint64_t)lane_get(entry, __builtin_ctzll(d4)) + (lane & 31u)];
                    }
                    apply_op<T, RB>(v, cur, i, code, m4, recs + c + i, tid);
                } else {
                    apply_op<T, RB>(v, cur, i, code, m4n, recs + c + i, tid);
                    if (__builtin_expect(is4, 0)) {
                        d4 &= d4 - 1;
                        if (d4) m4n = m4tab[32 * (uint64_t)lane_get(entry, __builtin_ctzll(d4)) + (lane & 31u)];
                    }
                }
            }
            c += 64;
            if (c >= oe) break;
            cur = load_ops<T, RB>(recs, c, oe, lane);
        }
        pw = npw;
        ob = nob;
        oe = noe;
        if constexpr (kAhead) cur = nxt;
        else cur = load_ops<T, RB>(recs, ob, oe, lane);
    }
#pragma unroll
    for (int r = 0; r < E; ++r) amp[base + st_t + span_sum<RB, uint64_t>((uint32_t)r, P->st_reg)] = v[r];
}

// One FOp by one switch.  REG, LANE: register-bit and thread-bit controls.
template <typename T, int RB, int RBIT, bool REG, bool LANE>
__device__ __forceinline__ void one_dense(typename C2<T>::type (&v)[1 << RB], const FOne<T>& op, bool sel)
{
    using V = typename C2<T>::type;
    T m[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) m[k] = op.m[k];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (LANE) m[k] = sel ? m[k] : (k == 0 || k == 6) ? T(1) : T(0);
        // products with scalar registers are slower in complex64 (200 dense gates on 26 qubits 3.43 ms, 2.84 so)
        else if (sizeof(T) == 4) asm("" : "+v"(m[k]));
    }
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if (r0 & (1 << RBIT)) continue;
        if (REG && ((uint32_t)r0 & op.rmask) != op.rmask) continue;  // uniform over the wave
        apply2<T, V>(m, v[r0], v[r0 | (1 << RBIT)]);
    }
}

// 4x4 on every register quad, the whole matrix in scalar registers.
template <typename T, int RB, int B1, int B2>
__device__ __forceinline__ void one_dense4(typename C2<T>::type (&v)[1 << RB], const T* __restrict__ m)
{
    using V = typename C2<T>::type;
#pragma unroll
    for (int r0 = 0; r0 < (1 << RB); ++r0) {
        if ((r0 >> B1) & 1 || (r0 >> B2) & 1) continue;
        const int r[4] = {r0, r0 | (1 << B1), r0 | (1 << B2), r0 | (1 << B1) | (1 << B2)};
        const V x[4] = {v[r[0]], v[r[1]], v[r[2]], v[r[3]]};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // one product or multiply-add per statement
            T re = m[8 * i] * x[0].x;
            T im = m[8 * i] * x[0].y;
            re = -m[8 * i + 1] * x[0].y + re;
            im = m[8 * i + 1] * x[0].x + im;
#pragma unroll
            for (int j = 1; j < 4; ++j) {
                const T mr = m[2 * (4 * i + j)], mi = m[2 * (4 * i + j) + 1];
                re = mr * x[j].x + re;
                re = -mi * x[j].y + re;
                im = mr * x[j].y + im;
                im = mi * x[j].x + im;
            }
            v[r[i]].x = re;
            v[r[i]].y = im;
        }
    }
}

template <typename T, int RB>
__device__ __forceinline__ void apply_one(typename C2<T>::type (&v)[1 << RB], const FOne<T>& op, uint32_t tid,
                                          const T* __restrict__ m4tab)
{
    const uint32_t rmask = op.rmask;
    const bool sel = (tid & op.tmask) == op.tmask;
    switch (op.kind) {
#define QS_O(B)                                                                                           \
    case kCoreA + B: if constexpr (RB > B) core_case<T, RB, B, false>(v, op.m[0], op.m[1]); break;        \
    case kCoreB + B: if constexpr (RB > B) core_case<T, RB, B, true>(v, op.m[0], op.m[1]); break;         \
    case kNot + B: if constexpr (RB > B) not_case<T, RB, B, 5>(v); break;                                 \
    case kNotM + B: if constexpr (RB > B) notm_case<T, RB, B>(v, rmask, sel); break;                      \
    case kOneDense + B: if constexpr (RB > B) one_dense<T, RB, B, false, false>(v, op, sel); break; \
    case kOneDense + 5 + B: if constexpr (RB > B) one_dense<T, RB, B, true, false>(v, op, sel); break; \
    case kOneDense + 10 + B: if constexpr (RB > B) one_dense<T, RB, B, false, true>(v, op, sel); break; \
    case kOneDense + 15 + B: if constexpr (RB > B) one_dense<T, RB, B, true, true>(v, op, sel); break; \
    case kOneDiag + B: if constexpr (RB > B) diag_case<T, RB, B>(v, op.m, rmask, sel); break;
        QS_O(0) QS_O(1) QS_O(2) QS_O(3) QS_O(4)
#undef QS_O
#define QS_O(P)                                                                                           \
    case kDense4 + P:                                                                                     \
        if constexpr (RB > kPairB2[P]) one_dense4<T, RB, kPairB1[P], kPairB2[P]>(v, m4tab + 32 * op.aux); \
        break;
        QS_O(0) QS_O(1) QS_O(2) QS_O(3) QS_O(4) QS_O(5) QS_O(6) QS_O(7) QS_O(8) QS_O(9)
#undef QS_O
    case kPhase: phase_case<T, RB, 0>(v, sel ? op.m[0] : T(1), sel ? op.m[1] : T(0), rmask); break;
    default: break;
    }
    if (op.cx) phase_case<T, RB, 0>(v, op.m[0], op.m[1], rmask | (1u << (op.cx - 1)));
}

// One tile of a pass whose time goes into 4x4s or full 2x2s (op_gain): an op at
// a time, its record and matrix read through the scalar cache, whose latency
// other waves hide.  The records of process_tile save that latency and pay in
// issue slots: a complex128 4x4 gets its 32 values with 64 v_readlanes, a
// quarter of its multiply-adds' time.  200 two-qubit gates on 26 qubits in
// 12-qubit tiles: 19.3 ms by records, 14.7 so in complex128, 10.9 and 8.5 in
// complex64; 200 one-qubit gates 3.6 and 4.9, 2.3 and 2.6.
template <typename T, int TB, int RB>
__device__ __forceinline__ void process_tile_ops(typename C2<T>::type* __restrict__ amp, const FPass* __restrict__ P,
                                                 const FOne<T>* __restrict__ ops, const T* __restrict__ m4tab,
                                                 uint64_t tile, typename C2<T>::type* lds, uint32_t tid,
                                                 bool zero_init = false)
{
    using V = typename C2<T>::type;
    const int nph = P->nphases, nlay = nph + P->final_transpose;
    const uint64_t ld_t = span_sum<TB, uint64_t>(tid, P->ld_thr), st_t = span_sum<TB, uint64_t>(tid, P->st_thr);
    const uint64_t base = expand(tile, P->outside);
    V v[1 << RB];
    if (zero_init) {  // the tile of |0..0>: nothing to read
#pragma unroll
        for (int r = 0; r < (1 << RB); ++r) {
            v[r].x = base + ld_t + span_sum<RB, uint64_t>((uint32_t)r, P->ld_reg) == 0 ? T(1) : T(0);
            v[r].y = T(0);
        }
    } else {
#pragma unroll
        for (int r = 0; r < (1 << RB); ++r) v[r] = amp[base + ld_t + span_sum<RB, uint64_t>((uint32_t)r, P->ld_reg)];
    }
    for (int ph = 0; ph < nlay; ++ph) {
        if (ph > 0) {
            uint4 F[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) F[k] = ((const uint4*)&P->ph[ph])[k];
            const auto word = [&](int e) {
                const uint4 w = F[e / 4];
                return e & 2 ? (e & 1 ? w.w : w.z) : (e & 1 ? w.y : w.x);
            };
            relayout<T, TB, RB>(v, lds, word, tid);
        }
        if (ph == nph) break;
        for (uint32_t o = P->first_op[ph]; o < P->first_op[ph + 1]; ++o) {
            const FOne<T>& op = ops[o];
            if ((base & op.gmask) != op.gmask) continue;  // same for the whole tile
            apply_one<T, RB>(v, op, tid, m4tab);
        }
    }
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) amp[base + st_t + span_sum<RB, uint64_t>((uint32_t)r, P->st_reg)] = v[r];
}

template <typename T, int TB, int RB>
__global__ __launch_bounds__(1 << TB) void k_fused_ops(typename C2<T>::type* __restrict__ amp,
                                                       const FPass* __restrict__ P,
                                                       const FOne<T>* __restrict__ ops, const T* __restrict__ m4tab,
                                                       uint64_t ntiles)
{
    __shared__ typename C2<T>::type lds[1 << (TB + RB)];
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
        process_tile_ops<T, TB, RB>(amp, P, ops, m4tab, tile, lds, threadIdx.x);
}

template <typename T, int TB, int RB>
__global__ __launch_bounds__(1 << TB) void k_fused(typename C2<T>::type* __restrict__ amp,
                                                   const FPass* __restrict__ P,
                                                   const FRec<T>* __restrict__ recs, const T* __restrict__ m4tab,
                                                   uint64_t ntiles)
{
    using V = typename C2<T>::type;
    __shared__ V lds[1 << (TB + RB)];
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
        process_tile<T, TB, RB>(amp, P, recs, m4tab, tile, lds, threadIdx.x);
}

// Batched registers.  Every register's circuit is planned into passes; the
// work of pass level p is the list of items (register, its pass p, range of
// tiles) over all registers that have a pass p.  One launch per level runs
// its items, each workgroup taking items in a grid-stride loop; the launch
// boundary is the only synchronisation between the passes of a register, so
// no workgroup ever waits for another.  Tiles of the first pass can be
// produced as |0..0> instead of being read (init).
struct BatchReg {
    void* amp;
    int n;
    int npasses;
    uint32_t pass0;   // first pass of the register in the pass array
    uint32_t piece0;  // first of its pieces in the probability sums
    uint32_t logc, pad;
};

struct BatchItem {
    uint32_t reg, pass, tile0, tile1;
};

template <typename T, int TB, int RB, bool BYOP>
__global__ __launch_bounds__(1 << TB) void k_batch(const BatchReg* __restrict__ regs,
                                                   const BatchItem* __restrict__ items, int nitems,
                                                   const FPass* __restrict__ passes,
                                                   const void* __restrict__ ops, const T* __restrict__ m4tab,
                                                   int init)
{
    using V = typename C2<T>::type;
    __shared__ V lds[1 << (TB + RB)];
    const uint32_t tid = threadIdx.x;
    for (int i = blockIdx.x; i < nitems; i += gridDim.x) {
        const BatchItem it = items[i];
        const BatchReg R = regs[it.reg];
        const FPass* P = passes + R.pass0 + it.pass;
        const bool zi = init && it.pass == 0;
        for (uint32_t tile = it.tile0; tile < it.tile1; ++tile)
            if constexpr (BYOP) process_tile_ops<T, TB, RB>((V*)R.amp, P, (const FOne<T>*)ops, m4tab, tile, lds, tid, zi);
            else process_tile<T, TB, RB>((V*)R.amp, P, (const FRec<T>*)ops, m4tab, tile, lds, tid, zi);
    }
}

// Per-register probabilities, P(qubit q = 0) and the total, as compensated
// double sums.  A register is cut into 2^logc pieces of at least 4096
// amplitudes (BatchReg::logc), one workgroup each; k_batch_probs_final adds
// a register's pieces in a fixed order.  One workgroup per register left a
// batch's largest register to a single CU: 60 registers of 10..20 qubits in
// complex64 took 1,300 us.
struct ProbItem {
    uint32_t reg, piece;
};

template <typename T>
__global__ __launch_bounds__(256) void k_batch_probs(const BatchReg* __restrict__ regs,
                                                     const ProbItem* __restrict__ items, int q,
                                                     double* __restrict__ partials)
{
    using V = typename C2<T>::type;
    constexpr int U = 8;
    __shared__ double sh[4][4];
    const ProbItem it = items[blockIdx.x];
    const BatchReg R = regs[it.reg];
    const uint64_t len = 1ull << (R.n - R.logc);  // at least 512, the smallest register
    const uint64_t e0 = (uint64_t)it.piece * len;
    const V* amp = (const V*)R.amp + e0;
    NSum s0 = {0.0, 0.0}, st = {0.0, 0.0};
    for (uint64_t b = 0; b < len; b += 256 * U) {
        V a[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t e = b + 256 * j + threadIdx.x;
            a[j].x = a[j].y = T(0);
            if (b + 256 * j < len) a[j] = amp[e];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint64_t e = e0 + b + 256 * j + threadIdx.x;
            const double p = (double)a[j].x * (double)a[j].x + (double)a[j].y * (double)a[j].y;
            nadd(s0, ((e >> q) & 1) ? 0.0 : p);
            nadd(st, p);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        s0 = nmerge(s0, NSum{__shfl_xor(s0.s, off, 64), __shfl_xor(s0.c, off, 64)});
        st = nmerge(st, NSum{__shfl_xor(st.s, off, 64), __shfl_xor(st.c, off, 64)});
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[0][w] = s0.s;
        sh[1][w] = s0.c;
        sh[2][w] = st.s;
        sh[3][w] = st.c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        NSum a = {sh[0][0], sh[1][0]}, b = {sh[2][0], sh[3][0]};
        for (int k = 1; k < 4; ++k) {
            a = nmerge(a, NSum{sh[0][k], sh[1][k]});
            b = nmerge(b, NSum{sh[2][k], sh[3][k]});
        }
        double* o = partials + 4 * (uint64_t)blockIdx.x;
        o[0] = a.s;
        o[1] = a.c;
        o[2] = b.s;
        o[3] = b.c;
    }
}

// One wave per register; out[2 i] = P(q = 0), out[2 i + 1] = total.
__global__ __launch_bounds__(64) void k_batch_probs_final(const BatchReg* __restrict__ regs,
                                                          const double* __restrict__ partials,
                                                          double* __restrict__ out)
{
    const int i = blockIdx.x;
    const double* p = partials + 4 * (uint64_t)regs[i].piece0;
    NSum s0 = {0.0, 0.0}, st = {0.0, 0.0};
    for (uint32_t k = threadIdx.x; k < 1u << regs[i].logc; k += 64) {
        s0 = nmerge(s0, NSum{p[4 * k], p[4 * k + 1]});
        st = nmerge(st, NSum{p[4 * k + 2], p[4 * k + 3]});
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        s0 = nmerge(s0, NSum{__shfl_xor(s0.s, off, 64), __shfl_xor(s0.c, off, 64)});
        st = nmerge(st, NSum{__shfl_xor(st.s, off, 64), __shfl_xor(st.c, off, 64)});
    }
    if (threadIdx.x == 0) {
        out[2 * i] = s0.s + s0.c;
        out[2 * i + 1] = st.s + st.c;
    }
}

void fill_phase(FPhase& F, const Layout& from, const Layout& to, int K)
{
    const std::vector<uint32_t> img = swizzle(from, to, K);
    memset(F.wthr, 0, sizeof(F.wthr));
    memset(F.wreg, 0, sizeof(F.wreg));
    memset(F.rthr, 0, sizeof(F.rthr));
    memset(F.rreg, 0, sizeof(F.rreg));
    for (size_t b = 0; b < from.thr.size(); ++b) F.wthr[b] = img[from.thr[b]];
    for (size_t b = 0; b < from.reg.size(); ++b) F.wreg[b] = img[from.reg[b]];
    for (size_t b = 0; b < to.thr.size(); ++b) F.rthr[b] = img[to.thr[b]];
    for (size_t b = 0; b < to.reg.size(); ++b) F.rreg[b] = img[to.reg[b]];
}

using Cx = std::complex<double>;

// Sub-code of a phase or sign on the register bits of rmask.
int phase_sub(uint32_t rmask)
{
    const int n = __builtin_popcount(rmask);
    if (n == 0) return 0;
    const int b1 = __builtin_ctz(rmask);
    if (n == 1) return 1 + b1;
    return n == 2 ? 6 + pair_of(b1, 31 - __builtin_clz(rmask)) : 16;
}

// Multiply the amplitudes whose register bits `rmask`, thread bits `tmask`
// and outside qubits `gmask` are all 1 by f.
FOp phase_fop(uint32_t rmask, uint32_t tmask, uint64_t gmask, Cx f)
{
    FOp o;
    memset(&o, 0, sizeof(o));
    const int sub = phase_sub(rmask);
    const bool sign = f.real() == -1.0 && fabs(fabs(f.imag()) - kSinPi) < 1e-18 && sub < 16;
    o.kind = (sign ? kSign : kPhase) + sub;
    o.rmask = rmask;
    o.tmask = tmask;
    o.gmask = gmask;
    o.m[0] = f.real();
    o.m[1] = f.imag();
    return o;
}

FOp encode_op(const OpRec& op, const PassPlan& P, const Layout& L)
{
    FOp f;
    memset(&f, 0, sizeof(f));
    std::vector<int> local(64, -1);
    for (size_t j = 0; j < P.S.size(); ++j) local[P.S[j]] = (int)j;
    auto classify = [&](int q) {
        const int j = local[q];
        if (j < 0) {
            f.gmask |= 1ull << q;
            return;
        }
        for (size_t b = 0; b < L.reg.size(); ++b)
            if (L.reg[b] == j) {
                f.rmask |= 1u << b;
                return;
            }
        for (size_t b = 0; b < L.thr.size(); ++b)
            if (L.thr[b] == j) {
                f.tmask |= 1u << b;
                return;
            }
    };
    for (int q : op.ctrls) classify(q);
    if (op.kind == 2) return phase_fop(f.rmask, f.tmask, f.gmask, Cx(cos(op.angle), sin(op.angle)));
    const int jt = local[op.target];
    for (size_t b = 0; b < L.reg.size(); ++b)
        if (L.reg[b] == jt) f.rb = (int)b;
    if (op.kind == 1) {
        const int nr = __builtin_popcount(f.rmask);
        f.kind = f.tmask || nr > 1 ? kNotM + f.rb : kNot + 6 * f.rb + (nr ? __builtin_ctz(f.rmask) : 5);
        return f;
    }
    const bool diag = op.u[2] == 0.0 && op.u[3] == 0.0 && op.u[4] == 0.0 && op.u[5] == 0.0;
    f.kind = (diag ? kDiag : kOther) + f.rb;
    for (int k = 0; k < 8; ++k) f.m[k] = op.u[k];
    return f;
}

// Diagonal factors deferred by the lowering (see lower_passes): the true
// state is gsc times prod_q exp(i phi[q] x_q) over the qubits with has[q],
// times the stored state.  Which qubits carry a factor, and whether gsc was
// touched, depends only on the op structure, not on matrix values, so a
// batch with new parameters lowers to the same number of ops in every phase: a
// gate off from unitary (core_form -1) defers a phase of 0.  A circuit that runs
// alone is lowered anew (`alone`), and there such a gate defers nothing: 200 of
// them on 26 qubits complex128 5.4 ms, 6.1 with the phases.
struct Defer {
    double phi[64] = {};
    bool has[64] = {};
    Cx gsc = 1.0;
    bool gsc_used = false;
    int shrink = 0;  // cores since gsc was last multiplied in
};

// Every core scales gsc by |d0| >= 1/sqrt 2, and the stored state grows by
// the inverse; after this many cores gsc is multiplied in (2^-30 keeps
// complex64 amplitudes far from overflow, 2^-500 complex128 ones).
inline int max_shrink(int prec) { return prec == QS_C128 ? 1000 : 60; }

// A dense 2x2 gate U written as diag(d0, d1) times a unit-diagonal core:
// form 2: U = diag(u00, u11) [[1, k], [-conj(k), 1]], k = u01 / u00;
// form 3: U = diag(u01, u10) [[k, 1], [1, -conj(k)]], k = u00 / u01;
// whichever has |k| <= 1.  Form 0: U diagonal; form 1: anti-diagonal.  Both
// identities need U unitary; form -1 when that fails by more than 1e-14.
struct CoreForm {
    int form;
    Cx k, d0, d1;
};

CoreForm core_form(const Cx (&u)[2][2])
{
    if (u[0][1] == 0.0 && u[1][0] == 0.0) return {0, 0.0, u[0][0], u[1][1]};
    if (u[0][0] == 0.0 && u[1][1] == 0.0) return {1, 0.0, u[0][1], u[1][0]};
    if (std::abs(u[0][0]) >= std::abs(u[0][1])) {
        const Cx k = u[0][1] / u[0][0];
        if (std::abs(u[1][0] + u[1][1] * std::conj(k)) > 1e-14) return {-1, 0.0, 0.0, 0.0};
        return {2, k, u[0][0], u[1][1]};
    }
    const Cx k = u[0][0] / u[0][1];
    if (std::abs(u[1][1] + u[1][0] * std::conj(k)) > 1e-14) return {-1, 0.0, 0.0, 0.0};
    return {3, k, u[0][1], u[1][0]};
}

// What an op gains op by op over the records, where the chip is full.  Measured
// on 26 qubits with 200 ops of a kind, in units of 3 us (1.5 in complex64): a
// 4x4 8, a 2x2 with controls or not as a core 1, a core -2 (-1), a phase -3
// (-2).  Complex64 with 8 amplitudes a thread: such a 2x2 2, a NOT with controls
// and a diagonal 2x2 1, a phase -1; with 32: a 4x4 2, a 2x2 nothing.  Signs, of
// which several share a record, -6, but a batch's choice is not to depend on
// angles.
int op_gain(const OpRec& op, bool dbl, int RB)
{
    const bool narrow = !dbl && RB == 3, wide = !dbl && RB == 5;
    if (op.kind == 4) return wide ? 2 : 8;
    if (op.kind == 1) return narrow && !op.ctrls.empty();
    if (op.kind == 2) return op.ctrls.size() < 2 ? 0 : dbl ? -3 : narrow ? -1 : -2;
    Cx u[2][2];
    for (int i = 0; i < 4; ++i) u[i / 2][i % 2] = Cx(op.u[2 * i], op.u[2 * i + 1]);
    const int form = core_form(u).form;
    if (op.ctrls.empty() && form >= 0) return form < 2 ? 0 : dbl ? -2 : -1;
    return wide ? 0 : (narrow ? 2 : 1) - (form == 0);
}

bool gains_by_op(const std::vector<OpRec>& ops, const std::vector<int>& which, int prec, const FusedConfig& c)
{
    if (c.TB == 9 && c.RB == 5) return false;  // 14-qubit tiles: 12.2 ms either way for 200 4x4s on 26 qubits
    int gain = 0;
    for (int k : which) gain += op_gain(ops[k], prec == QS_C128, c.RB);
    return gain > 0;
}

// Device form of a planned pass list, appended to hp / hops / m4 (op
// indices in the phases are positions in hops; 4x4 ops index m4 in blocks
// of 32 values).  The ops are lowered on the way: an uncontrolled dense
// gate becomes its unit-diagonal core (half the multiply-adds) and its
// diagonal part, like every one-qubit phase, is deferred; the next dense or
// 4x4 op on that qubit takes the deferred phase into its matrix on the host
// (free), a NOT moves it, and the last pass multiplies in what is left.
void serialize(const std::vector<PassPlan>& plan, const std::vector<OpRec>& ops, int TB, int RB, int prec,
               bool alone, std::vector<FPass>& hp, std::vector<FOp>& hops, std::vector<double>& m4)
{
    const int K = TB + RB;
    Defer d;
    for (size_t p = 0; p < plan.size(); ++p) {
        const PassPlan& P = plan[p];
        const bool last_pass = p + 1 == plan.size();
        std::vector<int> local(64, -1);
        for (int j = 0; j < K; ++j) local[P.S[j]] = j;
        FPass F;
        memset(&F, 0, sizeof(F));
        F.nphases = (int)P.phases.size();
        F.outside = make_insert(P.S.data(), (int)P.S.size(), 0);
        const Layout& L0 = P.phases.front().lay;
        for (int b = 0; b < TB; ++b) {
            F.ld_thr[b] = 1ull << P.S[L0.thr[b]];
            F.st_thr[b] = 1ull << P.S[P.store.thr[b]];
        }
        for (int b = 0; b < RB; ++b) {
            F.ld_reg[b] = 1ull << P.S[L0.reg[b]];
            F.st_reg[b] = 1ull << P.S[P.store.reg[b]];
        }
        for (size_t ph = 0; ph < P.phases.size(); ++ph) {
            FPhase& Fp = F.ph[ph];
            const Layout& L = P.phases[ph].lay;
            const Layout& prev = ph ? P.phases[ph - 1].lay : L;
            fill_phase(Fp, prev, L, K);
            Fp.op_begin = F.first_op[ph] = (uint32_t)hops.size();
            auto reg_bit = [&](int q) {
                for (int b = 0; b < RB; ++b)
                    if (L.reg[b] == local[q]) return b;
                return -1;
            };
            auto flush = [&](int q) {  // multiply in the deferred phase of register-bit qubit q
                if (!d.has[q]) return;
                hops.push_back(phase_fop(1u << reg_bit(q), 0, 0, std::polar(1.0, d.phi[q])));
                d.phi[q] = 0.0;
                d.has[q] = false;
            };
            for (int idx : P.phases[ph].ops) {
                const OpRec& op = ops[idx];
                if (op.kind == 2) {
                    if (op.ctrls.size() == 1 && local[op.ctrls[0]] >= 0) {
                        d.phi[op.ctrls[0]] += op.angle;
                        d.has[op.ctrls[0]] = true;
                    } else {
                        hops.push_back(encode_op(op, P, L));
                    }
                    continue;
                }
                if (op.kind == 4) {  // uncontrolled 4x4 on two register bits
                    const int q1 = op.target, q2 = op.target2;
                    int b1 = reg_bit(q1), b2 = reg_bit(q2);
                    Cx m[4][4];
                    for (int i = 0; i < 4; ++i)
                        for (int c = 0; c < 4; ++c) {
                            const double a = ((c & 1) && d.has[q1] ? d.phi[q1] : 0.0) +
                                             ((c & 2) && d.has[q2] ? d.phi[q2] : 0.0);
                            m[i][c] = Cx(op.m4[2 * (4 * i + c)], op.m4[2 * (4 * i + c) + 1]) * std::polar(1.0, a);
                        }
                    d.phi[q1] = d.phi[q2] = 0.0;
                    d.has[q1] = d.has[q2] = false;
                    if (b1 > b2) {  // index bit 0 belongs to b1: exchange the two index bits
                        Cx t[4][4];
                        const int sw[4] = {0, 2, 1, 3};
                        for (int i = 0; i < 4; ++i)
                            for (int c = 0; c < 4; ++c) t[sw[i]][sw[c]] = m[i][c];
                        for (int i = 0; i < 4; ++i)
                            for (int c = 0; c < 4; ++c) m[i][c] = t[i][c];
                        std::swap(b1, b2);
                    }
                    FOp f;
                    memset(&f, 0, sizeof(f));
                    f.kind = kDense4 + pair_of(b1, b2);
                    f.aux = (uint32_t)(m4.size() / 32);
                    for (int i = 0; i < 4; ++i)
                        for (int c = 0; c < 4; ++c) {
                            m4.push_back(m[i][c].real());
                            m4.push_back(m[i][c].imag());
                        }
                    hops.push_back(f);
                    continue;
                }
                FOp f = encode_op(op, P, L);
                const int t = op.target, b = f.rb;
                const bool uncond = f.rmask == 0 && f.tmask == 0 && f.gmask == 0;
                if (op.kind == 1) {
                    if (f.tmask || f.gmask) {  // lane- or tile-dependent exchange: no deferred phase across it
                        flush(t);
                        hops.push_back(f);
                        continue;
                    }
                    if (!d.has[t]) {
                        hops.push_back(f);
                        continue;
                    }
                    // X exp(i a x_t) = exp(i a) exp(-i a x_t) X where the controls hold
                    const double a = d.phi[t];
                    if (uncond) {
                        hops.push_back(f);
                        d.gsc *= std::polar(1.0, a);
                        d.gsc_used = true;
                        d.phi[t] = -a;
                    } else if (__builtin_popcount(f.rmask) == 1) {
                        // exp(i a (x_t xor x_c)) = exp(i a x_t) exp(i a x_c) exp(-2 i a x_t x_c):
                        // one op for the NOT and the phase of both bits
                        const int c = P.S[L.reg[__builtin_ctz(f.rmask)]];
                        d.phi[c] += a;
                        d.has[c] = true;
                        const Cx e = std::polar(1.0, -2.0 * a);
                        f.cx = true;
                        f.rmask |= 1u << b;
                        f.m[0] = e.real();
                        f.m[1] = e.imag();
                        hops.push_back(f);
                    } else {
                        hops.push_back(f);
                        hops.push_back(phase_fop(f.rmask, 0, 0, std::polar(1.0, a)));
                        hops.push_back(phase_fop(f.rmask | (1u << b), 0, 0, std::polar(1.0, -2.0 * a)));
                    }
                    continue;
                }
                // dense 2x2 (kind 0)
                Cx u[2][2];
                for (int i = 0; i < 2; ++i)
                    for (int c = 0; c < 2; ++c) u[i][c] = Cx(op.u[2 * (2 * i + c)], op.u[2 * (2 * i + c) + 1]);
                if (!uncond) {
                    flush(t);
                    hops.push_back(f);
                    continue;
                }
                if (d.has[t]) {
                    u[0][1] *= std::polar(1.0, d.phi[t]);
                    u[1][1] *= std::polar(1.0, d.phi[t]);
                }
                const CoreForm cf = core_form(u);
                if (cf.form < 0) {  // not unitary to 1e-14: the full matrix, phase folded in
                    for (int i = 0; i < 2; ++i)
                        for (int c = 0; c < 2; ++c) {
                            f.m[2 * (2 * i + c)] = u[i][c].real();
                            f.m[2 * (2 * i + c) + 1] = u[i][c].imag();
                        }
                    f.kind = kOther + b;
                    d.phi[t] = 0.0;
                    if (alone) {
                        d.has[t] = false;
                        hops.push_back(f);
                        continue;
                    }
                } else {
                    const int kind_of[4] = {kNop, kNot + 6 * b + 5, kCoreA + b, kCoreB + b};
                    f.kind = kind_of[cf.form];
                    for (int k = 0; k < 8; ++k) f.m[k] = 0.0;
                    f.m[0] = cf.k.real();
                    f.m[1] = cf.k.imag();
                    d.gsc *= cf.d0;
                    d.phi[t] = std::arg(cf.d1 / cf.d0);
                }
                hops.push_back(f);
                d.gsc_used = true;
                d.has[t] = true;
                if (++d.shrink >= max_shrink(prec)) {  // a fixed point in the op structure
                    hops.push_back(phase_fop(0, 0, 0, d.gsc));
                    d.gsc = 1.0;
                    d.shrink = 0;
                }
            }
            if (last_pass && ph + 1 == P.phases.size()) {
                // multiply in every deferred factor, in the last layout
                for (int q = 0; q < 64; ++q) {
                    if (!d.has[q]) continue;
                    const Cx e = std::polar(1.0, d.phi[q]);
                    const int j = local[q];
                    if (j < 0) {
                        hops.push_back(phase_fop(0, 0, 1ull << q, e));
                    } else {
                        int rb = -1, tb = -1;
                        for (int b = 0; b < RB; ++b)
                            if (L.reg[b] == j) rb = b;
                        for (int b = 0; b < TB; ++b)
                            if (L.thr[b] == j) tb = b;
                        FOp f = rb >= 0 ? phase_fop(1u << rb, 0, 0, e) : phase_fop(0, 1u << tb, 0, e);
                        const std::vector<int>& nr = P.phases[ph].narrow;
                        f.lane = rb < 0 || (!nr.empty() && std::find(nr.begin(), nr.end(), j) == nr.end());
                        hops.push_back(f);
                    }
                    d.phi[q] = 0.0;
                    d.has[q] = false;
                }
                if (d.gsc_used) hops.push_back(phase_fop(0, 0, 0, d.gsc));
                d.gsc = 1.0;
                d.gsc_used = false;
            }
            Fp.op_end = F.first_op[ph + 1] = (uint32_t)hops.size();
        }
        const Layout& last = P.phases.back().lay;
        F.final_transpose = (last.reg == P.store.reg && last.thr == P.store.thr) ? 0 : 1;
        FPhase& fin = F.ph[P.phases.size()];
        fill_phase(fin, last, P.store, K);
        fin.op_begin = fin.op_end = 0;
        hp.push_back(F);
    }
}

// Tile shapes compiled in: (thread bits, register bits).  LDS holds the
// whole tile, so 2^K * element size <= 160 KiB.
struct Shape {
    int TB, RB;
};
// (8, 5) in complex128 would need 32 double2 registers per thread and spills
constexpr Shape kShapes128[] = {{6, 3}, {7, 3}, {8, 3}, {8, 4}, {9, 3}, {9, 4}, {10, 3}};
constexpr Shape kShapes64[] = {{6, 3}, {7, 3}, {8, 3}, {8, 4}, {9, 3}, {8, 5}, {9, 4}, {10, 3},
                               {9, 5}, {10, 4}};

template <typename T, int TB, int RB>
hipError_t launch_cfg(hipStream_t s, void* amp, const FPass* P, const void* recs, const void* m4, uint64_t ntiles)
{
    using V = typename C2<T>::type;
    uint64_t grid = ntiles;
    const uint64_t cap = 256ull * 16;
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL((k_fused<T, TB, RB>), dim3((unsigned)grid), dim3(1 << TB), 0, s, (V*)amp, P,
                       (const FRec<T>*)recs, (const T*)m4, ntiles);
    return hipGetLastError();
}

template <typename T, int TB, int RB>
hipError_t launch_ops_cfg(hipStream_t s, void* amp, const FPass* P, const void* ops, const void* m4, uint64_t ntiles)
{
    const uint64_t grid = std::min<uint64_t>(ntiles, 256 * 16);
    hipLaunchKernelGGL((k_fused_ops<T, TB, RB>), dim3((unsigned)grid), dim3(1 << TB), 0, s,
                       (typename C2<T>::type*)amp, P, (const FOne<T>*)ops, (const T*)m4, ntiles);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_ops_pass(hipStream_t s, const FusedConfig& c, void* amp, const FPass* P, const void* ops,
                           const void* m4, uint64_t ntiles)
{
#define QS_SHAPE(tb, rb) \
    if (c.TB == tb && c.RB == rb) return launch_ops_cfg<T, tb, rb>(s, amp, P, ops, m4, ntiles);
    QS_SHAPE(6, 3) QS_SHAPE(7, 3) QS_SHAPE(8, 3) QS_SHAPE(8, 4) QS_SHAPE(9, 3)
    QS_SHAPE(9, 4) QS_SHAPE(10, 3)
    if constexpr (sizeof(T) == 4) {
        QS_SHAPE(8, 5) QS_SHAPE(10, 4)
    }
#undef QS_SHAPE
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_fused_pass(hipStream_t s, const FusedConfig& c, void* amp, const FPass* P, const void* recs,
                             const void* m4, uint64_t ntiles)
{
#define QS_SHAPE(tb, rb) \
    if (c.TB == tb && c.RB == rb) return launch_cfg<T, tb, rb>(s, amp, P, recs, m4, ntiles);
    QS_SHAPE(6, 3) QS_SHAPE(7, 3) QS_SHAPE(8, 3) QS_SHAPE(8, 4) QS_SHAPE(9, 3)
    QS_SHAPE(9, 4) QS_SHAPE(10, 3)
    if constexpr (sizeof(T) == 4) {
        QS_SHAPE(8, 5) QS_SHAPE(9, 5) QS_SHAPE(10, 4)
    }
#undef QS_SHAPE
    return hipErrorInvalidValue;
}

}  // namespace

bool fused_shape_supported(int prec, int TB, int RB)
{
    if (prec == QS_C128) {
        for (const Shape& sh : kShapes128)
            if (sh.TB == TB && sh.RB == RB) return true;
    } else {
        for (const Shape& sh : kShapes64)
            if (sh.TB == TB && sh.RB == RB) return true;
    }
    return false;
}

FusedConfig default_fused_config(int prec, int k, int n)
{
    int K = std::min(k, n);
    K = std::min(K, prec == QS_C128 ? 13 : 14);
    FusedConfig c{0, 0, kPhMax};
    if (K < 9) return c;
    static const int tb_of[15] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 6, 7, 8, 8, 8, 9};
    c.TB = tb_of[K];
    if (prec == QS_C128 && K == 13) c.TB = 9;  // 16 registers per thread, not 32
    c.RB = K - c.TB;
    return c;
}

// Tile shapes of a batch: 16 registers per thread where the single-register
// default has 8 (tiles of 10 and 11 qubits).  A batch fills the chip with
// tiles, so fewer, longer waves per tile cost nothing, each op record then
// serves twice the amplitudes, and a 10-qubit tile is one wave, which needs no
// barriers (60 registers of 10..20 qubits: 2.38 -> 2.17 ms in complex64, 3.39
// -> 2.46 in complex128).
static FusedConfig batch_config(int prec, int k, int n)
{
    FusedConfig c = default_fused_config(prec, k, n);
    if (c.TB + c.RB == 10 || c.TB + c.RB == 11) {
        c.TB = c.TB + c.RB - 4;
        c.RB = 4;
    }
    return c;
}

// The passes of a batched register, planned for the default shape of its tile
// and then laid out for `c`, whose wider phases hold one or more planned
// phases each: the order of the ops, and so every rounding, is that of the
// default shape.
//
// A register whose circuit gains op by op (op_gain) keeps the default shape,
// and `c` becomes that: 256 registers of 10 qubits are 256 waves of the wider
// one, a quarter of the SIMDs, and 100 two-qubit gates on each took 189 us there,
// 133 so.  The choice is the register's own, so that its results do not depend
// on the batch.
static std::vector<PassPlan> batch_plan(const std::vector<OpRec>& ops, int n, int prec, FusedConfig& c, bool& by_op)
{
    const int K = c.TB + c.RB;
    const FusedConfig d = default_fused_config(prec, K, K);
    const int contig = std::min(4, d.TB);
    std::vector<PassPlan> plan = plan_passes(ops, n, d.TB, d.RB, kPhMax, 1 << 12, contig);
    // controlled NOTs gain nothing here: 100 on each of 60 registers of 17 qubits
    // in complex64, 10-qubit tiles, 385 us op by op, 298 by records of the wider shape
    std::vector<int> most;
    for (size_t k = 0; k < ops.size(); ++k)
        if (ops[k].kind != 1) most.push_back((int)k);
    by_op = gains_by_op(ops, most, prec, d);
    if (by_op) c = d;
    if (d.RB == c.RB) return plan;
    for (PassPlan& P : plan) {
        std::vector<PhasePlan> wide;
        for (size_t ph = 0; ph < P.phases.size();) {
            PhasePlan W = P.phases[ph];
            std::vector<int> regs = W.lay.reg;
            auto add = [&](const std::vector<int>& more, bool all) {
                std::vector<int> u = regs;
                for (int j : more)
                    if (std::find(u.begin(), u.end(), j) == u.end() && (!wide.empty() || j >= contig)) {
                        if (!all && (int)u.size() == c.RB) break;
                        u.push_back(j);
                    }
                for (int j : more)
                    if (all && std::find(u.begin(), u.end(), j) == u.end()) return false;
                if ((int)u.size() > c.RB) return false;
                regs = u;
                return true;
            };
            W.narrow = regs;
            for (++ph; ph < P.phases.size() && add(P.phases[ph].lay.reg, true); ++ph) {
                W.ops.insert(W.ops.end(), P.phases[ph].ops.begin(), P.phases[ph].ops.end());
                W.narrow = P.phases[ph].lay.reg;
            }
            // register bits to spare: the next phase's, else the highest
            if (ph < P.phases.size()) add(P.phases[ph].lay.reg, false);
            for (int j = K - 1; j >= 0 && (int)regs.size() < c.RB; --j) add({j}, false);
            std::sort(regs.begin(), regs.end());
            W.lay.reg = regs;
            W.lay.thr.clear();
            for (int j = 0; j < K; ++j)
                if (std::find(regs.begin(), regs.end(), j) == regs.end()) W.lay.thr.push_back(j);
            wide.push_back(W);
        }
        P.phases = wide;
        P.store = coalesced(wide.back().lay, contig) ? wide.back().lay : wide.front().lay;
    }
    return plan;
}

// The 4x4 table in the register's precision.
std::vector<char> m4_bytes(const std::vector<double>& m4, int prec)
{
    std::vector<char> out;
    if (prec == QS_C128) {
        out.assign((const char*)m4.data(), (const char*)(m4.data() + m4.size()));
    } else {
        std::vector<float> f(m4.begin(), m4.end());
        out.assign((const char*)f.data(), (const char*)(f.data() + f.size()));
    }
    if (out.empty()) out.resize(sizeof(double));
    return out;
}

namespace {

// Puts FOps of a phase into records, several to one where they can share a
// dispatch.  A record runs cores (ascending register bits), then a NOT (with
// its phase) or a phase, then signs.  An op joins the open record only where
// no rounding moves: NOTs and signs are exact and may change places with ops
// on other register bits, cores and phases keep their order.  Ops with
// thread-bit or outside controls, 4x4s and controlled dense gates stand alone.
// Signs on thread and outside bits alone (sub 0) commute with everything
// inside a lane and come first.  In complex128 a sign rounds (its turn), but no
// less where it stands than where it was; the signs of a record are of pi or
// all of -pi, and none is there twice.
template <typename T>
uint32_t bundle(const FOp* ops, uint32_t count, FRec<T>* out)
{
    uint32_t n = 0, core_bits = 0, not_bits = 0, sign_bits = 0;
    bool open = false, phase = false;
    auto put = [&](int at, const FOp& f, int count_m) {
        for (int k = 0; k < count_m; ++k) out[n - 1].m[at + k] = (T)f.m[k];
    };
    auto back = [](const FOp& f) { return f.m[1] < 0.0 ? (uint32_t)kcBack : 0u; };
    auto fresh = [&](bool joinable) {
        memset(&out[n], 0, sizeof(out[n]));
        ++n;
        core_bits = not_bits = sign_bits = 0;
        phase = false;
        open = joinable;
    };
    for (uint32_t k = 0; k < count; ++k) {
        const FOp& f = ops[k];
        if (f.kind != kSign) continue;
        fresh(false);
        out[n - 1].code = kcLane | back(f) | f.tmask << 16;
        out[n - 1].gmask = f.gmask;
    }
    open = false;
    for (uint32_t k = 0; k < count; ++k) {
        const FOp& f = ops[k];
        if (f.kind == kSign || f.kind == kNop) continue;
        const int cls = f.kind & 0xe0, sub = f.kind & 31;
        const bool plain = f.tmask == 0 && f.gmask == 0;
        if (plain && (cls == kCoreA || cls == kCoreB)) {
            const uint32_t bit = 1u << sub;
            if (!open || phase || core_bits >= bit || ((not_bits | sign_bits) & bit)) fresh(true);
            FRec<T>& r = out[n - 1];
            r.code |= kcCore;
            r.multi |= cls == kCoreA ? bit : bit << 5;
            put(2 * sub, f, 2);
            core_bits |= bit;
        } else if (plain && cls == kNot) {
            const uint32_t bits = f.rmask | 1u << f.rb;
            if (!open || not_bits || phase || (sign_bits & bits)) fresh(true);
            FRec<T>& r = out[n - 1];
            r.code |= kcNot;
            r.sub = 1u << sub;
            not_bits = bits;
            if (f.cx) {
                r.code |= kcPhase;
                r.ph = 1u << (phase_sub(f.rmask) - 1);
                put(10, f, 2);
                phase = true;
            }
        } else if (plain && cls == kPhase) {
            if (!open || phase) fresh(true);
            FRec<T>& r = out[n - 1];
            r.code |= kcPhase;
            r.multi |= f.rmask << 10;
            r.ph = f.lane ? kPhAny : f.rmask ? 1u << (sub - 1) : kPhAll;
            put(10, f, 2);
            phase = true;
        } else if (plain && cls == kSign) {
            const uint32_t bit = (1u << 15) << (sub - 1);
            const bool other = sign_bits && (out[n - 1].code & kcBack) != back(f);
            if (!open || (sizeof(T) == 8 && (other || (out[n - 1].multi & bit)))) fresh(true);
            FRec<T>& r = out[n - 1];
            r.code |= kcSign | back(f);
            r.multi ^= bit;  // in complex64 the same sign twice is none
            sign_bits |= f.rmask;
        } else {
            fresh(false);
            FRec<T>& r = out[n - 1];
            r.gmask = f.gmask;
            r.code = f.tmask << 16;
            r.multi = f.rmask << 10;
            r.sub = 1u << sub;
            switch (cls) {
            case kNot:
                r.code |= kcNot;
                break;
            case kNotM:
                r.code |= kcRare | kcNotM;
                break;
            case kPhase:
                r.code |= kcPhase;
                r.ph = sub ? 1u << (sub - 1) : f.tmask ? kPhAny : kPhAll;
                put(10, f, 2);
                break;
            case kSign:
                r.code |= kcSign | back(f);
                r.multi |= (1u << 15) << (sub - 1);
                break;
            case kDense4:
                r.code |= kcRare | kcDense4;
                memcpy(&r.m[10], &f.aux, sizeof(f.aux));
                break;
            default:  // (cores have no controls)
                r.code |= kcRare | kcOther;
                put(0, f, 8);
                break;
            }
        }
    }
    return n;
}

// Device records of the ops of the passes `hp`, in the ops' slots (fewer
// records than ops: the rest of a phase's slots stay unused), and one more:
// a wave reads the record at the begin of an empty range too.  Sets the ends
// of the phases' ranges.
template <typename T>
std::vector<char> rec_bytes_t(std::vector<FPass>& hp, const std::vector<FOp>& hops)
{
    std::vector<char> out((hops.size() + 1) * sizeof(FRec<T>), 0);
    FRec<T>* r = (FRec<T>*)out.data();
    for (FPass& P : hp)
        for (int ph = 0; ph < P.nphases; ++ph) {
            FPhase& F = P.ph[ph];
            F.op_end = F.op_begin + bundle<T>(hops.data() + F.op_begin, F.op_end - F.op_begin, r + F.op_begin);
        }
    return out;
}

std::vector<char> rec_bytes(std::vector<FPass>& hp, const std::vector<FOp>& hops, int prec)
{
    return prec == QS_C128 ? rec_bytes_t<double>(hp, hops) : rec_bytes_t<float>(hp, hops);
}

template <typename T>
std::vector<char> one_bytes_t(const std::vector<FOp>& hops)
{
    std::vector<char> out(hops.size() * sizeof(FOne<T>), 0);
    FOne<T>* o = (FOne<T>*)out.data();
    for (size_t k = 0; k < hops.size(); ++k, ++o) {
        const FOp& f = hops[k];
        const int cls = f.kind & 0xe0;
        o->kind = (uint32_t)f.kind;
        o->rmask = f.rmask;
        o->tmask = f.tmask;
        o->gmask = f.gmask;
        o->aux = f.aux;
        for (int i = 0; i < 8; ++i) o->m[i] = (T)f.m[i];
        if (cls == kNot) {
            const uint32_t bit = 1u << f.rb;
            if (f.cx) o->cx = f.rb + 1;
            o->rmask = f.rmask & ~bit;
            o->kind = (o->rmask ? kNotM : kNot) + f.rb;
        } else if (cls == kPhase || cls == kSign) {
            o->kind = kPhase;
        } else if (cls == kOther && f.kind != kNop) {
            const int b = f.kind & 7;
            o->kind = f.kind & 8 ? kOneDiag + b : kOneDense + b + (f.rmask ? 5 : 0) + (f.tmask ? 10 : 0);
        }
    }
    return out;
}

std::vector<char> one_bytes(const std::vector<FOp>& hops, int prec)
{
    return prec == QS_C128 ? one_bytes_t<double>(hops) : one_bytes_t<float>(hops);
}

}  // namespace

// The passes of one circuit for one register shape and tile, as uploaded.
struct FusedPlan {
    int nbits, kind, prec, TB, RB, max_phases;
    size_t nops;
    uint64_t version;
    size_t npasses, off_recs, off_ops, off_m4;
    std::vector<char> host;  // FPass[], op records, FOnes, 4x4 table
    std::vector<bool> by_op;  // passes run by k_fused_ops
};

namespace {



// The circuit's plan for this register and tile: the one it keeps, or a new
// one, which it keeps from then on.  Planning takes 0.3 ms or more for a few
// hundred ops, ten times what their kernels take on a small register.
std::shared_ptr<const FusedPlan> fused_plan(qs_reg r, qs_circuit_s* c, const FusedConfig& cfg)
{
    std::lock_guard<std::mutex> g(c->fused_mu);
    const FusedPlan* k = c->fused.get();
    if (k && k->nbits == r->nbits && k->kind == r->kind && k->prec == r->prec && k->TB == cfg.TB && k->RB == cfg.RB &&
        k->max_phases == cfg.max_phases && k->nops == c->ops.size() && k->version == c->version)
        return c->fused;
    // a density matrix runs as its 2N-qubit vector (Eq. 2): gates on q and
    // conj on q + N, channels as 4x4 superoperators on (q, q + N), as few of
    // them as possible: a 4x4 is a full product here, and joining them across
    // ops on other qubits takes 13 qubits, eight noisy layers from 15.1 to 10.1
    // ms in complex128 and from 8.4 to 5.5 in complex64
    std::vector<OpRec> dm_ops;
    if (r->kind == QS_DENSITY) dm_ops = dm_vector_ops(c->ops, r->n, true);
    const std::vector<OpRec>& ops = r->kind == QS_DENSITY ? dm_ops : c->ops;
    const std::vector<PassPlan> plan =
        plan_passes(ops, r->nbits, cfg.TB, cfg.RB, cfg.max_phases, 1 << 12, std::min(4, cfg.TB));
    std::vector<FPass> hp;
    std::vector<FOp> hops;
    std::vector<double> m4;
    serialize(plan, ops, cfg.TB, cfg.RB, r->prec, true, hp, hops, m4);
    std::shared_ptr<FusedPlan> p = std::make_shared<FusedPlan>();
    std::vector<char> ones;
    // op by op needs four waves for each SIMD to hide its latency: 200 two-qubit
    // gates in 12-qubit tiles took the same time either way on 20 qubits in
    // complex128 (one wave) and 21 in complex64, 1361 us by records and 1147 op by
    // op on 22, and 827 and 746
    const bool full = (1ull << (r->nbits - cfg.RB)) >= 256 * 4 * 4 * 64;
    for (const PassPlan& P : plan) p->by_op.push_back(full && gains_by_op(ops, P.ops, r->prec, cfg));
    if (std::find(p->by_op.begin(), p->by_op.end(), true) != p->by_op.end()) ones = one_bytes(hops, r->prec);
    const std::vector<char> m4b = m4_bytes(m4, r->prec), recs = rec_bytes(hp, hops, r->prec);
    p->nbits = r->nbits;
    p->kind = r->kind;
    p->prec = r->prec;
    p->TB = cfg.TB;
    p->RB = cfg.RB;
    p->max_phases = cfg.max_phases;
    p->nops = c->ops.size();
    p->version = c->version;
    p->npasses = hp.size();
    const size_t pbytes = hp.size() * sizeof(FPass);
    p->off_recs = (pbytes + 15) & ~(size_t)15;
    p->off_ops = (p->off_recs + recs.size() + 15) & ~(size_t)15;
    p->off_m4 = (p->off_ops + ones.size() + 255) & ~(size_t)255;
    p->host.resize(p->off_m4 + m4b.size());
    memcpy(p->host.data(), hp.data(), pbytes);
    memcpy(p->host.data() + p->off_recs, recs.data(), recs.size());
    if (!ones.empty()) memcpy(p->host.data() + p->off_ops, ones.data(), ones.size());
    memcpy(p->host.data() + p->off_m4, m4b.data(), m4b.size());
    c->fused = p;
    return p;
}

}  // namespace

qs_status run_fused_sv(qs_reg r, qs_circuit_s* c, FusedConfig cfg, int* passes_out)
{
    if (cfg.max_phases <= 0 || cfg.max_phases > kPhMax) cfg.max_phases = kPhMax;
    const int nbits = r->nbits;
    if (cfg.TB == 0 || cfg.TB + cfg.RB > nbits) {  // too small to tile: one kernel per op
        for (const OpRec& op : c->ops) {
            qs_status s = apply_op(r, op);
            if (s) return s;
        }
        if (passes_out) *passes_out = (int)c->ops.size();
        return QS_OK;
    }
    const std::shared_ptr<const FusedPlan> plan = fused_plan(r, c, cfg);
    // stream-ordered plan buffer: no device-wide synchronisation, so
    // registers on other streams keep running
    void* dbuf = nullptr;
    hipError_t e = hipMallocAsync(&dbuf, plan->host.size(), r->stream);
    if (e != hipSuccess) return hip_error(e, "plan buffer");
    // from pageable memory the copy has left the plan when the call returns
    e = hipMemcpyAsync(dbuf, plan->host.data(), plan->host.size(), hipMemcpyHostToDevice, r->stream);
    if (e != hipSuccess) {
        (void)hipFreeAsync(dbuf, r->stream);
        return hip_error(e, "plan upload");
    }
    const FPass* dP = (const FPass*)dbuf;
    const void* dO = (const char*)dbuf + plan->off_recs;
    const void* dS = (const char*)dbuf + plan->off_ops;
    const void* dM = (const char*)dbuf + plan->off_m4;
    const uint64_t ntiles = 1ull << (nbits - cfg.TB - cfg.RB);
    qs_status st = QS_OK;
    for (size_t p = 0; p < plan->npasses && st == QS_OK; ++p) {
        st = profiled(r, QS_K_FUSED, [&](int*) {
            if (plan->by_op[p])
                return r->prec == QS_C128 ? launch_ops_pass<double>(r->stream, cfg, r->amp, dP + p, dS, dM, ntiles)
                                          : launch_ops_pass<float>(r->stream, cfg, r->amp, dP + p, dS, dM, ntiles);
            return r->prec == QS_C128 ? launch_fused_pass<double>(r->stream, cfg, r->amp, dP + p, dO, dM, ntiles)
                                      : launch_fused_pass<float>(r->stream, cfg, r->amp, dP + p, dO, dM, ntiles);
        });
    }
    // released once the passes that read it have run
    e = hipFreeAsync(dbuf, r->stream);
    if (st) return st;
    if (e != hipSuccess) return hip_error(e, "plan free");
    if (passes_out) *passes_out = (int)plan->npasses;
    return QS_OK;
}

// ===========================================================================
// Batched registers (one persistent launch)

namespace {

template <typename T, int TB, int RB, bool BYOP>
hipError_t batch_launch_t(qs_batch_s* b, const qs_batch_s::Launch& L, int init)
{
    const char* base = (const char*)b->dbuf;
    const BatchItem* items = (const BatchItem*)(base + b->off_order);
    hipLaunchKernelGGL((k_batch<T, TB, RB, BYOP>), dim3(std::min(L.count, L.grid)), dim3(1 << TB), 0, b->stream,
                       (const BatchReg*)(base + b->off_regs), items + L.off, L.count,
                       (const FPass*)(base + b->off_passes), (const void*)(base + (BYOP ? b->off_ones : b->off_ops)),
                       (const T*)(base + b->off_m4), init);
    return hipGetLastError();
}

// The shapes of batch_plan: the batch's, and the default ones of circuits that
// gain op by op.
#define QS_BATCH_SHAPES(X)                                                        \
    X(6, 3, false) X(6, 4, false) X(7, 4, false) X(8, 4, false) X(9, 4, false)    \
    X(6, 3, true) X(7, 3, true) X(8, 3, true) X(8, 4, true)                       \
    if constexpr (sizeof(T) == 4) { X(8, 5, false) X(9, 5, false) X(8, 5, true) }               \
    else { X(9, 4, true) }

template <typename T>
hipError_t batch_launch_p(qs_batch_s* b, int init)
{
    for (const qs_batch_s::Launch& L : b->launches) {
        hipError_t e = hipErrorInvalidValue;
#define QS_B(tb, rb, byop) \
    if (L.TB == tb && L.RB == rb && L.by_op == byop) e = batch_launch_t<T, tb, rb, byop>(b, L, init);
        QS_BATCH_SHAPES(QS_B)
#undef QS_B
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, int TB, int RB, bool BYOP>
int batch_occupancy()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_batch<T, TB, RB, BYOP>, 1 << TB, 0) != hipSuccess) nb = 1;
    return nb < 1 ? 1 : nb;
}

template <typename T>
int batch_occupancy_p(int TB, int RB, bool by_op)
{
#define QS_O(tb, rb, byop) \
    if (TB == tb && RB == rb && by_op == byop) return batch_occupancy<T, tb, rb, byop>();
    QS_BATCH_SHAPES(QS_O)
#undef QS_O
    return 1;
}

}  // namespace

struct BatchPlans {
    std::vector<std::vector<PassPlan>> plans;  // per register
    std::vector<bool> placeholder;             // an empty circuit's identity pass
    std::vector<bool> by_op;
};

void batch_plans_free(BatchPlans* p) { delete p; }

qs_status batch_build(qs_batch_s* b, const std::vector<qs_reg>& regs,
                      const std::vector<const std::vector<OpRec>*>& circs, int tile_qubits)
{
    int nmin = 64;
    for (qs_reg r : regs) nmin = std::min(nmin, r->n);
    const FusedConfig cfg = batch_config(b->prec, tile_qubits, 64);
    if (cfg.TB == 0 || nmin < 9)
        return set_error(QS_E_ARG, "batched registers need at least 9 qubits and a tile of 9 or more");
    b->TB = cfg.TB;
    b->RB = cfg.RB;
    std::vector<FPass> hp;
    std::vector<FOp> hops;
    std::vector<double> m4;
    std::vector<BatchReg> hr(regs.size());
    std::vector<ProbItem> pieces;
    int maxpasses = 0;
    b->reg_TB.assign(regs.size(), 0);
    b->reg_RB.assign(regs.size(), 0);
    std::vector<uint64_t> per_item(regs.size());
    std::unique_ptr<BatchPlans> bp(new BatchPlans());
    b->reg_op_begin.assign(regs.size(), 0);
    b->reg_op_count.assign(regs.size(), 0);
    b->reg_m4_begin.assign(regs.size(), 0);
    b->reg_m4_count.assign(regs.size(), 0);
    for (size_t i = 0; i < regs.size(); ++i) {
        std::vector<OpRec> none;
        const std::vector<OpRec>* ops = circs[i];
        if (ops->empty()) {  // an empty circuit still gets one (identity) pass, which initialises
            OpRec id{};
            id.kind = 2;
            id.ctrls = {0};
            id.angle = 0.0;
            none.push_back(id);
            ops = &none;
        }
        // a register narrower than the batch tile is one tile of its own width
        FusedConfig rc = regs[i]->n >= cfg.TB + cfg.RB ? cfg : batch_config(b->prec, regs[i]->n, regs[i]->n);
        bool by_op;
        std::vector<PassPlan> plan = batch_plan(*ops, regs[i]->n, b->prec, rc, by_op);
        b->reg_TB[i] = rc.TB;
        b->reg_RB[i] = rc.RB;
        bp->by_op.push_back(by_op);
        per_item[i] = 1ull << (regs[i]->n - (rc.TB + rc.RB));  // tile count, for now
        hr[i].amp = regs[i]->amp;
        hr[i].n = regs[i]->n;
        hr[i].pass0 = (uint32_t)hp.size();
        hr[i].npasses = (int)plan.size();
        hr[i].pad = 0;
        hr[i].logc = (uint32_t)std::min(12, std::max(0, regs[i]->n - 12));
        hr[i].piece0 = (uint32_t)pieces.size();
        for (uint32_t k = 0; k < 1u << hr[i].logc; ++k) pieces.push_back(ProbItem{(uint32_t)i, k});
        maxpasses = std::max(maxpasses, (int)plan.size());
        b->reg_op_begin[i] = hops.size();
        b->reg_m4_begin[i] = m4.size();
        serialize(plan, *ops, rc.TB, rc.RB, b->prec, false, hp, hops, m4);
        b->reg_op_count[i] = hops.size() - b->reg_op_begin[i];
        b->reg_m4_count[i] = m4.size() - b->reg_m4_begin[i];
        bp->plans.push_back(std::move(plan));
        bp->placeholder.push_back(ops == &none);
    }
    // tiles per work item: up to 16, fewer when the batch holds too few
    // tiles to give the 256 CUs about 64 items each (60 registers of 10..20
    // qubits in complex64, kernel times of one build: 2.17 ms with 8 items per
    // CU, 1.58 with 16, 1.39 with 64 or more; now 1.55, and 1.60 by the clock)
    uint64_t total_tiles = 0;
    for (uint64_t t : per_item) total_tiles += t;
    const uint64_t per = std::max<uint64_t>(1, std::min<uint64_t>(16, total_tiles / 16384));
    // op by op about 8 waves for each SIMD: tiles of a register one after the other find
    // its ops in the scalar cache (32 registers of 20 qubits in complex64, 100
    // controlled gates on each: 1.55 ms with one tile an item, 0.97 with five)
    for (size_t i = 0; i < regs.size(); ++i) {
        const uint64_t items = 8192 >> (b->reg_TB[i] > 6 ? b->reg_TB[i] - 6 : 0);
        const uint64_t per_ops = std::min<uint64_t>(16, (total_tiles + items - 1) / items);
        per_item[i] = std::min(per_item[i], bp->by_op[i] ? per_ops : per);
    }
    if (hp.empty()) hp.push_back(FPass{});
    b->circ_ops.assign(circs.begin(), circs.end());
    b->host_ops = rec_bytes(hp, hops, b->prec);
    if (std::find(bp->by_op.begin(), bp->by_op.end(), true) != bp->by_op.end()) b->host_ones = one_bytes(hops, b->prec);
    b->reg_pass_begin.assign(regs.size(), 0);
    for (size_t i = 0; i < regs.size(); ++i) b->reg_pass_begin[i] = hr[i].pass0;
    b->host_m4 = m4;
    const std::vector<char> m4b = m4_bytes(m4, b->prec);
    // items level by level; within a level the largest registers first
    std::vector<uint32_t> byn(regs.size());
    for (size_t i = 0; i < byn.size(); ++i) byn[i] = (uint32_t)i;
    std::stable_sort(byn.begin(), byn.end(), [&](uint32_t a, uint32_t c) { return hr[a].n > hr[c].n; });
    std::vector<BatchItem> items;
    b->launches.clear();
    struct Kernel {
        int TB, RB;
        bool by_op;
        bool operator==(const Kernel& o) const { return TB == o.TB && RB == o.RB && by_op == o.by_op; }
    };
    auto kernel_of = [&](size_t i) { return Kernel{b->reg_TB[i], b->reg_RB[i], bp->by_op[i]}; };
    std::vector<Kernel> kernels{{cfg.TB, cfg.RB, false}};  // distinct ones, the batch shape's first
    for (size_t i = 0; i < regs.size(); ++i)
        if (std::find(kernels.begin(), kernels.end(), kernel_of(i)) == kernels.end()) kernels.push_back(kernel_of(i));
    for (int p = 0; p < maxpasses; ++p) {
        for (const Kernel& k : kernels) {
            const int off = (int)items.size();
            for (uint32_t i : byn) {
                if (p >= hr[i].npasses || !(kernel_of(i) == k)) continue;
                const uint64_t ntiles = 1ull << (hr[i].n - (k.TB + k.RB)), per = per_item[i];
                for (uint64_t t0 = 0; t0 < ntiles; t0 += per)
                    items.push_back(BatchItem{i, (uint32_t)p, (uint32_t)t0, (uint32_t)std::min(ntiles, t0 + per)});
            }
            const int count = (int)items.size() - off;
            if (count == 0) continue;
            const int per_cu = b->prec == QS_C128 ? batch_occupancy_p<double>(k.TB, k.RB, k.by_op)
                                                  : batch_occupancy_p<float>(k.TB, k.RB, k.by_op);
            b->launches.push_back({k.TB, k.RB, k.by_op, off, count, (int)(256L * per_cu)});
        }
    }
    b->nitems = (int)items.size();
    auto align = [](size_t x) { return (x + 255) & ~(size_t)255; };
    b->off_regs = 0;
    b->off_order = align(hr.size() * sizeof(BatchReg));
    b->off_passes = align(b->off_order + items.size() * sizeof(BatchItem));
    b->off_ops = align(b->off_passes + hp.size() * sizeof(FPass));
    b->off_ones = align(b->off_ops + b->host_ops.size());
    b->off_m4 = align(b->off_ones + b->host_ones.size());
    b->off_pieces = align(b->off_m4 + m4b.size());
    b->npieces = (int)pieces.size();
    const size_t total = align(b->off_pieces + pieces.size() * sizeof(ProbItem));
    b->off_partials = total;  // written by the device only
    std::vector<char> host(total, 0);
    memcpy(host.data() + b->off_pieces, pieces.data(), pieces.size() * sizeof(ProbItem));
    memcpy(host.data() + b->off_regs, hr.data(), hr.size() * sizeof(BatchReg));
    memcpy(host.data() + b->off_order, items.data(), items.size() * sizeof(BatchItem));
    memcpy(host.data() + b->off_passes, hp.data(), hp.size() * sizeof(FPass));
    memcpy(host.data() + b->off_ops, b->host_ops.data(), b->host_ops.size());
    if (!b->host_ones.empty()) memcpy(host.data() + b->off_ones, b->host_ones.data(), b->host_ones.size());
    memcpy(host.data() + b->off_m4, m4b.data(), m4b.size());
    // stream-ordered allocation and upload: creating a batch does not wait
    // for work on other streams (a plain free or a synchronous copy would)
    b->host_plan = std::move(host);
    hipError_t e = hipMallocAsync(&b->dbuf, total + pieces.size() * 4 * sizeof(double), b->stream);
    if (e != hipSuccess) return hip_error(e, "batch plan buffer");
    e = hipMemcpyAsync(b->dbuf, b->host_plan.data(), total, hipMemcpyHostToDevice, b->stream);
    if (e != hipSuccess) return hip_error(e, "batch plan upload");
    b->grid = b->launches.empty() ? 1 : b->launches.front().grid;
    b->passes_total = (int)hp.size();
    b->plans = bp.release();
    return QS_OK;
}

qs_status batch_update(qs_batch_s* b)
{
    // lower every register's plan again with the circuits' current values: the
    // structure (and so the slots of its ops) is unchanged; the kernel data
    // (matrices, core coefficients, deferred phases) and the phases' ranges of
    // records follow the parameters
    const size_t rsz = b->prec == QS_C128 ? sizeof(FRec<double>) : sizeof(FRec<float>);
    const size_t osz = b->prec == QS_C128 ? sizeof(FOne<double>) : sizeof(FOne<float>);
    FPass* passes = (FPass*)(b->host_plan.data() + b->off_passes);
    for (size_t i = 0; i < b->regs.size(); ++i) {
        if (b->plans->placeholder[i]) continue;
        std::vector<FPass> hp;
        std::vector<FOp> hops;
        std::vector<double> m4;
        serialize(b->plans->plans[i], *b->circ_ops[i], b->reg_TB[i], b->reg_RB[i], b->prec, false, hp, hops, m4);
        if (hops.size() != b->reg_op_count[i] || m4.size() != b->reg_m4_count[i])
            return set_error(QS_E_ARG, "a batched circuit changed its structure");
        for (FOp& f : hops)
            if ((f.kind & 0xe0) == kDense4) f.aux += (uint32_t)(b->reg_m4_begin[i] / 32);
        const std::vector<char> recs = rec_bytes(hp, hops, b->prec);
        memcpy(b->host_ops.data() + b->reg_op_begin[i] * rsz, recs.data(), hops.size() * rsz);
        if (b->plans->by_op[i]) {
            const std::vector<char> ones = one_bytes(hops, b->prec);
            memcpy(b->host_ones.data() + b->reg_op_begin[i] * osz, ones.data(), ones.size());
        }
        const uint32_t first = (uint32_t)b->reg_op_begin[i];
        for (size_t p = 0; p < hp.size(); ++p) {
            FPass& P = passes[b->reg_pass_begin[i] + p];
            for (int ph = 0; ph < hp[p].nphases; ++ph) {
                P.ph[ph].op_begin = first + hp[p].ph[ph].op_begin;
                P.ph[ph].op_end = first + hp[p].ph[ph].op_end;
            }
            for (int ph = 0; ph <= hp[p].nphases; ++ph) P.first_op[ph] = first + hp[p].first_op[ph];
        }
        std::copy(m4.begin(), m4.end(), b->host_m4.begin() + b->reg_m4_begin[i]);
    }
    // from pageable memory the copies have left the host tables when the
    // calls return; on the batch stream they follow earlier runs and precede
    // later ones
    hipError_t e = hipMemcpyAsync((char*)b->dbuf + b->off_ops, b->host_ops.data(), b->host_ops.size(),
                                  hipMemcpyHostToDevice, b->stream);
    if (e != hipSuccess) return hip_error(e, "batch parameter upload");
    if (!b->host_ones.empty()) {
        e = hipMemcpyAsync((char*)b->dbuf + b->off_ones, b->host_ones.data(), b->host_ones.size(),
                           hipMemcpyHostToDevice, b->stream);
        if (e != hipSuccess) return hip_error(e, "batch parameter upload");
    }
    e = hipMemcpyAsync((char*)b->dbuf + b->off_passes, passes, (size_t)b->passes_total * sizeof(FPass),
                       hipMemcpyHostToDevice, b->stream);
    if (e != hipSuccess) return hip_error(e, "batch parameter upload");
    if (!b->host_m4.empty()) {
        b->host_m4b = m4_bytes(b->host_m4, b->prec);
        e = hipMemcpyAsync((char*)b->dbuf + b->off_m4, b->host_m4b.data(), b->host_m4b.size(), hipMemcpyHostToDevice,
                           b->stream);
        if (e != hipSuccess) return hip_error(e, "batch parameter upload");
    }
    return QS_OK;
}

hipError_t batch_launch(qs_batch_s* b, int init)
{
    return b->prec == QS_C128 ? batch_launch_p<double>(b, init) : batch_launch_p<float>(b, init);
}

hipError_t batch_probs_launch(qs_batch_s* b, int q, double* dev_out)
{
    char* base = (char*)b->dbuf;
    const BatchReg* regs = (const BatchReg*)(base + b->off_regs);
    const ProbItem* items = (const ProbItem*)(base + b->off_pieces);
    double* partials = (double*)(base + b->off_partials);
    if (b->prec == QS_C128)
        hipLaunchKernelGGL(k_batch_probs<double>, dim3(b->npieces), dim3(256), 0, b->stream, regs, items, q, partials);
    else
        hipLaunchKernelGGL(k_batch_probs<float>, dim3(b->npieces), dim3(256), 0, b->stream, regs, items, q, partials);
    hipLaunchKernelGGL(k_batch_probs_final, dim3(b->count), dim3(64), 0, b->stream, regs, partials, dev_out);
    return hipGetLastError();
}

}  // namespace qs
