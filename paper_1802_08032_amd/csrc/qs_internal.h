// Internal declarations shared by the C-ABI layer and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <complex>

#include "qstate.h"

namespace qs {

// Bits to insert into a compact loop index, at the positions set in `at`.
// After insertion the bits in `ones` are set (controls), the rest are 0.  Two
// words: as a list of positions the kernels read them one after the other
// through the scalar cache before they could form an address, which the
// smallest registers saw.
struct BitInsert {
    uint64_t at, ones;
};

// 2x2 complex matrix, row-major, real/imag interleaved.
template <typename T>
struct Mat2 {
    T m[8];
};

struct Launch {
    hipStream_t stream;
    int device;
};

// Builds the insertion spec for the given positions (any order) and ones mask.
BitInsert make_insert(const int* positions, int count, uint64_t ones);

// --- state-vector kernels -------------------------------------------------
// Every amplitude 0 except `index`, which becomes (re, im).  Write-only.
template <typename T> hipError_t launch_init_basis(const Launch& L, void* amp, uint64_t len, uint64_t index,
                                                   double re, double im);
template <typename T> hipError_t launch_gate(const Launch& L, void* amp, int nbits, int t,
                                             const int* ctrls, int nc, const Mat2<T>& u, int* klass);
template <typename T> hipError_t launch_not(const Launch& L, void* amp, int nbits, int t,
                                            const int* ctrls, int nc);
// Multiply by f every amplitude with all bits of `mask` set, except those
// that also have all bits of `skip` set (skip == 0: no exception).
template <typename T> hipError_t launch_phase(const Launch& L, void* amp, int nbits, uint64_t mask,
                                              uint64_t skip, double fre, double fim);

// --- density-matrix kernels ------------------------------------------------
// Phase f on the rows with all bits of `rmask` set, conj(f) on the columns.
template <typename T> hipError_t launch_dm_phase(const Launch& L, void* rho, int N, uint64_t rmask, double fre,
                                                 double fim);
template <typename T> hipError_t launch_dm_gate(const Launch& L, void* rho, int N, int t,
                                                const int* ctrls, int nc, const Mat2<T>& u);
template <typename T> hipError_t launch_dm_channel(const Launch& L, void* rho, int N, int t,
                                                   int channel, double p);

// --- reductions and collapse ----------------------------------------------
// Sum of |alpha|^2 split by bit q (q < 0: one total sum in out[0]).  Writes
// {sum over bit q == 0, sum over bit q == 1} as doubles to `dev_out`.
// (device or pinned host memory).  `partials` must hold 2 * 2 * kReduceBlocks doubles.
constexpr int kReduceBlocks = 1024;
template <typename T> hipError_t launch_prob_sv(const Launch& L, const void* amp, int nbits, int q,
                                                double* partials, double* dev_out);
// Sum of |alpha|^2 over the indices whose bit q equals `outcome`, reading
// only those (half the state when q is at least the line bits: 3 for
// complex128, 4 for complex64).  Writes {sum, 0} to `dev_out`.
template <typename T> hipError_t launch_prob_half_sv(const Launch& L, const void* amp, int nbits, int q,
                                                     int outcome, double* partials, double* dev_out);
template <typename T> hipError_t launch_prob_dm(const Launch& L, const void* rho, int N, int q,
                                                double* partials, double* dev_out);
// out[j] = sum of part[i * cols + j] over rows i = 0..rows-1 (compensated,
// in row order).
hipError_t launch_sum_columns(const Launch& L, const double* part, int rows, int cols, double* out);
template <typename T> hipError_t launch_collapse_sv(const Launch& L, void* amp, int nbits, int q,
                                                    int outcome, double scale);
template <typename T> hipError_t launch_collapse_dm(const Launch& L, void* rho, int N, int q,
                                                    int outcome, double scale);

// Register scratch (device doubles): reduction partials, then
// two k-qubit matrices of up to 32 x 32 complex entries (a gate and its
// conjugate, or a superoperator).
constexpr int kScratchMatOff = 4 * kReduceBlocks;
constexpr int kScratchMatDoubles = 2 * 32 * 32 * 2;
constexpr int kScratchDoubles = kScratchMatOff + kScratchMatDoubles;

// --- k-qubit groups, initialisation variants, overlaps ---------------------
// Replace every group of 2^k amplitudes (k = 1..5 targets; matrix index bit j
// <-> targets[j]) whose control bits are all 1 by m times it; m is 2^k x 2^k,
// row-major, rounded to T once.  dev_m: device memory for 2^k x 2^k complex T
// pairs (written here, on the stream, for k >= 4).
template <typename T> hipError_t launch_group_gate(const Launch& L, void* amp, int nbits, const int* targets,
                                                   int k, const int* ctrls, int nc, const std::complex<double>* m,
                                                   T* dev_m);
// rho <- U rho U^dagger, U = m on two targets (4 x 4, as above): U on the rows
// and conj(U) on the columns.
template <typename T> hipError_t launch_dm_two(const Launch& L, void* rho, int N, const int* targets,
                                               const std::complex<double>* m);
// Every amplitude set to (re, im).  Write-only.
template <typename T> hipError_t launch_init_fill(const Launch& L, void* amp, uint64_t len, double re, double im);
// rho = |psi><psi| in the Eq. 2 layout; psi holds 2^N amplitudes.
template <typename T> hipError_t launch_dm_from_pure(const Launch& L, void* rho, int N, const void* psi);
// dev_out = {Re, Im} of sum_i conj(a_i) b_i (compensated, in double).
template <typename T> hipError_t launch_inner_sv(const Launch& L, const void* a, const void* b, int nbits,
                                                 double* partials, double* dev_out);
// dev_out = {Re, Im} of <psi| rho |psi> (compensated, in double).
template <typename T> hipError_t launch_fid_dm(const Launch& L, const void* rho, int N, const void* psi,
                                               double* partials, double* dev_out);

// --- measure-all ----------------------------------------------------------
constexpr int kHistBlocks = 256;
constexpr int kMaxMeasured = 64;  // qubits
struct Draws {
    double u[kMaxMeasured];
};
// What one group of qubits hands to the next (device memory).
struct MeasureState {
    double g, re, im;
    uint64_t pattern, pos;
    int err, pad;
};
// Device memory for the stages (in doubles), and pinned host memory for what
// they return: an error flag, the probabilities, the outcomes.
constexpr size_t kMeasureDoubles = 2 * 1024 * (size_t)kHistBlocks + 2 * 1024 + sizeof(MeasureState) / sizeof(double);
constexpr size_t kHostDoubles = 1 + 2 * kMaxMeasured;
// Outcomes of qubits shift .. min(shift + 10, n) - 1, after the stages before
// it on the same stream and with the same `buf`; the last stage also forms
// the entry that launch_measure_basis writes.
template <typename T> hipError_t launch_measure_stage(const Launch& L, const void* amp, int n, bool dm, int shift,
                                                      const Draws& draws, double* buf, double* res);
template <typename T> hipError_t launch_measure_basis(const Launch& L, void* amp, uint64_t len, const double* buf);
// dst <- src, `len` amplitudes.
template <typename T> hipError_t launch_copy(const Launch& L, void* dst, const void* src, uint64_t len);

}  // namespace qs
