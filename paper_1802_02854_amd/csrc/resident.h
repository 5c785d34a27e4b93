// Krylov sequences of small clusters, each run whole by one workgroup, and the
// multi-shift update of finished coefficient lists.
#pragma once

#include "kernels.h"

namespace ftk {

// clusters whose vector, or one plane of it, a workgroup keeps in its registers and LDS
constexpr int kResidentMinSites = 6;
constexpr int kResidentMaxSites = 14;
constexpr int kResidentPlanes = 13;  // from here on a plane at a time, with a carry buffer
constexpr int kFewMinSites = 13;    // from here on a few sequences run in lockstep instead
// whether sequences of op run resident (by size, unless a form of H v is forced)
bool resident(const HvOp &op);

// what the start vectors of a run are made from
enum ResidentLoad {
    kLoadSpin,  // S^alpha_Q phi: sq[op]
    kLoadPair,  // polarization vector op % 4 of (A phi, B phi): a[op / 4], b[op / 4]
};
struct ResidentSeq {
    const double2 *phi;
    int op;
    int out;          // row of the sequence's state and coefficients
    double shift_re;  // E_m
};

struct ResidentRun {
    const ResidentSeq *seq;  // device, one per workgroup
    const SqParams *sq;      // device
    const SpinOpParams *a, *b;
    double *chi;             // the start vectors, 2 * 2^N doubles each; NULL: phi itself
    SeqState *st;            // [rows]
    double *alpha, *beta;    // [rows][stride]
    int stride;
    double tol;              // breakdown threshold
    int k0, k1;              // steps [k0, k1); k0 > 0 resumes from carry
    double *carry;           // per sequence w_{k-1}, w_{k-2} (4 * 2^N doubles); NULL for a whole run
                             // below kResidentPlanes sites
    double *vout;            // NULL, or per sequence the vectors w_{k-1} of these steps...
    size_t vstride;          // ... this many doubles apart
};
// chi of n_seq sequences
void launch_start_vectors(int n_sites, ResidentLoad load, const ResidentRun &run, int n_seq, hipStream_t s);
// n_seq sequences of the steps given, one workgroup each
void launch_resident(const HvOp &op, const ResidentRun &run, int n_seq, hipStream_t s);

// The multi-shift update of finished sequences (rows 0 .. n_seq - 1) from their
// recorded coefficients: g = norm2 * G per shift, st->max_resid from the last step.
struct ShiftRun {
    SeqState *st;
    const double *alpha, *beta;  // [n_seq][stride]
    int stride;
    const double *omega;
    int n_omega;
    double eta;
    double *g;  // [n_seq][n_omega] complex
};
void launch_shifts(const ShiftRun &run, int n_seq, hipStream_t s);
// The same for the steps [k0, k1) of sequences that stop once the largest residual
// over the shifts, per unit right-hand side, is <= rtol: a sequence that does so at
// one of them ends there (done, its step count).  sh [n_seq][n_omega] holds the
// shifts' state between calls; g is written every time.
void launch_shifts_until(const ShiftRun &run, int k0, int k1, double rtol, ShiftState *sh, int n_seq, hipStream_t s);

// debug build: the bounds checks' counters of these kernels (device_checks.h)
bool resident_checks_read(unsigned int out[3], bool clear);

}  // namespace ftk
