// chains.hpp -- filter and smoother by overlapped chains: models that change at
// every step, and packed sequences with a model each (nx, ny <= 4).
//
// A filter that follows its state forgets where it started.  The sequences are
// cut into chains of l steps; every chain runs the sequential recursion from
// `warm` steps before it, started from the prior, and the moments it enters its
// own steps with are compared with those its predecessor ended with.  The first
// chain of a sequence starts from the prior itself, so where all of them agree
// to rounding every chain has the sequential filter's values.  Chains that do
// not agree run once more from the predecessor's end; if one still differs (see
// kSame in chains.hip), or a factorisation failed, the flag ctl[0] is cleared and the general scan
// kernels, which follow in the stream and return at once otherwise, do the
// work.  The smoother does the same backwards.  With one time-invariant model per
// sequence, covariances that have settled are not run again: there a chain is the
// means alone.
#pragma once
#include "pks_internal.h"

namespace pks {
namespace chains {

constexpr int kState = 32;           // doubles of a chain's moments: tiles of P and of the mean
constexpr int kModel = 96;           // doubles of a time-invariant model's settled values: six tiles

struct Args {
    int nx, ny, B;
    int smooth;                  // filter + smoother (else the filter alone)
    int reset;
    int each;                    // one prior per sequence
    int64_t total;
    const int64_t* offsets;      // device [B+1]; nullptr: one sequence
    const double *F, *u, *Q, *H, *d, *R, *m0, *P0;     // one row per step (time-varying) or per sequence
    const void* y;
    void *m, *P, *ms, *Ps;
    int* status;
    int* ctl;                    // [0] 1: this path has done the work; [4], [5], [6] notes of the pilots
    int64_t l, warm, max_chains;
    int64_t* first;              // [B+1] chains of the sequences before
    int* sequence;               // [chains] a chain's sequence (packed sequences)
    double* model;               // [B][kModel] settled values (time-invariant models)
    double near;                 // see kSame (time-varying models)
    int* forgets;                // [chains] the first difference was within `near`
    int* head;                   // [B][2] steps after which P and Ps have settled, in 16 (0: they have not)
    double *entry, *end[2];      // [chains][kState] moments that a chain entered and ended with
};

bool applies(int nx, int ny, int32_t B, int64_t total, bool mixed, bool tv, bool smooth);
bool layout(Args& a, char* base, size_t bytes, bool tv);
hipError_t launch(const Args& a, bool mixed, bool tv, hipStream_t s);

}  // namespace chains
}  // namespace pks
