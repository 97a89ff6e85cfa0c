// Coarse-grid solver of the pressure preconditioner: ten Jacobi-PCG
// iterations from zero on the assembled N = 1 operator (Karp et al., arXiv
// 2207.07098, Sec. II-B).
#pragma once

#include <vector>

#include "sem_internal.h"

namespace sem {

// Entries of a row are stored slot-major ([width][ld], ld rows padded to the
// alignment), padded with (own row, 0.0) to a multiple of kCoarseUnroll.
constexpr int kCoarseIterations = 10;
constexpr int kCoarseUnroll = 9;

struct CoarsePlan {
    int64_t n = 0, ld = 0;            // rows (coarse unique nodes), padded
    int width = 0;                    // entries per row
    std::vector<int32_t> ids;         // [width][ld] column of every entry
    // device (inside the caller's workspace)
    int32_t *idx = nullptr;
    double *val = nullptr, *dinv = nullptr;
    double *r = nullptr, *z = nullptr, *w = nullptr, *p = nullptr;
    double *part = nullptr;
    CgState *state = nullptr;         // one per half iteration; the last is the result
    double *b = nullptr, *x = nullptr;  // right-hand side (cleared by the solve), solution
};

// Sparsity pattern from the connectivity of the N = 1 context (host).
void coarse_pattern(sem_ctx coarse, CoarsePlan &plan);
size_t coarse_bytes(const CoarsePlan &plan);
// Takes its arrays from ws, uploads the pattern and assembles the operator
// from the coarse context's factors; clears the right-hand side b.
hipError_t coarse_bind(sem_ctx coarse, CoarsePlan &plan, char *ws, double *b, double *x,
                       hipStream_t s);
// x = ten PCG iterations on A x = b; b is zero afterwards.  Asynchronous.  A
// non-finite value makes x NaN and is left in coarse_result's status.
hipError_t coarse_solve(const CoarsePlan &plan, hipStream_t s);
const CgState *coarse_result(const CoarsePlan &plan);

}  // namespace sem
