// Host-side helpers shared by the library's entry-point sources.
#pragma once

#include <string>

#include "alm_bm.h"

namespace almbm {

// Records msg as the calling thread's last error (alm_bm_last_error) and
// returns s.
alm_bm_status set_error(alm_bm_status s, const std::string& msg);

// Default grid of the row kernels for n rows: one block per 16 rows up to 512 blocks,
// beyond that one per 64 rows up to 1024; at least 8, a multiple of 8 (one share per XCD).
int row_blocks(long n);

}  // namespace almbm

// For tests: the eigenvalue run of alm_bm_lanczos_min_eig with a chosen number of
// restarts and order of sums (ordered = 0: as a solve runs it).  v: device n.  tri: host
// 2 x max_iter, the last pass's alpha, then its beta.  out: host, {theta, residual, steps
// of all passes, steps that the last pass enqueued}.  Synchronises the stream.
extern "C" alm_bm_status alm_bm_internal_lanczos(alm_bm_problem* p, const double* y, int32_t max_iter, double tol,
                                                 uint64_t seed, int32_t restarts, int32_t ordered, double* v,
                                                 double* tri, double* out, hipStream_t st);
