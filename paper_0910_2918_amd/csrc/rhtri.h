// Roberts-Higham from a tridiagonal start matrix (rhtri.hip), called by
// rh.hip under its lock.
#pragma once

#include "nk_internal.h"

namespace nk {

// RH steps that tri_rh_run takes in closed form for this batch, 0 = none
int tri_rh_steps(int batch, int ld, int maxn, int scaling, int maxit);

// S (dense S_0 = H of every matrix, leading dimension ld) <- S_L after L
// steps; sing: [batch] zeroed flags; sched: [batch][nsched] learned corrections or null.  *sums (host
// memory, valid once the stream has been waited for): per matrix the pairs
// |S_{n+1} - mu_n S_n|^2, |S_{n+1}|^2 of the L steps, then nonzero if the
// closed form does not cover the matrix (rhtri.hip); neither S nor the sums
// then mean anything, and tri_rh_retake puts S_0 back.  Returns 1, with S
// unchanged, when there is no memory for the workspace.
int tri_rh_run(int batch, int ld, int maxn, const int* nvec, int* sing, const TriIn& h, C64* S, int scaling,
               const double* sched, int nsched, int L, const double** sums, hipStream_t st);

// After tri_rh_run with the same batch and L: S <- S_m, m = steps[b] (device
// array) where it is positive, S_0 where it is negative, unchanged where zero.
int tri_rh_retake(int batch, int ld, int maxn, const int* nvec, const int* steps, const TriIn& h, C64* S, int L,
                  hipStream_t st);

}  // namespace nk
