// Spin projection, neighbour and job-table helpers shared by the stencil
// kernels (stencil.hip, split.hip).
#pragma once
#include "device_util.h"

namespace ovl {

// Chiral basis: gamma_mu = [[0, A_mu], [A_mu^dag, 0]] with A_k = -i sigma_k,
// A_4 = 1.  For the lower half-spinor d = (psi_2, psi_3):
//   (1 -+ gamma_mu) psi = [ h ; -+ A^dag h ],  h = psi_up -+ A_mu d,
// so each hop moves a 2-spin x 3-colour half-spinor through the link.

// h = psi_up - A d (forward, sg = -1) or psi_up + A d (backward, sg = +1)
template <typename R>
__device__ __forceinline__ void project(int mu, R sg, cx<R> p0, cx<R> p1, cx<R> p2, cx<R> p3,
                                        cx<R>& h0, cx<R>& h1) {
    cx<R> a0, a1;  // A_mu (p2, p3)
    switch (mu) {
        case 0: a0 = tmi(p3); a1 = tmi(p2); break;
        case 1: a0 = -p3; a1 = p2; break;
        case 2: a0 = tmi(p2); a1 = ti(p3); break;
        default: a0 = p2; a1 = p3; break;
    }
    h0 = p0 + sg * a0;
    h1 = p1 + sg * a1;
}

// acc_up += u ; acc_dn += sg * A_mu^dag u
template <typename R>
__device__ __forceinline__ void reconstruct(int mu, R sg, cx<R> (&acc)[4][3],
                                            const cx<R> (&u)[2][3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<R> u0 = u[0][c], u1 = u[1][c];
        cx<R> b0, b1;  // A^dag (u0, u1)
        switch (mu) {
            case 0: b0 = ti(u1); b1 = ti(u0); break;
            case 1: b0 = u1; b1 = -u0; break;
            case 2: b0 = ti(u0); b1 = tmi(u1); break;
            default: b0 = u0; b1 = u1; break;
        }
        acc[0][c] = acc[0][c] + u0;
        acc[1][c] = acc[1][c] + u1;
        acc[2][c] = acc[2][c] + sg * b0;
        acc[3][c] = acc[3][c] + sg * b1;
    }
}

__device__ __forceinline__ uint32_t nbr(const Geom& g, uint32_t s, const int (&coord)[4], int mu,
                                        bool fwd) {
    const uint32_t sd = (uint32_t)g.stride[mu];
    const int L = g.L[mu];
    const int cm = coord[mu];
    if (fwd) return (cm == L - 1) ? s - (uint32_t)(L - 1) * sd : s + sd;
    return (cm == 0) ? s + (uint32_t)(L - 1) * sd : s - sd;
}

// Block -> (job, tile) of a job-table stencil launch.  Job j owns blocks
// [sten_b0, sten_b0 + pad8(sten_nb)) of the grid, sten_b0 a multiple of 8,
// so its blocks go round-robin over all eight XCDs like those of a launch of
// its own (dispatch assigns block b to XCD b mod 8), and within the job the
// XCD-aware remap groups neighbouring tiles on one XCD.  A job that has
// finished, or iterates in the other precision, thus leaves every XCD, not
// a contiguous few, to the jobs still running.  Returns false for the
// job's padding blocks and for jobs in the other precision phase.
__device__ __forceinline__ bool job_tile(const JobDesc* __restrict__ jobs, int njobs, int f,
                                         int& j, unsigned& tile) {
    const unsigned b = blockIdx.x;
    j = 0;
    while (j + 1 < njobs && b >= (unsigned)jobs[j + 1].sten_b0[f]) ++j;
    const JobDesc& J = jobs[j];
    if (J.phase != f) return false;  // this job iterates in the other precision
    const unsigned nb = (unsigned)J.sten_nb[f];
    tile = uniform(xcd_remap(b - (unsigned)J.sten_b0[f], (nb + 7u) & ~7u));
    return tile < nb;
}

}  // namespace ovl
