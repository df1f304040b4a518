// H_W on the caller's vectors (HIP, gfx950): out = H_W in in one launch on the
// row-major layout [n][V][spin][colour] of the C ABI, with no packing pass.
//
// Four neighbouring lanes share a site, lane a holding spin a: a site's 192
// bytes are read and written by one quad of lanes in three 16-byte accesses,
// so a wave's accesses cover whole lines without a transposition.  The spin
// projection needs one exchange within the quad (a DPP quad permutation), the
// reconstruction another.  Lanes 0 and 1 take the forward hop of a direction,
// lanes 2 and 3 the backward hop:
//   forward  h = psi_up - A psi_dn      (lanes 0, 1), u = U_mu(x) h:
//            acc_up += u, acc_dn -= A^dag u;
//   backward h = psi_dn + A^dag psi_up  (lanes 2, 3), u = U_mu(x-mu)^dag h:
//            acc_dn += u, acc_up += A u,
// (1 + gamma_mu) psi being [A h ; h] as well as [h' ; A^dag h'].  In every
// lane the partner's term enters with one phase phi and returns with -phi:
//   phi = i, s1, i s1, s3 for mu = x, y, z, t, s1 = (+,-,+,-), s3 = (-,-,+,+).
// So every lane does a quarter of a site's arithmetic with a quarter of its
// accumulators.
//
// Packing to the tiled layout, the tiled stencil and unpacking moved three
// times the bytes in three launches; per call, that / this, in us: 4^4 x 1 (FP64)
// 15.5 / 8.5, 16^4 x 4 93.1 / 60.5, 16^3x32 x 12 474 / 351.  Bound: at the
// small end the launch and the call; from 16^4 on the vector memory path,
// which moves each site's eight neighbours and eight links through L2 and L1
// (2.3 KB per site and source, 0.4 KB of it from memory).  Two sources per
// lane sharing the links took 250 registers and were slower (362 us).
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "hop.h"
#include "kernels.h"

#include <type_traits>

namespace ovl {

// lane l of every quad reads lane P_l of its quad
template <int P0, int P1, int P2, int P3>
__device__ __forceinline__ double quad_perm(double v) {
    constexpr int ctrl = P0 | (P1 << 2) | (P2 << 4) | (P3 << 6);
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// the partner of direction mu: spins (0,3), (1,2) for x and y, (0,2), (1,3) for z and t
template <int MU, typename R>
__device__ __forceinline__ cx<R> partner(cx<R> v) {
    if constexpr (MU < 2) return mk<R>(quad_perm<3, 2, 1, 0>(v.re), quad_perm<3, 2, 1, 0>(v.im));
    else return mk<R>(quad_perm<2, 3, 0, 1>(v.re), quad_perm<2, 3, 0, 1>(v.im));
}
// a + sgn phi b
template <int MU, typename R>
__device__ __forceinline__ cx<R> add_phase(cx<R> a, R sgn, cx<R> b, R s1, R s3) {
    const R f = sgn * (MU == 0 ? R(1) : MU == 3 ? s3 : s1);
    if constexpr (MU == 0 || MU == 2) return mk<R>(a.re - f * b.im, a.im + f * b.re);
    else return mk<R>(a.re + f * b.re, a.im + f * b.im);
}

// WIDE: 64-bit byte offsets, for lattices on which 32 bits do not reach every
// site (offsets32).
template <int LNK, bool WIDE>
__global__ __launch_bounds__(kBlock, 2) void k_hw_quad(const double2* __restrict__ in,
                                                       double2* __restrict__ out,
                                                       const double2* __restrict__ U, Geom g,
                                                       double kappa, int nrhs, int order) {
    typedef double R;
    constexpr uint32_t NE = LNK ? 6 : 9;  // stored elements per link
    const unsigned tile = uniform(xcd_remap(blockIdx.x, gridDim.x));
    const unsigned ntile = gridDim.x / (unsigned)nrhs;
    const int n = (int)uniform(order ? tile / ntile : tile % (unsigned)nrhs);
    const int tb = (int)uniform(order ? tile % ntile : tile / (unsigned)nrhs);
    const uint32_t V = (uint32_t)g.V, Vt = (uint32_t)g.Vt;
    const uint32_t st = (uint32_t)tb * (kBlock / 4) + (threadIdx.x >> 2);
    const bool valid = st < V;
    const uint32_t s = valid ? st : V - 1;  // lanes past the lattice load a real site
    const uint32_t a = threadIdx.x & 3u;
    const bool up = a < 2;
    const R s1 = (a & 1) ? R(-1) : R(1), s3 = up ? R(-1) : R(1);
    const R ci = up ? R(1) : R(-1);
    uint32_t rem = s;
    int coord[4];
    coord[0] = (int)(rem % (uint32_t)g.L[0]); rem /= (uint32_t)g.L[0];
    coord[1] = (int)(rem % (uint32_t)g.L[1]); rem /= (uint32_t)g.L[1];
    coord[2] = (int)(rem % (uint32_t)g.L[2]);
    coord[3] = (int)(rem / (uint32_t)g.L[2]);
    typedef typename std::conditional<WIDE, int64_t, uint32_t>::type Off;
    const double2* src = in + (size_t)n * 12 * V;
    auto spin = [&](uint32_t site, cx<R> (&v)[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = ld<R>(src, (Off)site * 12u + 3u * a + (uint32_t)c);
    };
    auto link = [](uint32_t e, uint32_t site) -> Off {
        if constexpr (WIDE) return tix64(e, site, NE);
        else return tix(e, site, NE);
    };
    cx<R> acc[3] = {mk<R>(0, 0), mk<R>(0, 0), mk<R>(0, 0)};
    auto direction = [&](auto muc) {
        constexpr int MU = decltype(muc)::value;
        const uint32_t fw = nbr(g, s, coord, MU, true), bw = nbr(g, s, coord, MU, false);
        // the site of the lane's own hop, the one its partner needs, and the link's
        const uint32_t nv = up ? fw : bw, nw = up ? bw : fw, ls = up ? s : bw;
        const double2* Um = U + (size_t)MU * NE * Vt;
        cx<R> m[3][3], v[3], w[3];
#pragma unroll
        for (uint32_t e = 0; e < NE; ++e) m[e / 3][e % 3] = ld<R>(Um, link(e, ls));
        spin(nw, w);
        spin(nv, v);
        if constexpr (LNK == 1) {
            // row 2 = lsgn * conj(row0 x row1), lsgn the boundary sign in the stored rows
            const int edge = up ? g.L[MU] - 1 : 0;
            const R lsgn = (coord[MU] == edge && g.bc[MU] < 0) ? R(-1) : R(1);
            const cx<R> c0 = m[0][1] * m[1][2] - m[0][2] * m[1][1];
            const cx<R> c1 = m[0][2] * m[1][0] - m[0][0] * m[1][2];
            const cx<R> c2 = m[0][0] * m[1][1] - m[0][1] * m[1][0];
            m[2][0] = mk<R>(lsgn * c0.re, -lsgn * c0.im);
            m[2][1] = mk<R>(lsgn * c1.re, -lsgn * c1.im);
            m[2][2] = mk<R>(lsgn * c2.re, -lsgn * c2.im);
        }
        // backward lanes take the transpose (and conjugate h and u instead of it)
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int d = c + 1; d < 3; ++d) {
                const cx<R> x = m[c][d], y = m[d][c];
                m[c][d] = up ? x : y;
                m[d][c] = up ? y : x;
            }
        cx<R> h[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            h[c] = add_phase<MU, R>(v[c], R(1), partner<MU, R>(w[c]), s1, s3);
            h[c].im *= ci;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            cx<R> u = mk<R>(0, 0);
#pragma unroll
            for (int d = 0; d < 3; ++d) fma_(u, m[c][d], h[d]);
            u.im *= ci;
            acc[c] = add_phase<MU, R>(acc[c] + u, R(-1), partner<MU, R>(u), s1, s3);
        }
    };
    using std::integral_constant;
    direction(integral_constant<int, 2>{});
    direction(integral_constant<int, 0>{});
    direction(integral_constant<int, 1>{});
    direction(integral_constant<int, 3>{});
    if (!valid) return;
    double2* o = out + (size_t)n * 12 * V;
    cx<R> p[3];
    spin(s, p);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        // D psi = psi - kappa acc ; H = gamma5 D
        cx<R> hv = p[c] - kappa * acc[c];
        if (!up) hv = -hv;
        stc<R>(o, (Off)s * 12u + 3u * a + (uint32_t)c, hv);
    }
}

void launch_hw(const double2* in, double2* out, const double2* U, const Geom& g, double kappa,
               int nrhs, int lnk, hipStream_t s) {
    // Block order.  A tile's sources back to back share its links in L2; once
    // input and output outgrow the 256 MB last-level cache, tiles back to back
    // (which share neighbours) win.  Input vectors, sources / tiles back to back,
    // in us, launches in a row: 16^4 x 4 (48 MiB) 53.0 / 55.0, x 12 (144) 149.8 /
    // 161.4, x 15 (180) 204.1 / 211.7, x 16 (192) 229.9 / 224.8, 16^3x32 x 8 (192)
    // 230.1 / 239.7, x 9 (216) 269.7 / 257.1, 16^4 x 20 (240) 314.3 / 288.4,
    // 16^3x32 x 12 (288) 380.5 / 340.6.
    const int order = (size_t)g.V * nrhs * 12 * sizeof(double2) > ((size_t)192 << 20);
    const unsigned ntile = (unsigned)((g.V + kBlock / 4 - 1) / (kBlock / 4));
    const dim3 grid(ntile * (unsigned)nrhs);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(kBlock), 0, s, in, out, U, g, kappa, nrhs, order);
    };
    if (offsets32(g.Vt, sizeof(double2))) {
        if (lnk) go(k_hw_quad<1, false>);
        else go(k_hw_quad<0, false>);
    } else {
        if (lnk) go(k_hw_quad<1, true>);
        else go(k_hw_quad<0, true>);
    }
}

}  // namespace ovl
