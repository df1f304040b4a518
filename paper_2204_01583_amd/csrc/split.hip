// The seed iteration for small problems (HIP, gfx950): one kernel per
// iteration, one hop per lane.
//
// Where a whole iteration is a few hundred waves, its time is the chain of
// dependent loads, not bandwidth: at 8^4 with one source the stencil with one
// lane per site ran 16 blocks, each through nine dependent rounds of loads
// (13.2 us per launch), and the update kernel another chain (5.9 us).  Here a
// block takes one 64-site layout tile with eight waves, wave (mu, direction)
// taking that hop of the 64 sites, so a tile's loads are all in flight at
// once and the hop needs no branch on mu within a wave; the half-spinors meet
// in LDS, and six waves finish two components of every site each.  The
// kernel also forms r_k = r_{k-1} - alpha q_{k-1} as it loads (see the fused
// iteration in stencil.hip, whose order of work it shares), so an iteration
// is one launch: 9.8 us at 8^4, 14.2 us at 12x10x6x14 with two sources (FP64;
// the two kernels 19.1 and 21.1 us).  Bound: the launch and its chain of loads
// (counter and job, slot base, residuals and partials, second batch) up to
// one round of blocks, then the neighbours' doubled bytes.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "hop.h"
#include "kernels.h"
#include "seed_iter.h"

namespace ovl {

constexpr int kSplitThreads = 8 * kTile;  // one wave per hop of a tile

// loads that are the same for the whole wave, through the scalar cache.  The
// kernel that reads a value does not write it, with one exception: a source's
// status, which its first slice block sets in the launch that finds the error.
// Either value will do there: every block finds the same error in the same
// partials, and a block that already sees it set does what it would do then.
template <typename T>
__device__ __forceinline__ T sload(const T* p) {
    typedef const __attribute__((address_space(4))) T C;
    return *(C*)p;
}

// Block `tile` of job J: the blocks of one source are nslices slice blocks,
// then one block per layout tile.
template <typename R, int LNK>
__device__ __forceinline__ void iter_split_block(const JobDesc& J, int k, unsigned tile) {
    constexpr int f = sizeof(R) == 4 ? 1 : 0;
    constexpr int NT = kSplitThreads;
    constexpr uint32_t NE = LNK ? 6 : 9;  // stored elements per link
    const ShiftDev& sh = J.sh;
    const int ntile = J.nsb, per = ntile + sh.nslices;
    const int n = (int)uniform(tile / (unsigned)per), b = (int)uniform(tile % (unsigned)per);
    SrcState& S = J.st[n];
    const int lane = (int)(threadIdx.x & 63), w = (int)uniform(threadIdx.x >> 6);
    __shared__ double shm[4 * NT / 64];

    // the state of the source and the previous kernel's partials, requested
    // before anything waits
    const int status = sload(&S.status);
    const int* cp = sh.cnt + ((size_t)((k - 1) & 1) * sh.nsrc + n) * kMaxSlices;
    int active = 0;
#pragma unroll
    for (int q = 0; q < kMaxSlices; ++q) {
        const int c = sload(cp + q);
        active += q < sh.nslices ? c : 0;
    }
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (k > 0) {
        const double4* pw = J.part_w + (size_t)((k - 1) & 1) * J.part_stride + (size_t)n * ntile;
        for (int q = lane; q < ntile; q += 64) {
            const double4 v = pw[q];
            a[0] += v.x;
            a[1] += v.y;
            a[2] += v.z;
            a[3] += v.w;
        }
    }
    const bool live = status == 0 && k <= sh.maxk && active > 0;

    // every wave sums the partials itself (a fixed order: strided per lane,
    // then the butterfly), so the scalars need no barrier
    auto scalars = [&]() {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] += __shfl_xor(a[i], o, 64);
        return seed_scalars_of(a);
    };

    if (b < sh.nslices) {
        // slice block: the shift scalars of iteration k-1
        int* cnt_next = sh.cnt + ((size_t)(k & 1) * sh.nsrc + n) * kMaxSlices + b;
        if (!live) {
            // a finished source stays finished (its counts go to zero); past the
            // iteration limit the counts are kept for the host
            if (k <= sh.maxk && threadIdx.x == 0) *cnt_next = 0;
            return;
        }
        if (k == 0) {
            // sweep forms: the first sweep's window starts one iteration before
            // the first, which leaves every p_j as it is
            const int j = b * kBlock + (int)threadIdx.x;
            if (J.swc != nullptr && threadIdx.x < kBlock && j < sh.J) {
                const size_t o = (size_t)n * sh.J + j;
                double2* c = J.swc + o * (size_t)(J.rmask + 1) * 3;
                c[0] = c[1] = make_double2(0, 0);
                c[2] = make_double2(1, 0);
                J.swn[o] = 1;
            }
            return;
        }
        const SeedScalars sc = scalars();
        if (sc.status) {
            if (threadIdx.x == 0) {
                if (b == 0) S.status = sc.status;
                *cnt_next = 0;
            }
            return;
        }
        if (b == 0 && threadIdx.x == 0) {
            S.alpha[(k - 1) & 1] = sc.alpha;
            S.beta[(k - 1) & 1] = sc.beta;
            S.rr[(k - 1) & 1] = sc.rr;
            S.iter = k;
            if (sh.seed != nullptr) {
                double2* sd = sh.seed + ((size_t)n * (sh.maxk + 1) + (k - 1)) * 3;
                sd[0] = sc.alpha;
                sd[1] = sc.beta;
                sd[2] = make_double2(sc.rr, sc.rrn);
            }
        }
        advance_shift_slice<NT>(J, S, n, b, k - 1, sc, shm);
        return;
    }
    if (!live) return;

    const uint32_t V = (uint32_t)J.g.V, Vt = (uint32_t)J.g.Vt;
    const int tb = b - sh.nslices;
    const uint32_t st = (uint32_t)tb * kTile + (uint32_t)lane;
    const bool valid = st < V;
    const uint32_t s = valid ? st : V - 1;  // padding lanes load a real site
    uint32_t rem = s;
    int coord[4];
    coord[0] = (int)(rem % (uint32_t)J.g.L[0]); rem /= (uint32_t)J.g.L[0];
    coord[1] = (int)(rem % (uint32_t)J.g.L[1]); rem /= (uint32_t)J.g.L[1];
    coord[2] = (int)(rem % (uint32_t)J.g.L[2]);
    coord[3] = (int)(rem / (uint32_t)J.g.L[2]);
    const int mu = w >> 1;
    const bool fwd = (w & 1) == 0;
    const uint32_t nb = nbr(J.g, s, coord, mu, fwd);
    const uint32_t lsite = fwd ? s : nb;
    const size_t n12 = (size_t)12 * Vt;
    auto vec_base = [&](int kk) -> C2<R>* {
        if (J.form == OVL_FORM_BASIS)
            return reinterpret_cast<C2<R>*>(sload(J.slots + kk / kSlotChunk) +
                                            (size_t)(kk % kSlotChunk) * J.slot_bytes) + (size_t)n * n12;
        return static_cast<C2<R>*>(J.r[f]) + (size_t)(kk & J.rmask) * J.rpp + (size_t)n * n12;
    };
    const C2<R>* rin = vec_base(k > 0 ? k - 1 : 0);
    C2<R>* rout = vec_base(k);
    C2<R>* qbase = static_cast<C2<R>*>(J.q[f]) + (size_t)n * n12;
    const C2<R>* qin = qbase + (size_t)((k - 1) & 1) * J.qpp;
    C2<R>* qout = qbase + (size_t)(k & 1) * J.qpp;
    const C2<R>* Um = static_cast<const C2<R>*>(J.U[f]) + (size_t)mu * NE * Vt;

    // This hop's operands and, for the finishing waves, the site's own two
    // components: colour w % 3 of the upper (w < 3) or lower spins.  FP64
    // takes them in two batches, the third colour's q, the links and the own
    // components after two colours are projected, which keeps the kernel at 128
    // registers, so that two blocks share a CU and a launch of up to 512 tiles
    // runs in one round (316 tiles: 14.2 us a launch; 19.4 with 182 registers
    // in one batch, where 64 tiles took 9.4 against 9.8).
    constexpr int kB = sizeof(R) == 8 ? 2 : 3;  // colours of q in the first batch
    cx<R> pv[4][3], qv[4][3], m[3][3], ro[2], qo[2], h[2][3];
    const int half = w / 3, col = w % 3;
    const uint32_t o0 = tix((uint32_t)(6 * (half & 1) + col), s, 12), o1 = o0 + 3 * kTile;
    auto own = [&]() {
        ro[0] = ld<R>(rin, o0);
        ro[1] = ld<R>(rin, o1);
        qo[0] = qo[1] = mk<R>(0, 0);
        if (k > 0) {
            qo[0] = ld<R>(qin, o0);
            qo[1] = ld<R>(qin, o1);
        }
    };
    auto rest = [&]() {
        if (k > 0)
#pragma unroll
            for (int c = kB; c < 3; ++c)
#pragma unroll
                for (int p = 0; p < 4; ++p) qv[p][c] = ld<R>(qin, tix((uint32_t)(3 * p + c), nb, 12));
#pragma unroll
        for (int e = 0; e < (LNK ? 6 : 9); ++e)
            m[e / 3][e % 3] = ld<R>(Um, tix((uint32_t)e, lsite, NE));
    };
#pragma unroll
    for (int c = 0; c < 12; ++c) pv[c / 3][c % 3] = ld<R>(rin, tix((uint32_t)c, nb, 12));
    if (k > 0)
#pragma unroll
        for (int c = 0; c < kB; ++c)
#pragma unroll
            for (int p = 0; p < 4; ++p) qv[p][c] = ld<R>(qin, tix((uint32_t)(3 * p + c), nb, 12));
    if constexpr (kB == 3) {
        rest();
        own();
    }
    SeedScalars sc{};
    sc.alpha = make_double2(0, 0);
    sc.beta = make_double2(0, 0);
    if (k > 0) {
        sc = scalars();
        if (sc.status) return;  // the slice block records it
    }
    const R ar = (R)sc.alpha.x, ai = (R)sc.alpha.y;
    auto sub = [&](cx<R>& r, const cx<R>& q) {
        r = mk<R>(r.re - (ar * q.re - ai * q.im), r.im - (ar * q.im + ai * q.re));
    };
    const R sg = fwd ? R(-1) : R(1);
    auto projected = [&](int c) {
        if (k > 0)
#pragma unroll
            for (int p = 0; p < 4; ++p) sub(pv[p][c], qv[p][c]);
        project<R>(mu, sg, pv[0][c], pv[1][c], pv[2][c], pv[3][c], h[0][c], h[1][c]);
    };
#pragma unroll
    for (int c = 0; c < kB; ++c) projected(c);
    if constexpr (kB < 3) {
        __builtin_amdgcn_sched_barrier(0);
        rest();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = kB; c < 3; ++c) projected(c);
        __builtin_amdgcn_sched_barrier(0);
        own();  // in flight during the product and the exchange
    }

    // the hop: half-spinor u = U h (forward) or U^dag h (backward)
    if constexpr (LNK == 1) {
        const int edge = fwd ? J.g.L[mu] - 1 : 0;
        const R ls = (coord[mu] == edge && J.g.bc[mu] < 0) ? R(-1) : R(1);
        const cx<R> c0 = m[0][1] * m[1][2] - m[0][2] * m[1][1];
        const cx<R> c1 = m[0][2] * m[1][0] - m[0][0] * m[1][2];
        const cx<R> c2 = m[0][0] * m[1][1] - m[0][1] * m[1][0];
        m[2][0] = mk<R>(ls * c0.re, -ls * c0.im);
        m[2][1] = mk<R>(ls * c1.re, -ls * c1.im);
        m[2][2] = mk<R>(ls * c2.re, -ls * c2.im);
    }
    __shared__ C2<R> lu[8][6][kTile];  // [hop][3 spin + colour][site]
    const R ci = fwd ? R(1) : R(-1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        cx<R> u0 = mk<R>(0, 0), u1 = mk<R>(0, 0);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            cx<R> l = fwd ? m[c][d] : m[d][c];
            l.im *= ci;
            fma_(u0, l, h[0][d]);
            fma_(u1, l, h[1][d]);
        }
        C2<R> v;
        v.x = u0.re; v.y = u0.im;
        lu[w][c][lane] = v;
        v.x = u1.re; v.y = u1.im;
        lu[w][3 + c][lane] = v;
    }
    __syncthreads();
    if (k > 0) {
        sub(ro[0], qo[0]);
        sub(ro[1], qo[1]);
    }

    double t[4] = {0.0, 0.0, 0.0, 0.0};
    if (w < 6 && valid) {
        // acc += u (upper spins) or the lower half sg A^dag u of every hop
        cx<R> a0 = mk<R>(0, 0), a1 = mk<R>(0, 0);
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            const C2<R> x0 = lu[d][col][lane], x1 = lu[d][3 + col][lane];
            const cx<R> u0 = mk<R>(x0.x, x0.y), u1 = mk<R>(x1.x, x1.y);
            if (half == 0) {
                a0 = a0 + u0;
                a1 = a1 + u1;
            } else {
                const R sd = (d & 1) ? R(1) : R(-1);
                cx<R> b0, b1;  // A^dag (u0, u1)
                switch (d >> 1) {
                    case 0: b0 = ti(u1); b1 = ti(u0); break;
                    case 1: b0 = u1; b1 = -u0; break;
                    case 2: b0 = ti(u0); b1 = tmi(u1); break;
                    default: b0 = u0; b1 = u1; break;
                }
                a0 = a0 + sd * b0;
                a1 = a1 + sd * b1;
            }
        }
        const R kap = (R)J.kappa, zr = (R)J.zs.x, zi = (R)J.zs.y;
        const R br = (R)sc.beta.x, bi = (R)sc.beta.y;
        const bool acc2 = J.h != nullptr && k > 0;
        const double2 hk = acc2 ? J.h[(size_t)n * (sh.maxk + 1) + k] : make_double2(0, 0);
        double2* sacc = J.s64 + (size_t)n * n12;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const cx<R> r = ro[i], av = i ? a1 : a0;
            const uint32_t o = i ? o1 : o0;
            if (k > 0) stc<R>(rout, o, r);
            // H r = gamma5 (r - kappa acc); q_k = z_s r - H r + beta q_{k-1}
            cx<R> hv = r - kap * av;
            if (half) hv = -hv;
            cx<R> q = mk<R>(zr * r.re - zi * r.im - hv.re, zr * r.im + zi * r.re - hv.im);
            q.re += br * qo[i].re - bi * qo[i].im;
            q.im += br * qo[i].im + bi * qo[i].re;
            stc<R>(qout, o, q);
            t[0] += (double)r.re * (double)q.re + (double)r.im * (double)q.im;
            t[1] += (double)r.re * (double)q.im - (double)r.im * (double)q.re;
            t[2] += (double)q.re * (double)q.re + (double)q.im * (double)q.im;
            t[3] += (double)r.re * (double)r.re + (double)r.im * (double)r.im;
            if (acc2) {
                double2 sv = sacc[o];
                sv.x += hk.x * (double)r.re - hk.y * (double)r.im;
                sv.y += hk.x * (double)r.im + hk.y * (double)r.re;
                sacc[o] = sv;
            }
        }
    } else if (w < 6) {
        // padding sites of the last layout tile stay zero in every output
        const uint32_t p0 = tix((uint32_t)(6 * half + col), st, 12), p1 = p0 + 3 * kTile;
        stc<R>(qout, p0, mk<R>(0, 0));
        stc<R>(qout, p1, mk<R>(0, 0));
        if (k > 0) {
            stc<R>(rout, p0, mk<R>(0, 0));
            stc<R>(rout, p1, mk<R>(0, 0));
        }
    }
    block_sum4<NT>(t, shm);
    if (threadIdx.x == 0)
        J.part_w[(size_t)(k & 1) * J.part_stride + (size_t)n * ntile + tb] =
            make_double4(t[0], t[1], t[2], t[3]);
}

template <typename R, int LNK>
__global__ __launch_bounds__(kSplitThreads, 4) void k_iter_split(const JobDesc* __restrict__ jobs,
                                                              int njobs,
                                                              const int* __restrict__ kread,
                                                              int* __restrict__ kwrite) {
    const int k = sload(kread);
    if (blockIdx.x == 0 && threadIdx.x == 0) *kwrite = k + 1;
    const int f = sizeof(R) == 4 ? 1 : 0;
    int j;
    unsigned tile;
    if (!job_tile(jobs, njobs, f, j, tile)) return;
    iter_split_block<R, LNK>(jobs[j], k, tile);
}

int split_tiles(const Geom& g) { return (int)(g.Vt / kTile); }
int split_grid_blocks(const Geom& g, int nrhs, int nslices) {
    return (split_tiles(g) + nslices) * nrhs;
}

template <typename R>
void launch_iter_split(const JobDesc* jobs, int njobs, const int* kread, int* kwrite,
                       int total_blocks, int lnk, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    auto go = [&](auto kern) {
        if (ev0)
            hipExtLaunchKernelGGL(kern, dim3(total_blocks), dim3(kSplitThreads), 0, s, ev0, ev1, 0,
                                  jobs, njobs, kread, kwrite);
        else
            hipLaunchKernelGGL(kern, dim3(total_blocks), dim3(kSplitThreads), 0, s, jobs, njobs,
                               kread, kwrite);
    };
    if (lnk) go(k_iter_split<R, 1>);
    else go(k_iter_split<R, 0>);
}
template void launch_iter_split<double>(const JobDesc*, int, const int*, int*, int, int,
                                        hipStream_t, hipEvent_t, hipEvent_t);
template void launch_iter_split<float>(const JobDesc*, int, const int*, int*, int, int, hipStream_t,
                                       hipEvent_t, hipEvent_t);

}  // namespace ovl
