// adjoint.hip -- discrete adjoint of one TRT pull step (lbm_step_adjoint).
//
// Forward step f^{t+1} = Phi(P f^t; ns): P is the pull gather through the
// adjacency (a permutation of PDF slots), Phi the per-cell collision with
// partial bounce-back.  Its transpose is applied per cell:
//   mu = lambda^{t+1}[.][m]                        (coalesced rows)
//   nu = (dPhi/dg)^T mu                            (local 19x19, in closed form)
//   lambda^t[A_k(m)] = nu_k                        (scatter through the same
//                                                   adjacency; A_0 = own slot)
// Every slot of lambda^t is written by exactly one (cell, direction) because
// P is a permutation, so the scatter needs no atomics.  The closed form:
//   with j the pre-collision momentum, m0 = sum w mu, m1 = sum w mu c,
//   m2 = sum w mu (c.j) c, mu+- = (mu_k +- mu_opp)/2:
//   nu_k = (1-ns)[mu_k - s+ mu+_k - s- mu-_k + s+ (m0 + 9 c_k.m2 - 3 m0 c_k.j)
//                 + 3 s- c_k.m1] + ns mu_opp(k)
//   grad[m] += sum_i mu_i (g_opp(i) - f*_i)
// which follows from d e+_i/d g_k = w_i [1 + 9 (c_i.j)(c_i.c_k) - 3 j.c_k] and
// d e-_i/d g_k = 3 w_i c_i.c_k.
#include "lbm_device.hpp"
#include "lbm_host.hpp"

namespace lbm {

constexpr int kAdjBlock = 256;
// Bytes per cell (sweep_launch): lambda^{t+1}, lambda^t, and f_t twice, since
// every step of the reverse sweep reads another state.
constexpr size_t kAdjCellBytes = 4 * Q * sizeof(double);

// Beyond 384 MiB steps with plain stores alternate their direction (8-bit codes,
// 0.96 / 1.5 / 2.0 / 3.3 / 7.8 M cells 87.6 / 157.8 / 194.9 / 332.9 / 771 -> 84.4 /
// 147.9 / 182.1 / 323.7 / 766 us).  A step is one of a reverse sweep over the same
// arrays: where those stay in the cache it takes no hints, like a call of several
// sweeps.
inline SweepLaunch adjoint_launch(int32_t flags, int64_t n) {
    constexpr SweepRule rule = {size_t(384) << 20, false, false, false};
    return sweep_launch(flags, n, kAdjCellBytes, rule, kResidentSweeps);
}

// Waves per SIMD that the kernels are built for.  A cell holds 38 gathered and
// read values in FP64, and the compiler takes 188 registers (two waves) unless
// told to fit three (168, nothing spilled; four would spill 46).  Three waves
// keep more loads in flight, two leave more of the caches to each: 8-bit codes, us
// with three / two waves, plain stores 0.20 / 0.96 / 1.5 / 2.0 / 2.1 M cells 19.6 /
// 21.9, 84.4 / 89.4, 147.9 / 150.7, 182.1 / 185.4, 205.0 / 205.0, then within 1 %
// of each other to 4 M and 768 / 763 at 7.8 M; nontemporal stores 0.96 / 1.5 / 1.76 /
// 1.94 / 2.1 / 4.9 M 101.1 / 102.7, 171.0 / 172.7, 185.2 / 181.0, 200.5 / 195.7,
// 233.2 / 226.3, 533 / 518.
constexpr size_t kAdjThreeWaves = size_t(1280) << 20, kAdjThreeWavesNT = size_t(960) << 20;

template <class F>
lbm_status with_policy_waves(int policy, int64_t n, F&& f) {
    return with_policy(policy, [&](auto pol) {
        constexpr size_t three = pol == kStreamNT ? kAdjThreeWavesNT : kAdjThreeWaves;
        return size_t(n) * kAdjCellBytes <= three ? f(pol, std::integral_constant<int, 3>{})
                                                  : f(pol, std::integral_constant<int, 2>{});
    });
}
static_assert(kAdjBlock == kCodeTile, "a workgroup of k_adjoint_coded is one code tile");

// The adjoint of one cell m whose 19 slots A (A[0] = m, A[k+1] = the slot it
// pulls direction k + 1 from) are known.
template <bool PBB, int POL>
__device__ __forceinline__ void adjoint_cell(const double* __restrict__ f_t, const uint32_t* A,
                                             const double* __restrict__ ns,
                                             const double* __restrict__ lam_next,
                                             double* __restrict__ lam_t,
                                             double* __restrict__ grad, int64_t m,
                                             int64_t stride, const TrtConst& c) {
    double g[Q], mu[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) g[k] = f_t[A[k]];
#pragma unroll
    for (int k = 0; k < Q; ++k) mu[k] = ld_stream<POL>(lam_next + k * stride + m);  // own column, read once
    const CellMoments<double> cm = cell_moments(g);
    const double s = PBB ? ns[m] : 0.0;
    if constexpr (PBB) {
        // sum of mu_i (g_opp(i) - f*_i), one pair of f* at a time
        const TrtCell<double> t(cm, c);
        double acc = mu[0] * (g[0] - t.rest(g[0]));
#pragma unroll
        for (int k = 0; k < NPAIR; ++k) {
            const int a = 2 * k + 1, b = 2 * k + 2;
            double fa, fb;
            t.pair(k, g[a], g[b], c, fa, fb);
            acc += mu[a] * (g[b] - fa) + mu[b] * (g[a] - fb);
        }
        if (grad) grad[m] += acc;
    }
    // moments of w mu
    double m0 = W0 * mu[0], m1x = 0, m1y = 0, m1z = 0, m2x = 0, m2y = 0, m2z = 0;
#pragma unroll
    for (int k = 0; k < NPAIR; ++k) {
        const int a = 2 * k + 1, b = 2 * k + 2;
        const double w = pair_weight(k);
        const double cj = PCX[k] * cm.jx + PCY[k] * cm.jy + PCZ[k] * cm.jz;
        const double sum = w * (mu[a] + mu[b]), dif = w * (mu[a] - mu[b]);
        m0 += sum;
        m1x += PCX[k] * dif;
        m1y += PCY[k] * dif;
        m1z += PCZ[k] * dif;
        m2x += PCX[k] * cj * sum;
        m2y += PCY[k] * cj * sum;
        m2z += PCZ[k] * cj * sum;
    }
    const double sp = c.sp, sm = c.sm;
    const double P = sp * m0;
    double nu0 = mu[0] - sp * mu[0] + P;
    if constexpr (PBB) nu0 = (1.0 - s) * nu0 + s * mu[0];
    st<double, double, POL == kStreamNT>(lam_t + A[0], nu0);
#pragma unroll
    for (int k = 0; k < NPAIR; ++k) {
        const int a = 2 * k + 1, b = 2 * k + 2;
        const double cj = PCX[k] * cm.jx + PCY[k] * cm.jy + PCZ[k] * cm.jz;
        const double cm1 = PCX[k] * m1x + PCY[k] * m1y + PCZ[k] * m1z;
        const double cm2 = PCX[k] * m2x + PCY[k] * m2y + PCZ[k] * m2z;
        const double Qd = sp * (9.0 * cm2 - 3.0 * m0 * cj) + 3.0 * sm * cm1;
        const double mup = 0.5 * (mu[a] + mu[b]), mum = 0.5 * (mu[a] - mu[b]);
        double na = mu[a] - sp * mup - sm * mum + P + Qd;
        double nb = mu[b] - sp * mup + sm * mum + P - Qd;
        if constexpr (PBB) {
            na = (1.0 - s) * na + s * mu[b];
            nb = (1.0 - s) * nb + s * mu[a];
        }
        st<double, double, POL == kStreamNT>(lam_t + A[a], na);
        st<double, double, POL == kStreamNT>(lam_t + A[b], nb);
    }
}

template <bool PBB, int POL, int WAVES>
__global__ __launch_bounds__(kAdjBlock, WAVES) void k_adjoint(const double* __restrict__ f_t,
                                                       const uint32_t* __restrict__ adj,
                                                       const double* __restrict__ ns,
                                                       const double* __restrict__ lam_next,
                                                       double* __restrict__ lam_t,
                                                       double* __restrict__ grad, int64_t n,
                                                       int64_t stride, TrtConst c,
                                                       XcdMap map) {
    const int64_t m = logical_block(map) * kAdjBlock + threadIdx.x;
    if (m >= n) return;
    uint32_t A[Q];
    A[0] = uint32_t(m);
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) A[k + 1] = ld_stream<POL>(adj + k * stride + m);
    adjoint_cell<PBB, POL>(f_t, A, ns, lam_next, lam_t, grad, m, stride, c);
}

// Same, with the slots rebuilt from the adjacency codes of
// lbm_compress_adjacency (a workgroup is one 256-cell code tile): with C8 the
// 8-bit codes of a narrow tile (lbm_narrow_codes), otherwise the 16-bit codes;
// a tile with escapes reads adj.  The branch is uniform over the workgroup and
// every form rebuilds the same slots, so the result does not depend on it.
template <bool PBB, int POL, bool C8, int WAVES>
__global__ __launch_bounds__(kAdjBlock, WAVES) void k_adjoint_coded(const double* __restrict__ f_t,
                                                             const int8_t* __restrict__ codes8,
                                                             const int16_t* __restrict__ codes,
                                                             const int32_t* __restrict__ tile_rec,
                                                             const uint32_t* __restrict__ adj,
                                                             const double* __restrict__ ns,
                                                             const double* __restrict__ lam_next,
                                                             double* __restrict__ lam_t,
                                                             double* __restrict__ grad, int64_t n,
                                                             int64_t stride, TrtConst c,
                                                             XcdMap map) {
    const int64_t tile = logical_block(map);
    const int64_t m = tile * kAdjBlock + threadIdx.x;
    if (m >= n) return;
    const int32_t* rec = tile_rec + tile * kCodeRec;  // uniform over the workgroup
    uint32_t A[Q];
    A[0] = uint32_t(m);
    const uint32_t S = uint32_t(stride), mm = uint32_t(m);
    if (C8 && rec[Q] != 0) {
        int32_t cd[Q - 1];
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) cd[k] = ld_stream<POL>(codes8 + k * stride + m);
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) {
            const uint32_t i = k + 1;
            A[i] = cd[k] == int32_t(kCode8Bounce) ? uint32_t(opp(int(i))) * S + mm
                                                  : i * S + uint32_t(rec[k]) + mm + uint32_t(cd[k]);
        }
    } else if (rec[Q - 1] != 0) {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) A[k + 1] = ld_stream<POL>(adj + k * stride + m);
    } else {
        int32_t cd[Q - 1];
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) cd[k] = ld_stream<POL>(codes + k * stride + m);
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) {
            const uint32_t i = k + 1;
            A[i] = cd[k] == kCodeBounce ? uint32_t(opp(int(i))) * S + mm
                                        : i * S + uint32_t(rec[k]) + mm + uint32_t(cd[k]);
        }
    }
    adjoint_cell<PBB, POL>(f_t, A, ns, lam_next, lam_t, grad, m, stride, c);
}

// Seed lambda^T = dJ/df^T for J = (1/n) sum_m (j_x(m) + G_x/2): the slot a cell
// pulls for direction i carries c_ix / n; every other slot is 0.
__global__ __launch_bounds__(kAdjBlock) void k_adjoint_seed(const uint32_t* __restrict__ adj,
                                                            double* __restrict__ lam_t, int64_t n,
                                                            int64_t stride, double inv_n) {
    const int64_t m = int64_t(blockIdx.x) * kAdjBlock + threadIdx.x;
    if (m >= n) return;
    lam_t[m] = 0.0;
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) lam_t[adj[k * stride + m]] = double(vel_x(k + 1)) * inv_n;
}

}  // namespace lbm

using namespace lbm;

extern "C" lbm_status lbm_step_adjoint(const lbm_params* p, int64_t n, int64_t stride,
                                       const uint32_t* adj, const void* f_t, const double* ns,
                                       const double* lam_next, double* lam_t, double* grad_ns,
                                       void* stream) {
    if (!valid_params(p) || !adj || !lam_t || n <= 0) return LBM_EINVAL;
    if (p->storage != LBM_F64 && p->storage != LBM_F64_SHIFTED) return LBM_EINVAL;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    hipStream_t s = as_stream(stream);
    const unsigned grid = unsigned((n + kAdjBlock - 1) / kAdjBlock);
    if (!lam_next) {
        k_adjoint_seed<<<grid, kAdjBlock, 0, s>>>(adj, lam_t, n, stride, 1.0 / double(n));
        return after_launch();
    }
    if (!f_t) return LBM_EINVAL;
    const TrtConst c = make_trt_const(*p);
    const double* f = static_cast<const double*>(f_t);
    // the sweep's launch options: workgroup-to-XCD mapping, memory policy
    const SweepLaunch l = adjoint_launch(p->flags, n);
    const XcdMap map = l.towards(lam_t < lam_next);
    return with_policy_waves(l.policy, n, [&](auto pol, auto waves) {
        if (ns) k_adjoint<true, pol, waves><<<l.grid, l.block, 0, s>>>(f, adj, ns, lam_next, lam_t, grad_ns, n, stride, c, map);
        else k_adjoint<false, pol, waves><<<l.grid, l.block, 0, s>>>(f, adj, ns, lam_next, lam_t, nullptr, n, stride, c, map);
        return after_launch();
    });
}

namespace lbm {

template <bool C8>
lbm_status step_adjoint_coded(const lbm_params* p, int64_t n, int64_t stride,
                              const int8_t* codes8, const int16_t* codes,
                              const int32_t* tile_records, const uint32_t* adj, const void* f_t,
                              const double* ns, const double* lam_next, double* lam_t,
                              double* grad_ns, void* stream) {
    if (!valid_params(p) || (C8 && !codes8) || !codes || !tile_records || !adj || !f_t ||
        !lam_next || !lam_t || n <= 0)
        return LBM_EINVAL;
    if (p->storage != LBM_F64 && p->storage != LBM_F64_SHIFTED) return LBM_EINVAL;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    hipStream_t s = as_stream(stream);
    const TrtConst c = make_trt_const(*p);
    const double* f = static_cast<const double*>(f_t);
    const SweepLaunch l = adjoint_launch(p->flags, n);
    const XcdMap map = l.towards(lam_t < lam_next);
    return with_policy_waves(l.policy, n, [&](auto pol, auto waves) {
        if (ns) k_adjoint_coded<true, pol, C8, waves><<<l.grid, l.block, 0, s>>>(f, codes8, codes, tile_records, adj, ns, lam_next, lam_t, grad_ns, n, stride, c, map);
        else k_adjoint_coded<false, pol, C8, waves><<<l.grid, l.block, 0, s>>>(f, codes8, codes, tile_records, adj, ns, lam_next, lam_t, nullptr, n, stride, c, map);
        return after_launch();
    });
}

}  // namespace lbm

extern "C" lbm_status lbm_step_adjoint_c16(const lbm_params* p, int64_t n, int64_t stride,
                                           const int16_t* codes, const int32_t* tile_records,
                                           const uint32_t* adj, const void* f_t,
                                           const double* ns, const double* lam_next,
                                           double* lam_t, double* grad_ns, void* stream) {
    return step_adjoint_coded<false>(p, n, stride, nullptr, codes, tile_records, adj, f_t, ns,
                                     lam_next, lam_t, grad_ns, stream);
}

extern "C" lbm_status lbm_step_adjoint_c8(const lbm_params* p, int64_t n, int64_t stride,
                                          const int8_t* codes8, const int16_t* codes,
                                          const int32_t* tile_records, const uint32_t* adj,
                                          const void* f_t, const double* ns,
                                          const double* lam_next, double* lam_t,
                                          double* grad_ns, void* stream) {
    return step_adjoint_coded<true>(p, n, stride, codes8, codes, tile_records, adj, f_t, ns,
                                    lam_next, lam_t, grad_ns, stream);
}
