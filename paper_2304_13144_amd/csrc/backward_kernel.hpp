// Gradient of the fitting objective (MLIP-3 paper eq. 7) with respect to
// theta, given the upstream gradients gE = dL/dE, gF = dL/dF, gS = dL/dS.
//
// Because F = -dE/dx and S = -dE/deps, the force and stress terms are
// -d/dtheta of one directional derivative of E: along x -> x + t gF and
// eps = t gS every pair vector moves by
//     dr_ij = gF_j - gF_i + gS r_ij,
// and dE/dt = sum_i dV_i/dt with dV_i/dt = sum_j g_ij . dr_ij.  So
//     dL/dtheta = sum_i [ gE_cfg(i) dV_i/dtheta - d(dV_i/dt)/dtheta ].
// Per neighborhood (moments recomputed, nothing stored per pair):
//   * tangent moments  Mdot_k = sum_j d(f_mu m_k)/dr . dr_ij;
//   * the contraction program run on dual numbers (value, tangent) gives
//     B_alpha and Bdot_alpha, dV/dM and its tangent H Mdot;
//   * theta = xi_alpha:   gE B_alpha - Bdot_alpha;  theta = xi_0[z_i]: gE;
//   * theta = c^(beta)_{mu,z_i,z}: sum over pairs with z_j = z of
//       gE Q_beta P_mu - [ Q_beta (Phat_mu + grad P_mu . dr) + Q'_beta (rhat . dr) P_mu ]
//     with P_mu = sum_{k in mu} (dV/dM_k) m_k and Phat_mu the same with H Mdot.
// Two launches: the moments, their tangents and the dual contraction of 64
// neighborhoods per block (nothing but dV/dM and H Mdot leaves it), then the
// pairs.  Each neighborhood's contributions are stored column by column
// (entry (i, k) at cols[k * ldn + i]: the N_lin columns of xi, then the c block
// of its own central species), and a column reduction in FP64 adds them in a
// fixed order, the c block under the neighborhood's species.  (The rows over
// all of theta that this replaces held zeros for the other central species
// and were written 8 bytes per cache line, and the contraction ran on one lane
// per neighborhood and spilled: 1.85 ms of a training step's 2.76 ms at level
// 20, 10,357 atoms; these two launches take 0.13 ms and the step 0.52 to 0.57.)
#pragma once

#include "efs_kernel.hpp"

namespace mtp {
namespace ad {   // dual numbers; fma for them is found by argument-dependent lookup

template <typename T> struct Dual {
    T v, d;
    Dual() = default;
    __device__ constexpr Dual(T x) : v(x), d(T(0)) {}
    __device__ constexpr Dual(T x, T y) : v(x), d(y) {}
    __device__ Dual &operator+=(const Dual &o) {
        v += o.v;
        d += o.d;
        return *this;
    }
};
template <typename T> __device__ inline Dual<T> operator*(const Dual<T> &a, const Dual<T> &b) {
    return Dual<T>(a.v * b.v, ::fma(a.v, b.d, a.d * b.v));
}
template <typename T> __device__ inline Dual<T> operator+(const Dual<T> &a, const Dual<T> &b) {
    return Dual<T>(a.v + b.v, a.d + b.d);
}
template <typename T> __device__ inline Dual<T> fma(const Dual<T> &a, const Dual<T> &b, const Dual<T> &c) {
    return Dual<T>(::fma(a.v, b.v, c.v), ::fma(a.v, b.d, ::fma(a.d, b.v, c.d)));
}

// products with constants and coefficients, which carry no tangent
template <typename T> struct Plain { using type = T; };
template <typename T> __device__ inline Dual<T> cmul(typename Plain<T>::type c, const Dual<T> &x) {
    return Dual<T>(c * x.v, c * x.d);
}
template <typename T>
__device__ inline Dual<T> cfma(typename Plain<T>::type c, const Dual<T> &x, const Dual<T> &y) {
    return Dual<T>(::fma(c, x.v, y.v), ::fma(c, x.d, y.d));
}

}  // namespace ad
using ad::Dual;

// receives B_alpha (value, tangent) and writes gE B - Bdot into its column
// (padded to whole blocks of 64 neighborhoods, as for ColSink)
template <typename T> struct GradSink {
    T *cols;
    int64_t ldn;
    uint32_t row;
    T gE;
    struct Ref {
        T *col;
        uint32_t row;
        T gE;
        __device__ void operator=(const Dual<T> &b) const { col[row] = fma(gE, b.v, -b.d); }
    };
    __device__ Ref operator[](int a) const { return Ref{cols + (int64_t)a * ldn, row, gE}; }
};

template <typename T> struct LdsDual {   // moment k (value and tangent) of one neighborhood
    const T *v, *d;
    __device__ Dual<T> operator[](int k) const { return Dual<T>(v[k * 64], d[k * 64]); }
};

template <typename T> __device__ inline void pair_dr(const BwdArgs &b, int64_t atom, int64_t slot, T x, T y, T z,
                                                     T &d0, T &d1, T &d2) {
    d0 = d1 = d2 = T(0);
    if (b.gF) {
        const int j = b.nbr_j[slot];
        d0 = T(b.gF[3 * j] - b.gF[3 * atom]);
        d1 = T(b.gF[3 * j + 1] - b.gF[3 * atom + 1]);
        d2 = T(b.gF[3 * j + 2] - b.gF[3 * atom + 2]);
    }
    if (b.gS) {
        const double *W = b.gS + 9 * (int64_t)b.atom_cfg[atom];
        d0 = fma(T(W[0]), x, fma(T(W[1]), y, fma(T(W[2]), z, d0)));
        d1 = fma(T(W[3]), x, fma(T(W[4]), y, fma(T(W[5]), z, d1)));
        d2 = fma(T(W[6]), x, fma(T(W[7]), y, fma(T(W[8]), z, d2)));
    }
}

// ---- tangent moments ------------------------------------------------------
// reduce-scattered over the K lanes of the neighborhood of c, as
// moments_scattered does
template <typename T, int L, int K>
__device__ inline void tangent_moments_scattered(const BwdArgs &b, const AtomCtx &c, const T *c_s,
                                                 T (&Md)[(Level<L>::NC + K - 1) / K * K]) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD, NCP = (NC + K - 1) / K * K;
    const EfsArgs &a = b.e;
    const int nt = a.n_types;
    const int sub = threadIdx.x % K;
    const T rc = T(a.r_cut);
    const T xs = T(2.0 / (a.r_cut - a.r_min));
    const T x0 = T(-(a.r_min + a.r_cut) / (a.r_cut - a.r_min));
#pragma unroll
    for (int k = 0; k < NCP; ++k) Md[k] = T(0);
    const SpeciesEnds species(c);
    for (int p = sub; p < c.ntot; p += K) {
        const int zj = species(p);
        const T x = T(c.rp[3 * p]), y = T(c.rp[3 * p + 1]), z = T(c.rp[3 * p + 2]);
        const T r = sqrt(efs::norm2(x, y, z));
        if (!(r < rc)) continue;
        T d0, d1, d2;
        pair_dr<T>(b, c.atom, c.atom * (int64_t)a.max_nbrs + p, x, y, z, d0, d1, d2);
        const T rdot = (x * d0 + y * d1 + z * d2) / r;
        T f[NR], fp[NR];
        {
            const T u = fma(r, xs, x0), dd = rc - r, cut = dd * dd, dcut = T(-2) * dd;
            T Tb[NPOLY], dT[NPOLY];
            Tb[0] = T(1);
            Tb[1] = u;
            dT[0] = T(0);
            dT[1] = T(1);
#pragma unroll
            for (int q = 2; q < NPOLY; ++q) {
                Tb[q] = fma(T(2) * u, Tb[q - 1], -Tb[q - 2]);
                dT[q] = fma(T(2) * u, dT[q - 1], fma(T(2), Tb[q - 1], -dT[q - 2]));
            }
#pragma unroll
            for (int mu = 0; mu < NR; ++mu) {
                const CoefRow<T> cm = coef_row(c_s, mu, c.zi, zj, nt);
                T s = T(0), sp = T(0);
#pragma unroll
                for (int q = 0; q < NPOLY; ++q) {
                    s = fma(cm[q], Tb[q], s);
                    sp = fma(cm[q], dT[q], sp);
                }
                f[mu] = s * cut;
                fp[mu] = fma(sp * xs, cut, s * dcut);
            }
        }
        T mono[20];
        efs::monomials(x, y, z, mono);
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int mu = LV::comp_mu[k];
            T gdot = T(0);
            if (LV::comp_dmonox[k] >= 0)
                gdot = fma(T(LV::comp_dfacx[k]) * mono[LV::comp_dmonox[k] < 0 ? 0 : LV::comp_dmonox[k]], d0, gdot);
            if (LV::comp_dmonoy[k] >= 0)
                gdot = fma(T(LV::comp_dfacy[k]) * mono[LV::comp_dmonoy[k] < 0 ? 0 : LV::comp_dmonoy[k]], d1, gdot);
            if (LV::comp_dmonoz[k] >= 0)
                gdot = fma(T(LV::comp_dfacz[k]) * mono[LV::comp_dmonoz[k] < 0 ? 0 : LV::comp_dmonoz[k]], d2, gdot);
            Md[k] = fma(fp[mu] * rdot, mono[LV::comp_mono[k]], fma(f[mu], gdot, Md[k]));
        }
    }
    efs::reduce_scatter<T, NCP, K>(Md, sub);
}

// ---- moments, tangents and the dual contraction -----------------------------
// 64 neighborhoods per block, eight lanes each for the moments, eight
// wavefronts (clusters) for the contraction.
template <typename T, int L>
__global__ __launch_bounds__(512) void bwd_moments_contract(const BwdArgs b) {
    using LV = Level<L>;
    constexpr int K = 8, NC = LV::NC, NR = LV::NRAD, NCP = (NC + K - 1) / K * K;
    const EfsArgs &a = b.e;
    __shared__ T c_s[NR * MAX_TYPES * MAX_TYPES * NPOLY];
    __shared__ T sM[NCP][64], sD[NCP][64];
    __shared__ Dual<T> sum[Fact<L, K>::template rows<Dual<T>>()][64];
    const int sub = threadIdx.x % K, la = threadIdx.x / K;
    const AtomCtx c = atom_ctx<K, 64 * K>(a);
    const PairVector first(a, c, sub);
    load_coefs<T, NR, 64 * K>(a, c_s);
    __syncthreads();
    {
        T M[NCP];
        moments_scattered<T, L, K>(a, c, c_s, first, M);
#pragma unroll
        for (int i = 0; i < NCP / K; ++i) sM[sub * (NCP / K) + i][la] = M[i];
    }
    {
        T M[NCP];
        tangent_moments_scattered<T, L, K>(b, c, c_s, M);
#pragma unroll
        for (int i = 0; i < NCP / K; ++i) sD[sub * (NCP / K) + i][la] = M[i];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.x * 64 + lane;
    const bool live = slot < a.n_atoms;
    const T gE = live && b.gE ? T(b.gE[b.atom_cfg[slot]]) : T(0);
    T *dv = static_cast<T *>(a.dmbuf) + slot, *dt = static_cast<T *>(b.dtbuf) + slot;
    const auto out = [&](int k, const Dual<T> &v) {
        if (live) {
            dv[(int64_t)k * a.n_atoms] = v.v;
            dt[(int64_t)k * a.n_atoms] = v.d;
        }
    };
    fact_body<Dual<T>, L, true, K>(LdsDual<T>{&sM[0][lane], &sD[0][lane]}, XiPtr<T>{xi_of<T>(a)},
                                   GradSink<T>{static_cast<T *>(b.cols), a.ldn, (uint32_t)slot, gE}, sum, out,
                                   [](const Dual<T> &) {});
}

// ---- the c block of the own central species ----------------------------------
// K lanes per neighborhood; dV/dM and H Mdot of the block's neighborhoods in
// LDS, where the K lanes read the same word (in registers they cost 4 NC
// VGPRs per lane)
template <typename T, int L, int K>
__global__ __launch_bounds__(256) void bwd_pairs(const BwdArgs b) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD, NL = LV::NLIN, ND = NR * NPOLY;
    const EfsArgs &a = b.e;
    __shared__ T s_dv[NC][256 / K], s_dt[NC][256 / K];
    const int nt = a.n_types;
    const int sub = threadIdx.x % K, la = threadIdx.x / K;
    const AtomCtx c = atom_ctx<K>(a);
    const T rc = T(a.r_cut);
    const T xs = T(2.0 / (a.r_cut - a.r_min));
    const T x0 = T(-(a.r_min + a.r_cut) / (a.r_cut - a.r_min));
    {
        const T *pv = static_cast<const T *>(a.dmbuf);
        const T *pt = static_cast<const T *>(b.dtbuf);
        // loaded unconditionally, in bounds, so that all loads are in flight together
        constexpr int N = (NC + K - 1) / K;
        T v[N], t[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int64_t at = (int64_t)(i * K + sub < NC ? i * K + sub : NC - 1) * a.n_atoms + (c.live ? c.slot : 0);
            v[i] = pv[at];
            t[i] = pt[at];
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i * K + sub < NC) {
                s_dv[i * K + sub][la] = c.live ? v[i] : T(0);
                s_dt[i * K + sub][la] = c.live ? t[i] : T(0);
            }
    }
    __syncthreads();
    const T gE = (c.live && b.gE) ? T(b.gE[b.atom_cfg[c.atom]]) : T(0);
    T *cols = static_cast<T *>(b.cols) + (int64_t)NL * a.ldn + c.slot;   // the c columns, [t][mu][beta]
    int gstart = 0;
    for (int t = 0; t < nt; ++t) {
        T acc[ND];
#pragma unroll
        for (int k = 0; k < ND; ++k) acc[k] = T(0);
        for (int qq = sub; qq < tcount(c, t); qq += K) {
            const int p = gstart + qq;
            const T x = T(c.rp[3 * p]), y = T(c.rp[3 * p + 1]), z = T(c.rp[3 * p + 2]);
            const T r = sqrt(efs::norm2(x, y, z));
            if (!(r < rc)) continue;
            T d0, d1, d2;
            pair_dr<T>(b, c.atom, c.atom * (int64_t)a.max_nbrs + p, x, y, z, d0, d1, d2);
            const T rdot = (x * d0 + y * d1 + z * d2) / r;
            T Q[NPOLY], Qp[NPOLY];
            {
                const T u = fma(r, xs, x0), dd = rc - r, cut = dd * dd, dcut = T(-2) * dd;
                T Tb[NPOLY], dT[NPOLY];
                Tb[0] = T(1);
                Tb[1] = u;
                dT[0] = T(0);
                dT[1] = T(1);
#pragma unroll
                for (int q = 2; q < NPOLY; ++q) {
                    Tb[q] = fma(T(2) * u, Tb[q - 1], -Tb[q - 2]);
                    dT[q] = fma(T(2) * u, dT[q - 1], fma(T(2), Tb[q - 1], -dT[q - 2]));
                }
#pragma unroll
                for (int q = 0; q < NPOLY; ++q) {
                    Q[q] = Tb[q] * cut;
                    Qp[q] = fma(dT[q] * xs, cut, Tb[q] * dcut);
                }
            }
            T mono[20];
            efs::monomials(x, y, z, mono);
            T P[NR], Ph[NR], GP[NR];
#pragma unroll
            for (int mu = 0; mu < NR; ++mu) P[mu] = Ph[mu] = GP[mu] = T(0);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const int mu = LV::comp_mu[k];
                const T m = mono[LV::comp_mono[k]];
                const T dv = s_dv[k][la];
                P[mu] = fma(dv, m, P[mu]);
                Ph[mu] = fma(s_dt[k][la], m, Ph[mu]);
                T gdot = T(0);
                if (LV::comp_dmonox[k] >= 0)
                    gdot = fma(T(LV::comp_dfacx[k]) * mono[LV::comp_dmonox[k] < 0 ? 0 : LV::comp_dmonox[k]], d0, gdot);
                if (LV::comp_dmonoy[k] >= 0)
                    gdot = fma(T(LV::comp_dfacy[k]) * mono[LV::comp_dmonoy[k] < 0 ? 0 : LV::comp_dmonoy[k]], d1, gdot);
                if (LV::comp_dmonoz[k] >= 0)
                    gdot = fma(T(LV::comp_dfacz[k]) * mono[LV::comp_dmonoz[k] < 0 ? 0 : LV::comp_dmonoz[k]], d2, gdot);
                GP[mu] = fma(dv, gdot, GP[mu]);
            }
#pragma unroll
            for (int mu = 0; mu < NR; ++mu) {
                const T w1 = fma(gE, P[mu], -(Ph[mu] + GP[mu]));   // multiplies Q_beta
                const T w2 = -rdot * P[mu];                         // multiplies Q'_beta
#pragma unroll
                for (int q = 0; q < NPOLY; ++q)
                    acc[mu * NPOLY + q] = fma(w1, Q[q], fma(w2, Qp[q], acc[mu * NPOLY + q]));
            }
        }
        efs::reduce_scatter<T, ND, K>(acc, sub);
        if (c.live) {
#pragma unroll
            for (int i = 0; i < ND / K; ++i) cols[(int64_t)(t * ND + sub * (ND / K) + i) * a.ldn] = acc[i];
        }
        gstart += tcount(c, t);
    }
}

template <int L, typename T> int launch_backward_level_t(const BwdArgs &b);

#define MTP_BWD_LEVEL_T(LEVEL, TT)                                                                        \
    template <> int launch_backward_level_t<LEVEL, TT>(const BwdArgs &b) {                                \
        const int64_t n = b.e.n_atoms;                                                                    \
        if (n == 0) return 0;                                                                             \
        hipLaunchKernelGGL((bwd_moments_contract<TT, LEVEL>), dim3((unsigned)((n + 63) / 64)), dim3(512), \
                           0, b.e.stream, b);                                                             \
        hipLaunchKernelGGL((bwd_pairs<TT, LEVEL, 8>), dim3((unsigned)((n + 31) / 32)), dim3(256), 0,      \
                           b.e.stream, b);                                                                \
        return (int)hipGetLastError();                                                                    \
    }

}  // namespace mtp
