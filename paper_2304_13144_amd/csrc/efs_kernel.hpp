// Fused per-neighborhood kernel: radial functions -> moments -> contraction
// -> site energy -> dV/dM -> pair gradients, virial and (optionally) the row
// b_i = dV_i/dtheta.  Included by one generated translation unit per level.
//
// Work decomposition: LANES consecutive lanes of a wavefront share one
// neighborhood.  Each lane walks every LANES-th pair of the list and keeps
// its own partial moments in registers; a butterfly of cross-lane shuffles
// then gives every lane the full moments.  The contraction program (Level<L>,
// generated at build time) runs in registers.  The pair loop is walked a
// second time for the gradients, one neighbor species after the other, so
// the radial-coefficient part of b_i needs only N_rad x N_polyn accumulators.
//
// Pair gradient (paper eqs. 3-4; V from eq. 2):
//   g_ij = dV_i/dr_ij = sum_mu [ f'_mu(r) P_mu r_hat + f_mu(r) grad P_mu ],
//   P_mu(r) = sum_{k in mu} (dV/dM_k) x^a y^b z^c  (k = component (mu; a,b,c)).
// b-row entries of c (eq. 4): dV_i/dc^(beta)_{mu,z_i,z} = sum_{j: z_j = z} Q_beta(r_ij) P_mu(r_ij),
// Q_beta = T_beta(x) (R_cut - r)^2.
//
// Rows are FP64 in every form and stored column-major: entry (i, k) at
// brow[k * ldn + i], so that the lanes of a wavefront (consecutive
// neighborhoods) write consecutive words of one column.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "device_util.hpp"
#include "kernel_args.hpp"

namespace mtp {

template <int L> struct Level;

namespace efs {

template <typename T> __device__ inline T xor_shuffle(T v, int mask) { return __shfl_xor(v, mask, 64); }

// Reduce-scatter over the K lanes of a group (sub = lane % K): afterwards
// v[0 .. M/K) of lane sub holds the group totals of v[sub M/K .. (sub+1) M/K).
// Each round halves the live values (the lane whose bit O is set keeps the
// upper half), so it takes M (1 - 1/K) shuffles instead of the M log2 K of a
// butterfly all-reduce.
template <typename T, int M, int N, int O> __device__ inline void rs_step(T (&v)[M], int sub) {
    if constexpr (O >= 1) {
        const bool up = (sub & O) != 0;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const T send = up ? v[i] : v[i + N / 2];
            const T keep = up ? v[i + N / 2] : v[i];
            v[i] = keep + xor_shuffle(send, O);
        }
        rs_step<T, M, N / 2, O / 2>(v, sub);
    }
}
template <typename T, int M, int K> __device__ inline void reduce_scatter(T (&v)[M], int sub) {
    static_assert(M % K == 0, "reduce_scatter: M must be a multiple of K");
    rs_step<T, M, M, K / 2>(v, sub);
}

// x^2 + y^2 + z^2, its roundings spelled out: left to the compiler, which of
// the products is rounded changes with the code around it
template <typename T> __device__ inline T norm2(T x, T y, T z) { return fma(z, z, fma(x, x, y * y)); }

// monomials x^a y^b z^c, a+b+c <= 3, in the order of monomial_index()
template <typename T> __device__ inline void monomials(T x, T y, T z, T (&m)[20]) {
    m[0] = T(1); m[1] = x; m[2] = y; m[3] = z;
    m[4] = x * x; m[5] = x * y; m[6] = x * z; m[7] = y * y; m[8] = y * z; m[9] = z * z;
    m[10] = m[4] * x; m[11] = m[4] * y; m[12] = m[4] * z; m[13] = m[7] * x; m[14] = m[5] * z;
    m[15] = m[9] * x; m[16] = m[7] * y; m[17] = m[7] * z; m[18] = m[9] * y; m[19] = m[9] * z;
}

}  // namespace efs

// theta = [xi_0 (n_types) | xi_alpha (n_lin) | c] in the arithmetic type T
template <typename T> __device__ inline const T *theta_of(const EfsArgs &a);
template <> __device__ inline const double *theta_of<double>(const EfsArgs &a) { return a.th64; }
template <> __device__ inline const float *theta_of<float>(const EfsArgs &a) { return a.th32; }
template <typename T> __device__ inline const T *xi0_of(const EfsArgs &a) { return theta_of<T>(a); }
template <typename T> __device__ inline const T *xi_of(const EfsArgs &a) { return theta_of<T>(a) + a.n_types; }
template <typename T> __device__ inline const T *coef_of(const EfsArgs &a) {
    return theta_of<T>(a) + a.n_types + a.n_lin;
}

template <typename T> struct XiPtr {      // xi_alpha, read where the program needs it
    const T *p;
    __device__ T operator[](int k) const { return p[k]; }
};

// Per-neighborhood context shared by the pair kernels.
struct AtomCtx {
    bool live;
    int64_t slot, atom;
    int zi, ntot;
    int tc[MAX_TYPES];
    const double *rp;
};

// BS: the launch's block size, a compile-time constant (blockDim.x is read
// from the dispatch packet: one more dependent load before the first real one)
template <int K, int BS = 256> __device__ inline AtomCtx atom_ctx(const EfsArgs &a, int64_t blk = -1) {
    AtomCtx c;
    const int nt = a.n_types;
    c.slot = (blk < 0 ? (int64_t)blockIdx.x : blk) * (BS / K) + threadIdx.x / K;
    c.live = c.slot < a.n_atoms;
    c.atom = c.live ? (a.atom_list ? (int64_t)a.atom_list[c.slot] : c.slot) : 0;
    int zi = c.live ? a.type[c.atom] : 0;
    c.zi = zi < 0 ? 0 : (zi >= nt ? nt - 1 : zi);
    c.ntot = 0;
#pragma unroll
    for (int t = 0; t < MAX_TYPES; ++t) {
        c.tc[t] = (c.live && t < nt) ? a.tcnt[c.atom * nt + t] : 0;
        c.ntot += c.tc[t];
    }
    c.rp = a.r + c.atom * (int64_t)a.max_nbrs * 3;
    return c;
}

// neighbors of species t, picked by masks: a runtime index into c.tc would
// put the whole context in scratch memory, and a read of the counts again is
// a memory latency in the pair loop
__device__ inline int tcount(const AtomCtx &c, int t) {
    int n = 0;
#pragma unroll
    for (int k = 0; k < MAX_TYPES; ++k) n |= c.tc[k] & -(int)(t == k);
    return n;
}

// Species of list position p (species come in order; p below the total)
struct SpeciesEnds {
    int e[MAX_TYPES - 1];
    __device__ explicit SpeciesEnds(const AtomCtx &c) {
        e[0] = c.tc[0];
#pragma unroll
        for (int k = 1; k < MAX_TYPES - 1; ++k) e[k] = e[k - 1] + c.tc[k];
    }
    __device__ int operator()(int p) const {
        int z = 0;
#pragma unroll
        for (int k = 0; k < MAX_TYPES - 1; ++k) z += p >= e[k] ? 1 : 0;
        return z;
    }
};

// The pair vector of list position p of c, loaded in bounds whatever p is
struct PairVector {
    double x, y, z;
    __device__ PairVector(const EfsArgs &a, const AtomCtx &c, int p) {
        const double *r = c.rp + 3 * (p < a.max_nbrs ? p : a.max_nbrs - 1);
        x = r[0];
        y = r[1];
        z = r[2];
    }
};

// The radial coefficients c_{mu, z_i, z_j, beta} in LDS as
// [mu][beta][z_i][z_j], the species padded to MAX_TYPES: the lanes of a
// wavefront, whose pairs have different (z_i, z_j), read one (mu, beta) at a
// time from one 16-word row (no bank conflicts; the parameter order
// [mu][z_i][z_j][beta] puts them NPOLY words apart), and beta steps by a
// constant offset.
constexpr int COEF_TT = MAX_TYPES * MAX_TYPES;
// (The caller's barrier.)
template <typename T, int NR, int BS = 256> __device__ inline void load_coefs(const EfsArgs &a, T *c_s) {
    const T *cg = coef_of<T>(a);
    const int nt = a.n_types, ntt = nt * nt;
    const int ncoef = NR * ntt * NPOLY;
    for (int k = threadIdx.x; k < ncoef; k += BS) {
        const int b = k % NPOLY, pair = (k / NPOLY) % ntt, mu = k / (NPOLY * ntt);
        c_s[(mu * NPOLY + b) * COEF_TT + (pair / nt) * MAX_TYPES + pair % nt] = cg[k];
    }
}
template <typename T> struct CoefRow {   // c_{mu, z_i, z_j, beta} over beta, from the LDS copy
    const T *p;
    __device__ T operator[](int b) const { return p[b * COEF_TT]; }
};
template <typename T> __device__ inline CoefRow<T> coef_row(const T *c_s, int mu, int zi, int zj, int) {
    return CoefRow<T>{c_s + mu * NPOLY * COEF_TT + zi * MAX_TYPES + zj};
}

// ---- kernel 1: moments (eq. 3), LANES lanes per neighborhood -------------
// Latency-bound in the small, so nothing in the pair loop waits for memory but
// the next pair vector (the species of a position came from counts read again
// at each change: FP32, 19,652 atoms, level 16, with the contraction 30.2 ->
// 20.8 us).
// Moments of the neighborhood of c, reduce-scattered over its K lanes: on
// return M[i] of lane sub holds component sub NCP/K + i (NCP = NC padded to
// a multiple of K).  c_s: the radial coefficients, already in LDS; next: the
// lane's first pair vector, loaded by the caller before its barrier.
template <typename T, int L, int K>
__device__ inline void moments_scattered(const EfsArgs &a, const AtomCtx &c, const T *c_s, PairVector next,
                                         T (&M)[(Level<L>::NC + K - 1) / K * K]) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD;
    const int nt = a.n_types;
    const int sub = threadIdx.x % K;
    const T rc = T(a.r_cut);
    const T xs = T(2.0 / (a.r_cut - a.r_min));
    const T x0 = T(-(a.r_min + a.r_cut) / (a.r_cut - a.r_min));
    constexpr int NCP = (NC + K - 1) / K * K;   // padded for the reduce-scatter
#pragma unroll
    for (int k = 0; k < NCP; ++k) M[k] = T(0);
    const SpeciesEnds species(c);
    for (int p = sub; p < c.ntot; p += K) {
        const int zj = species(p);
        const T x = T(next.x), y = T(next.y), z = T(next.z);
        next = PairVector(a, c, p + K < c.ntot ? p + K : p);   // in flight while this one is used
        const T r = sqrt(efs::norm2(x, y, z));
        if (!(r < rc)) continue;
        T fm[NR];
        {
            const T u = fma(r, xs, x0), d = rc - r, cut = d * d;
            T Tb[NPOLY];
            Tb[0] = T(1);
            Tb[1] = u;
#pragma unroll
            for (int b = 2; b < NPOLY; ++b) Tb[b] = fma(T(2) * u, Tb[b - 1], -Tb[b - 2]);
#pragma unroll
            for (int mu = 0; mu < NR; ++mu) {
                const CoefRow<T> cm = coef_row(c_s, mu, c.zi, zj, nt);
                T s = T(0);
#pragma unroll
                for (int b = 0; b < NPOLY; ++b) s = fma(cm[b], Tb[b], s);
                fm[mu] = s * cut;
            }
        }
        T mono[20];
        efs::monomials(x, y, z, mono);
#pragma unroll
        for (int k = 0; k < NC; ++k) M[k] = fma(fm[LV::comp_mu[k]], mono[LV::comp_mono[k]], M[k]);
    }
    efs::reduce_scatter<T, NCP, K>(M, sub);
}

template <typename T, int L, int K>
__global__ __launch_bounds__(256) void efs_moments(const EfsArgs a) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD;
    constexpr int NCP = (NC + K - 1) / K * K;
    __shared__ T c_s[NR * MAX_TYPES * MAX_TYPES * NPOLY];
    const int sub = threadIdx.x % K;
    const AtomCtx c = atom_ctx<K>(a);
    const PairVector first(a, c, sub);
    load_coefs<T, NR>(a, c_s);
    __syncthreads();
    T M[NCP];
    moments_scattered<T, L, K>(a, c, c_s, first, M);
    if (c.live) {
        T *out = static_cast<T *>(a.mbuf);
#pragma unroll
        for (int i = 0; i < NCP / K; ++i) {
            const int k = sub * (NCP / K) + i;
            if (k < NC) out[(int64_t)k * a.n_atoms + c.slot] = M[i];
        }
    }
}

// ---- kernel 2: contraction, site energy (eq. 2), dV/dM -------------------
// One block holds 64 neighborhoods (one per lane) and NW = four or eight
// wavefronts that share the contraction program.  FP64 (and FP32 above level
// 16) runs the factorised program (fact_body), FP32 up to level 16 the
// expanded one (expanded_body).
template <typename T> struct ColLoad {   // component k of one neighborhood, [k][n] layout
    const T *p;
    int64_t s;
    __device__ T operator[](int k) const { return p[k * s]; }
};
// receives B_alpha into column c0 + alpha of the FP64 rows: a uniform column
// base plus the lane's row index, consecutive lanes writing consecutive words
// (columns are padded to whole blocks of 64 rows: lanes past the last
// neighborhood write the padding, without a branch around every store)
struct ColSink {
    double *p;
    int64_t s;
    int c0;
    uint32_t row;
    struct Ref {
        double *col;
        uint32_t row;
        __device__ void operator=(const double &v) const { col[row] = v; }
    };
    __device__ Ref operator[](int k) const { return Ref{p + (int64_t)(c0 + k) * s, row}; }
};
struct NoSink {
    struct Ref {
        template <typename V> __device__ void operator=(const V &) const {}
    };
    __device__ Ref operator[](int) const { return Ref{}; }
};

template <typename T> struct LdsCol {   // component k of one neighborhood, [k][64] in LDS
    const T *p;
    __device__ T operator[](int k) const { return p[k * 64]; }
};

// products with constants and coefficients (which carry no tangent when the
// program runs on dual numbers)
__device__ inline double cmul(double c, double x) { return c * x; }
__device__ inline float cmul(float c, float x) { return c * x; }
__device__ inline double cfma(double c, double x, double y) { return fma(c, x, y); }
__device__ inline float cfma(float c, float x, float y) { return fma(c, x, y); }

// between the graphs of a cluster: no instruction is scheduled across, so
// that the graphs are not interleaved, which would hold the intermediates of
// many at once
#define MTP_FACT_SCHED() __builtin_amdgcn_sched_barrier(0)

template <typename T, int L> constexpr bool expanded_program() {
    return sizeof(T) == sizeof(float) && Level<L>::EXPANDED;
}

// xi_alpha into LDS for the factorised program: read there by a wavefront as
// one word, in order with its other LDS reads; a scalar load is waited for
// together with everything outstanding.  256,000 atoms at level 16: 223 -> 203
// us for moments and contraction, level 24: 237 -> 226 (the expanded program
// reads xi in runs and is faster from scalar loads: 20.4 us, 26.6 from LDS, at
// 19,652 atoms).  (The caller's barrier.)
template <typename T, int L> constexpr int xi_words() { return expanded_program<T, L>() ? 1 : Level<L>::NLIN; }
template <typename T, int L, int BS> __device__ inline void load_xi(const EfsArgs &a, T *s_xi) {
    if constexpr (!expanded_program<T, L>()) {
        const T *xi = xi_of<T>(a);
        for (int k = threadIdx.x; k < Level<L>::NLIN; k += BS) s_xi[k] = xi[k];
    }
}

// The clusters of the factorised program for NW wavefronts.
template <int L, int NW> struct Fact {
    using LV = Level<L>;
    static_assert(NW == 4 || NW == 8, "four or eight clusters");
    static constexpr int MAXC = NW == 4 ? LV::FMAX4 : LV::FMAX8;
    static constexpr int ROWS = LV::NC + LV::NPROD;          // dV/dM, then the sums X_p
    static constexpr int SLICE = (ROWS + NW - 1) / NW;
    static constexpr int ncomp(int P) {
        if constexpr (NW == 4) return LV::fncomp4[P];
        else return LV::fncomp8[P];
    }
    static constexpr int comp(int P, int i) {
        if constexpr (NW == 4) return LV::fcomp4[P][i];
        else return LV::fcomp8[P][i];
    }
    // position of sum k in cluster P's list, or -1
    static constexpr int find(int P, int k) {
        for (int i = 0; i < ncomp(P); ++i)
            if (comp(P, i) == k) return i;
        return -1;
    }
    static constexpr bool is_low(int k) {
        for (int i = 0; i < LV::NLOWC; ++i)
            if (LV::low_comp[i] == k) return true;
        return false;
    }
    // first of cluster P's sums where every cluster has rows of its own
    static constexpr int base(int P) {
        int n = 0;
        for (int Q = 0; Q < P; ++Q) n += ncomp(Q);
        return n;
    }
    // Every cluster's sums side by side in LDS, one barrier, each total added
    // by the wavefront that needs it: where that leaves the block its room on
    // the compute unit (beside the moments; eight wavefronts fill one by their
    // registers, of four wavefronts two blocks do).  Otherwise one row per
    // sum, and NW steps with a barrier each: 864 atoms at level 16 16.2 us,
    // side by side 13.0; 16 configurations at level 12 10.6 and 9.2.
    template <typename T> static constexpr bool side_by_side() {
        return (base(NW) + LV::NC) * 64 * sizeof(T) <= (NW == 8 ? 112 : 64) * 1024;
    }
    template <typename T> static constexpr int rows() { return side_by_side<T>() ? (base(NW) > 0 ? base(NW) : 1) : ROWS; }
    template <int P, typename T, int... I>
    static __device__ __forceinline__ void put(const T (&d)[MAXC], T (*sum)[64], int lane,
                                               std::integer_sequence<int, I...>) {
        ((sum[base(P) + I][lane] = d[I]), ...);
    }
    // the total of sum k, clusters in order
    template <int k, int P, typename T> static __device__ __forceinline__ void take(T (*sum)[64], int lane, T &v) {
        constexpr int i = find(P, k);
        if constexpr (i >= 0) {
            constexpr bool first = [] {
                for (int Q = 0; Q < P; ++Q)
                    if (find(Q, k) >= 0) return false;
                return true;
            }();
            const T x = sum[base(P) + i][lane];
            v = first ? x : v + x;
        }
    }
    template <int k, typename T, int... P>
    static __device__ __forceinline__ T total(T (*sum)[64], int lane, std::integer_sequence<int, P...>) {
        T v = T(0);
        (take<k, P>(sum, lane, v), ...);
        return v;
    }
    template <int k, typename T> static __device__ __forceinline__ T total(T (*sum)[64], int lane) {
        return total<k, T>(sum, lane, std::make_integer_sequence<int, NW>{});
    }
    // wavefront P's components of dV/dM (all but the low ones, dealt out in turn)
    template <int P, int k, typename T, typename OUT>
    static __device__ __forceinline__ void out_one(T (*sum)[64], int lane, const OUT &out) {
        if constexpr (k % (NW - 1) == P && !is_low(k)) out(k, total<k>(sum, lane));
    }
    template <int P, typename T, typename OUT, int... K>
    static __device__ __forceinline__ void out_all(T (*sum)[64], int lane, const OUT &out,
                                                   std::integer_sequence<int, K...>) {
        (out_one<P, K>(sum, lane, out), ...);
    }
    template <typename T, int... Q>
    static __device__ __forceinline__ void take_products(T (*sum)[64], int lane, T *X, std::integer_sequence<int, Q...>) {
        ((X[Q] = total<LV::NC + Q>(sum, lane)), ...);
    }
    // Everything below is unrolled by index sequences, not loops: d must be
    // addressed by constants from the start to stay in registers.
    // cluster P's share of sum k (SET: the first to reach it)
    template <int P, int k, bool SET, typename T>
    static __device__ __forceinline__ void add_one(const T (&d)[MAXC], T (*sum)[64], int lane) {
        if constexpr (k < ROWS) {
            constexpr int i = find(P, k);
            if constexpr (SET) sum[k][lane] = i >= 0 ? d[i < 0 ? 0 : i] : T(0);
            else if constexpr (i >= 0) sum[k][lane] = sum[k][lane] + d[i];
        }
    }
    template <int P, int Q, bool SET, typename T, int... I>
    static __device__ __forceinline__ void add(const T (&d)[MAXC], T (*sum)[64], int lane,
                                               std::integer_sequence<int, I...>) {
        (add_one<P, Q * SLICE + I, SET>(d, sum, lane), ...);
    }
    template <int P, bool WB, typename T, typename MP, typename XP, typename BP>
    static __device__ __forceinline__ void cluster(const MP &M, const T (&p)[LV::NPROD], const XP &xi, const BP &sink,
                                                   T (&d)[MAXC]) {
        if constexpr (NW == 4) LV::template fact4<P, WB>(M, p, xi, sink, d);
        else LV::template fact8<P, WB>(M, p, xi, sink, d);
    }
    // the last wavefront's end: dV/dM of the low components, written out
    template <typename T, typename OUT, int... I>
    static __device__ __forceinline__ void low_out(const T *d, T (*sum)[64], int lane, const OUT &out,
                                                   std::integer_sequence<int, I...>) {
        if constexpr (side_by_side<T>()) (out(LV::low_comp[I], total<LV::low_comp[I]>(sum, lane) + d[I]), ...);
        else (out(LV::low_comp[I], sum[LV::low_comp[I]][lane] + d[I]), ...);
    }
};

// The code of this wavefront's cluster P, inside a function whose own arrays
// it uses: written out as a switch there, since a helper holding the branches
// is simplified by itself first, where stores to a caller's array merge under
// a selected address and the array ends in scratch memory.
#define MTP_WAVE_CASE(Q, ...)                    \
    case Q:                                      \
        if constexpr (Q < NW) {                  \
            constexpr int P = Q;                 \
            __VA_ARGS__;                         \
        }                                        \
        break;
#define MTP_BY_WAVE(...)                         \
    switch (wave) {                              \
        MTP_WAVE_CASE(0, __VA_ARGS__)            \
        MTP_WAVE_CASE(1, __VA_ARGS__)            \
        MTP_WAVE_CASE(2, __VA_ARGS__)            \
        MTP_WAVE_CASE(3, __VA_ARGS__)            \
        MTP_WAVE_CASE(4, __VA_ARGS__)            \
        MTP_WAVE_CASE(5, __VA_ARGS__)            \
        MTP_WAVE_CASE(6, __VA_ARGS__)            \
        MTP_WAVE_CASE(7, __VA_ARGS__)            \
    }
// step S of the reduction: wavefront P adds slice (P + S) % NW, so every
// wavefront works on a slice of its own and each sum has a fixed order
#define MTP_REDUCE_STEP(S)                                                                                       \
    if constexpr (S < NW) {                                                                                      \
        MTP_BY_WAVE(FA::template add<P, (P + S) % NW, S == 0>(d, sum, lane,                                      \
                                                              std::make_integer_sequence<int, FA::SLICE>{}))     \
        __syncthreads();                                                                                         \
    }

// The factorised contraction of one block's 64 neighborhoods: wavefront w
// runs cluster w forward and back on the moments M, the last one the low
// graphs besides; the shares of dV/dM and of the sums X_p are added in LDS
// (sum): side by side and then each total, or every wavefront on a slice of
// its own per step; then the last wavefront closes the low graphs with the X_p
// while the others write dV/dM.
// out(k, v): component k of dV/dM; site(V): the site energy (last wavefront).
// No graph value passes between wavefronts and the trie walk is not repeated
// by each, as in the expanded form.  Bound by latencies at two wavefronts per
// SIMD (256 VGPRs hold a cluster's sums and intermediates; the FP64 units are
// busy a quarter to two fifths of the time).  Level 24, 160 configurations,
// 76,930 atoms (energies, forces, stress): 1,539 us with the expanded program
// in 25 launches through memory, 225 us in this one launch; level 16, 16,384
// atoms with rows: 27.8 -> 18.1 us for this launch.
template <typename T, int L, bool WB, int NW, typename MP, typename XP, typename BP, typename OUT, typename SITE>
__device__ __forceinline__ void fact_body(const MP &M, const XP &xi, const BP &sink, T (*sum)[64], const OUT &out,
                                          const SITE &site) {
    using LV = Level<L>;
    using FA = Fact<L, NW>;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    constexpr int NLA = LV::NLOW > 0 ? LV::NLOW : 1, NCA = LV::NLOWC > 0 ? LV::NLOWC : 1;
    T gl[NLA], p[LV::NPROD], dz[NLA], V = T(0);
    p[0] = T(1);
    if constexpr (LV::NLOW > 0) LV::template low_values<T>(M, gl, p);
    {
        T d[FA::MAXC];
        MTP_BY_WAVE(FA::template cluster<P, WB>(M, p, xi, sink, d))
        if (wave == NW - 1) LV::template low_functions<WB>(gl, xi, sink, dz, V);
        if constexpr (FA::template side_by_side<T>()) {
            MTP_BY_WAVE(FA::template put<P>(d, sum, lane, std::make_integer_sequence<int, FA::ncomp(P)>{}))
            __syncthreads();
        } else {
            MTP_REDUCE_STEP(0)
            MTP_REDUCE_STEP(1)
            MTP_REDUCE_STEP(2)
            MTP_REDUCE_STEP(3)
            MTP_REDUCE_STEP(4)
            MTP_REDUCE_STEP(5)
            MTP_REDUCE_STEP(6)
            MTP_REDUCE_STEP(7)
        }
    }
    if (wave == NW - 1) {
        T X[LV::NPROD], d[NCA];
        if constexpr (FA::template side_by_side<T>()) {
            FA::take_products(sum, lane, X, std::make_integer_sequence<int, LV::NPROD>{});
        } else {
#pragma unroll
            for (int q = 0; q < LV::NPROD; ++q) X[q] = sum[LV::NC + q][lane];
        }
        LV::template low_coupling<T>(gl, p, X, dz, V);
        if constexpr (LV::NLOW > 0) {
            LV::template low_reverse<T>(M, dz, d);
            FA::low_out(d, sum, lane, out, std::make_integer_sequence<int, LV::NLOWC>{});
        }
        site(V);
    } else if constexpr (FA::template side_by_side<T>()) {
        MTP_BY_WAVE(FA::template out_all<P>(sum, lane, out, std::make_integer_sequence<int, LV::NC>{}))
    } else {
        for (int k = wave; k < LV::NC; k += NW - 1)
            if (!FA::is_low(k)) out(k, sum[k][lane]);
    }
}

// the rows' constant entries, in whole columns of 64 rows: the species
// one-hot, then zeros from column nt + NL on (the c part's blocks and the
// padding; the pair pass writes the neighborhood's own c block over them
// afterwards).  Issued first, so that they drain while the graph values are
// computed (no vector memory load follows that would wait for them)
template <int L, int NW> __device__ inline void constant_columns(const EfsArgs &a, int64_t slot, int wave) {
    if (slot >= a.n_atoms) return;
    const int nt = a.n_types;
    const int64_t atom = a.atom_list ? (int64_t)a.atom_list[slot] : slot;
    int zi = a.type[atom];
    zi = zi < 0 ? 0 : (zi >= nt ? nt - 1 : zi);
    double *rowp = a.brow + slot;
    const int c0 = nt + Level<L>::NLIN;
    for (int k = wave; k < nt + a.ldb - c0; k += NW) {
        const int col = k < nt ? k : c0 + (k - nt);
        rowp[(int64_t)col * a.ldn] = k == zi ? 1.0 : 0.0;
    }
}

// V + xi_0[z_i] of slot's atom
template <typename T> __device__ inline void write_site(const EfsArgs &a, int64_t slot, T V) {
    if (slot >= a.n_atoms || !a.site_e) return;
    const int nt = a.n_types;
    const int64_t atom = a.atom_list ? (int64_t)a.atom_list[slot] : slot;
    int zi = a.type[atom];
    zi = zi < 0 ? 0 : (zi >= nt ? nt - 1 : zi);
    a.site_e[atom] = double(V) + double(xi0_of<T>(a)[zi]);
}

// The expanded contraction (FP32): the graphs are split into NW parts;
// wavefront w evaluates the graph values of part w, all exchange them through
// LDS (sg), each runs the (short) trie walk for V and dV/dg, and wavefront w
// the reverse pass of part w.  The partial dV/dM are added in LDS (sdm) in a
// fixed order; sdm may be the storage of the moments M.
template <typename T, int L, typename MA, int NW>
__device__ inline void expanded_body(const EfsArgs &a, int64_t blk, const MA &M, T (*sg)[64], T (*sdm)[64]) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NG = LV::NGRAPH;
    static_assert(LV::NPART == 4 && LV::NPART8 == 8 && (NW == 4 || NW == 8), "four or eight parts");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t slot = blk * 64 + lane;
    {
        T g[NG];
        if constexpr (NW == 4) {
            switch (wave) {
                case 0: LV::template graphs_part<0>(M, g); break;
                case 1: LV::template graphs_part<1>(M, g); break;
                case 2: LV::template graphs_part<2>(M, g); break;
                default: LV::template graphs_part<3>(M, g); break;
            }
        } else {
            switch (wave) {
                case 0: LV::template graphs_part8<0>(M, g); break;
                case 1: LV::template graphs_part8<1>(M, g); break;
                case 2: LV::template graphs_part8<2>(M, g); break;
                case 3: LV::template graphs_part8<3>(M, g); break;
                case 4: LV::template graphs_part8<4>(M, g); break;
                case 5: LV::template graphs_part8<5>(M, g); break;
                case 6: LV::template graphs_part8<6>(M, g); break;
                default: LV::template graphs_part8<7>(M, g); break;
            }
        }
#pragma unroll
        for (int G = 0; G < NG; ++G)
            if ((NW == 4 ? LV::graph_part[G] : LV::graph_part8[G]) == wave) sg[G][lane] = g[G];
    }
    __syncthreads();
    T gin[NG], dg[NG];
#pragma unroll
    for (int G = 0; G < NG; ++G) gin[G] = sg[G][lane];
    T V = T(0);
    const XiPtr<T> xi{xi_of<T>(a)};
    LV::template trie<T, false>(gin, xi, NoSink{}, dg, V);
    T dMp[NC];
    if constexpr (NW == 4) {
        switch (wave) {
            case 0: LV::template reverse_part<0>(M, dg, dMp); break;
            case 1: LV::template reverse_part<1>(M, dg, dMp); break;
            case 2: LV::template reverse_part<2>(M, dg, dMp); break;
            default: LV::template reverse_part<3>(M, dg, dMp); break;
        }
    } else {
        switch (wave) {
            case 0: LV::template reverse_part8<0>(M, dg, dMp); break;
            case 1: LV::template reverse_part8<1>(M, dg, dMp); break;
            case 2: LV::template reverse_part8<2>(M, dg, dMp); break;
            case 3: LV::template reverse_part8<3>(M, dg, dMp); break;
            case 4: LV::template reverse_part8<4>(M, dg, dMp); break;
            case 5: LV::template reverse_part8<5>(M, dg, dMp); break;
            case 6: LV::template reverse_part8<6>(M, dg, dMp); break;
            default: LV::template reverse_part8<7>(M, dg, dMp); break;
        }
    }
    __syncthreads();   // every reverse part has read M
    for (int w = 0; w < NW; ++w) {
        if (wave == w) {
#pragma unroll
            for (int k = 0; k < NC; ++k) sdm[k][lane] = w == 0 ? dMp[k] : sdm[k][lane] + dMp[k];
        }
        __syncthreads();
    }
    if (slot < a.n_atoms) {
        T *dout = static_cast<T *>(a.dmbuf);
        for (int k = wave; k < NC; k += NW) dout[(int64_t)k * a.n_atoms + slot] = sdm[k][lane];
        if (wave == 0) write_site<T>(a, slot, V);
    }
}

// rows of LDS scratch the contraction needs besides the moments
template <typename T, int L, int NW> constexpr int scratch_rows() {
    if constexpr (expanded_program<T, L>()) return Level<L>::NGRAPH;
    else return Fact<L, NW>::template rows<T>();
}

// The contraction of the 64 neighborhoods of block blk, the moments read
// through M.  sM: the moments' LDS, or NULL when they are in memory.
template <typename T, int L, bool WB, int NW, typename MA>
__device__ __forceinline__ void contract_body(const EfsArgs &a, int64_t blk, const MA &M, const T *s_xi, T (*scratch)[64],
                                              T (*sM)[64]) {
    static_assert(!WB || sizeof(T) == sizeof(double), "rows are FP64");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t slot = blk * 64 + lane;
    const bool live = slot < a.n_atoms;
    if constexpr (WB) constant_columns<L, NW>(a, slot, wave);
    if constexpr (expanded_program<T, L>()) {
        expanded_body<T, L, MA, NW>(a, blk, M, scratch, sM);
    } else {
        T *dout = static_cast<T *>(a.dmbuf) + slot;
        const auto out = [&](int k, T v) {
            if (live) dout[(int64_t)k * a.n_atoms] = v;
        };
        const auto site = [&](T V) { write_site<T>(a, slot, V); };
        const XiPtr<T> xi{s_xi};
        if constexpr (WB)
            fact_body<T, L, true, NW>(M, xi, ColSink{a.brow, a.ldn, a.n_types, (uint32_t)slot}, scratch, out, site);
        else
            fact_body<T, L, false, NW>(M, xi, NoSink{}, scratch, out, site);
    }
}

// wavefronts of the contraction when the moments come through memory: four
// clusters, or eight where a quarter of the graphs is more than a wavefront's
// registers hold (level 24: 60 components and 150 intermediates); there the
// fused launch comes with eight lanes only
template <int L> constexpr int contract_waves() { return Level<L>::NGRAPH <= 128 ? 4 : 8; }

template <typename T, int L, bool WB>
__global__ __launch_bounds__(64 * contract_waves<L>()) void efs_contract(const EfsArgs a) {
    using LV = Level<L>;
    constexpr int NW = contract_waves<L>();
    __shared__ T scratch[scratch_rows<T, L, NW>()][64];
    __shared__ T sdm[expanded_program<T, L>() ? LV::NC : 1][64];
    __shared__ T s_xi[xi_words<T, L>()];
    load_xi<T, L, 64 * NW>(a, s_xi);
    __syncthreads();
    const int64_t slot = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const int64_t sl = slot < a.n_atoms ? slot : 0;
    contract_body<T, L, WB, NW>(a, blockIdx.x, ColLoad<T>{static_cast<const T *>(a.mbuf) + sl, a.n_atoms}, s_xi, scratch, sdm);
}

// Kernels 1 and 2 in one launch, K = NW = four or eight lanes per
// neighborhood (the block's threads hold the same 64 neighborhoods in both
// phases): the reduce-scattered moments go to LDS instead of memory, and
// after one barrier the contraction reads them there.
template <typename T, int L, bool WB, int K>
__device__ __forceinline__ void moments_contract(const EfsArgs &a) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD;
    constexpr int NCP = (NC + K - 1) / K * K;
    __shared__ T c_s[NR * MAX_TYPES * MAX_TYPES * NPOLY];
    __shared__ T sM[NCP][64];
    __shared__ T scratch[scratch_rows<T, L, K>()][64];
    __shared__ T s_xi[xi_words<T, L>()];
    const int sub = threadIdx.x % K;
    const AtomCtx c = atom_ctx<K, 64 * K>(a);
    const PairVector first(a, c, sub);
    load_coefs<T, NR, 64 * K>(a, c_s);
    load_xi<T, L, 64 * K>(a, s_xi);
    __syncthreads();
    {
        T M[NCP];
        moments_scattered<T, L, K>(a, c, c_s, first, M);
        const int la = threadIdx.x / K;
#pragma unroll
        for (int i = 0; i < NCP / K; ++i) sM[sub * (NCP / K) + i][la] = M[i];
    }
    __syncthreads();
    contract_body<T, L, WB, K>(a, blockIdx.x, LdsCol<T>{&sM[0][threadIdx.x & 63]}, s_xi, scratch, sM);
}

template <typename T, int L, bool WB>
__global__ __launch_bounds__(256) void efs_moments_contract(const EfsArgs a) {
    moments_contract<T, L, WB, 4>(a);
}

template <typename T, int L, bool WB>
__global__ __launch_bounds__(512) void efs_moments_contract8(const EfsArgs a) {
    moments_contract<T, L, WB, 8>(a);
}

// Chebyshev values (and derivatives) at u for the radial basis (eq. 4)
template <typename T, bool DERIV>
__device__ inline void chebyshev(T u, T (&Tb)[NPOLY], T (&dT)[NPOLY]) {
    Tb[0] = T(1);
    Tb[1] = u;
    if (DERIV) {
        dT[0] = T(0);
        dT[1] = T(1);
    }
#pragma unroll
    for (int b = 2; b < NPOLY; ++b) {
        Tb[b] = fma(T(2) * u, Tb[b - 1], -Tb[b - 2]);
        if (DERIV) dT[b] = fma(T(2) * u, dT[b - 1], fma(T(2), Tb[b - 1], -dT[b - 2]));
    }
}

// dE/dM of the block's neighborhoods in LDS, [k][neighborhood in block]: the
// K lanes of a neighborhood read the same word (broadcast); in registers
// they would cost 2 NC VGPRs per lane.  TD: the type dV/dM was computed in
// (FP64 when the FP32 pair gradients of the mixed form follow an FP64
// contraction that also fed the rows).
// FP64: as the entries of the full symmetric tensors (component k over the
// number of index orders that name it), the form mu_tensors works with.
template <typename LV> constexpr int mu_first(int mu) {   // a mu's components are consecutive, by monomial index
    int k = 0;
    while (LV::comp_mu[k] != mu) ++k;
    return k;
}
template <typename LV> constexpr int mu_count(int mu) {   // 1, 4, 10 or 20
    int n = 0;
    for (int k = 0; k < LV::NC; ++k) n += LV::comp_mu[k] == mu ? 1 : 0;
    return n;
}
template <typename LV> constexpr int index_orders(int k) {
    constexpr int by_mono[20] = {1, 1, 1, 1, 1, 2, 2, 1, 2, 1, 1, 3, 3, 3, 6, 3, 1, 3, 3, 1};
    return by_mono[LV::comp_mono[k]];
}
// bit s: component k0 + s is named by `orders` orders (known at compile time, so that no table is read)
template <typename LV, int K> constexpr unsigned orders_mask(int k0, int orders) {
    unsigned m = 0;
    for (int s = 0; s < K && k0 + s < LV::NC; ++s) m |= index_orders<LV>(k0 + s) == orders ? 1u << s : 0u;
    return m;
}
// In two parts, so that the loads are in flight together and beside the
// block's other first loads (one after the other, each behind a branch for
// the last block's idle lanes, they took a memory latency each: 13 at level
// 16 with four lanes).  The caller's barrier follows the second part.
template <typename T, typename LV, int K> struct DmLoad {
    static constexpr int N = (LV::NC + K - 1) / K;
    T v[N];
    template <typename TD> __device__ inline DmLoad(const EfsArgs &a, const AtomCtx &c, int sub, TD) {
        const TD *din = static_cast<const TD *>(a.dmbuf) + (c.live ? c.slot : 0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = i * K + sub;
            v[i] = T(din[(int64_t)(k < LV::NC ? k : LV::NC - 1) * a.n_atoms]);
        }
    }
    template <int I> __device__ inline void store_one(bool live, int sub, T (&s_dm)[LV::NC][256 / K]) const {
        const int k = I * K + sub;
        T x = live ? v[I] : T(0);
        if constexpr (sizeof(T) == sizeof(double)) {
            constexpr unsigned m2 = orders_mask<LV, K>(I * K, 2), m3 = orders_mask<LV, K>(I * K, 3),
                               m6 = orders_mask<LV, K>(I * K, 6);
            T w = T(1);
            if (m2) w = (m2 >> sub) & 1 ? T(0.5) : w;
            if (m3) w = (m3 >> sub) & 1 ? T(1.0 / 3.0) : w;
            if (m6) w = (m6 >> sub) & 1 ? T(1.0 / 6.0) : w;
            x *= w;
        }
        if (k < LV::NC) s_dm[k][threadIdx.x / K] = x;
    }
    template <int... I>
    __device__ inline void store(bool live, int sub, T (&s_dm)[LV::NC][256 / K], std::integer_sequence<int, I...>) const {
        (store_one<I>(live, sub, s_dm), ...);
    }
    __device__ inline void store(bool live, int sub, T (&s_dm)[LV::NC][256 / K]) const {
        store(live, sub, s_dm, std::make_integer_sequence<int, N>{});
    }
};

// FP64 pairs: P_mu(r) and its gradient from the symmetric tensors S of dE/dM
// (LDS, [component][neighborhood la]).  With t_nu = S_nu . r^(nu - 1), a
// vector, P = S_0 + sum_nu t_nu . r and grad P = sum_nu nu t_nu: 42 operations
// for degrees 0 to 3 where monomials and their derivatives take 62, and the
// ten cubic monomials are not held.  v: x y z; q: xx yy zz 2xy 2xz 2yz.
template <typename LV, int MU, typename T, int W>
__device__ __forceinline__ void mu_tensors(const T (&S)[LV::NC][W], int la, const T (&v)[3], const T (&q)[6], T &P,
                                           T (&G)[3]) {
    constexpr int K0 = mu_first<LV>(MU), N = mu_count<LV>(MU);
    static_assert(N == 1 || N == 4 || N == 10 || N == 20, "a mu has the tensors of all degrees up to its largest");
    const auto s = [&](int m) { return S[K0 + m][la]; };
    P = s(0);
    G[0] = G[1] = G[2] = T(0);
    if constexpr (N > 1) {
        T U[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) U[d] = G[d] = s(1 + d);
        if constexpr (N > 4) {
            const T t[3] = {fma(s(6), v[2], fma(s(5), v[1], s(4) * v[0])), fma(s(8), v[2], fma(s(7), v[1], s(5) * v[0])),
                            fma(s(9), v[2], fma(s(8), v[1], s(6) * v[0]))};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                U[d] += t[d];
                G[d] = fma(T(2), t[d], G[d]);
            }
        }
        if constexpr (N > 10) {
            const T t[3] = {
                fma(s(14), q[5], fma(s(12), q[4], fma(s(11), q[3], fma(s(15), q[2], fma(s(13), q[1], s(10) * q[0]))))),
                fma(s(17), q[5], fma(s(14), q[4], fma(s(13), q[3], fma(s(18), q[2], fma(s(16), q[1], s(11) * q[0]))))),
                fma(s(18), q[5], fma(s(15), q[4], fma(s(14), q[3], fma(s(19), q[2], fma(s(17), q[1], s(12) * q[0])))))};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                U[d] += t[d];
                G[d] = fma(T(3), t[d], G[d]);
            }
        }
        P = fma(U[2], v[2], fma(U[1], v[1], fma(U[0], v[0], P)));
    }
}
template <typename T> __device__ inline void quadratics(T x, T y, T z, T (&q)[6]) {
    q[0] = x * x; q[1] = y * y; q[2] = z * z;
    q[3] = (x + x) * y; q[4] = (x + x) * z; q[5] = (y + y) * z;
}

// r = sqrt(d2) and 1 / r from one reciprocal square root (Goldschmidt's
// iteration, two residual corrections of r, one of 1/r): 11 operations for
// the 27 of a square root and a division.  d2: a squared distance whose square
// is a normal number, or 0 (two atoms in one place, which the neighbor build
// reports): then r is 0, so that the pair counts in the rows as it does in the
// moments, and 1 / r is not a number, so that its force is none either.
__device__ inline void root(double d2, double &r, double &rinv) {
    const double y = __builtin_amdgcn_rsq(d2);
    double g = d2 * y, h = 0.5 * y;
    double e = fma(-h, g, 0.5);
    h = fma(h, e, h);
    g = fma(g, e, g);
    g = fma(fma(-g, g, d2), h, g);
    r = fma(fma(-g, g, d2), h, g);
    h += h;
    rinv = fma(fma(-r, h, 1.0), h, h);
    r = d2 == 0.0 ? 0.0 : r;
}

// What an FP64 pair adds, mu by mu, so that one mu's P and gradient are live
// at a time: to the force (f_mu grad P_mu), to its radial part (f_mu' P_mu)
// and to the row's sums (ROWS; cut T_beta P_mu).
template <typename LV, bool ROWS, int MU, typename T, int W, int ND>
__device__ __forceinline__ void add_mu(const T (&S)[LV::NC][W], int la, const T (&v)[3], const T (&q)[6],
                                       const T (&f)[LV::NRAD], const T (&fp)[LV::NRAD], const T (&Tb)[NPOLY], T cut,
                                       T &radial, T (&g)[3], T (&dc)[ND]) {
    T P, G[3];
    mu_tensors<LV, MU>(S, la, v, q, P, G);
    radial = fma(fp[MU], P, radial);
    if constexpr (mu_count<LV>(MU) > 1)
#pragma unroll
        for (int d = 0; d < 3; ++d) g[d] = fma(f[MU], G[d], g[d]);
    if constexpr (ROWS) {
        const T cP = cut * P;
#pragma unroll
        for (int b = 0; b < NPOLY; ++b) dc[MU * NPOLY + b] = fma(Tb[b], cP, dc[MU * NPOLY + b]);
    }
}
template <typename LV, bool ROWS, typename T, int W, int ND, int... MU>
__device__ __forceinline__ void add_all_mu(const T (&S)[LV::NC][W], int la, const T (&v)[3], const T (&q)[6],
                                           const T (&f)[LV::NRAD], const T (&fp)[LV::NRAD], const T (&Tb)[NPOLY],
                                           T cut, T &radial, T (&g)[3], T (&dc)[ND], std::integer_sequence<int, MU...>) {
    (add_mu<LV, ROWS, MU>(S, la, v, q, f, fp, Tb, cut, radial, g, dc), ...);
}
// the row's sums alone
template <typename LV, typename T, int W, int ND, int... MU>
__device__ __forceinline__ void add_rows(const T (&S)[LV::NC][W], int la, const T (&v)[3], const T (&q)[6],
                                         const T (&Tb)[NPOLY], T cut, T (&dc)[ND], std::integer_sequence<int, MU...>) {
    const auto one = [&](auto mu) {
        constexpr int M = decltype(mu)::value;
        T P, G[3];
        mu_tensors<LV, M>(S, la, v, q, P, G);
        const T cP = cut * P;
#pragma unroll
        for (int b = 0; b < NPOLY; ++b) dc[M * NPOLY + b] = fma(Tb[b], cP, dc[M * NPOLY + b]);
    };
    (one(std::integral_constant<int, MU>{}), ...);
}

// ---- kernel 3: pair gradients and virial; LANES per atom ------------------
// g_ij = dE_i/dr_ij = sum_mu [f_mu'(r) P_mu r_ij / r + f_mu(r) grad P_mu] with
// P_mu = sum_nu dE/dM_{mu,nu} (r_ij)^{(x)nu} (the moment tensors contracted
// with dE/dM); virial S_ab = -sum_j g_a r_b per atom.  G (gradients wanted,
// decided at compile time so that the stores in the pair loop are
// unconditional): the force's own part F_i = sum_j g_ij (FP64, lanes summed
// in a fixed order) is written per atom, and each g_ij is stored at the slot
// of the reverse pair (j, i) -- the gather then subtracts, for every atom,
// the gradients its neighbors hold of it as one contiguous run of its own
// slots, instead of following the reverse index pair by pair.
//
// What bounds it: at large n the scattered stores of the pair gradients (level
// 8, 524,288 atoms with 58 neighbors: 395 us, 270 with the stores in list
// order, 174 without them), else latencies at two or three wavefronts a SIMD
// (the registers): hence everything a block needs first is loaded at once, and
// one mu's tensors are in registers at a time.  256,000 atoms with 34
// neighbors, level 16 with rows: 410 -> 373 us; 160 configurations at level
// 24: 128 -> 97 us; 19,652 atoms FP32, level 16: 20.0 -> 19.0 us.
//
// R > 0 (FP64 only): the rest of the b row in the same pass (kernel 4's
// work, Sec. II.C) -- R = 2 (FULL) the radial-coefficient part
// dV_i/dc_{mu, z_i, z_j, beta} = sum_j T_beta(r_ij) (R_cut - r_ij)^2 P_mu(r_ij)
// from the P_mu and Chebyshev values the gradient already has (32 more FMAs
// per pair at N_rad = 4); the constant columns come from the contraction.
// The same sums in the same order as kernel 4 at the same lanes, so the rows
// are the same bit for bit.  s_col: the kept-column map (R = 2).
template <typename T, int L, int K, bool G, typename TD = T, int R = 0>
__device__ inline void efs_forces_body(const EfsArgs &a, int64_t blk, T *c_s, T (&s_dm)[Level<L>::NC][256 / K],
                                       int32_t *s_col = nullptr) {
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD, NL = LV::NLIN;
    constexpr int ND = NR * NPOLY;   // radial-coefficient sums per species (a multiple of K)
    static_assert(R == 0 || sizeof(T) == sizeof(double), "rows are FP64");
    const int nt = a.n_types;
    const int sub = threadIdx.x % K;
    const AtomCtx c = atom_ctx<K>(a, blk);
    PairVector next(a, c, sub);
    const int32_t *rslot = G ? a.rev + c.atom * (int64_t)a.max_nbrs : nullptr;   // set only with gradients
    int nrv = G ? rslot[sub < a.max_nbrs ? sub : a.max_nbrs - 1] : 0;
    {
        const DmLoad<T, LV, K> dm(a, c, sub, TD(0));
        load_coefs<T, NR>(a, c_s);
        if constexpr (R == 2)
            for (int k = threadIdx.x; k < NR * nt * nt * NPOLY; k += 256) s_col[k] = a.colmap[nt + NL + k];
        dm.store(c.live, sub, s_dm);
        __syncthreads();
    }
    double *brow = R > 0 && c.live ? a.brow + c.slot : nullptr;   // entry k at brow[k * ldn]
    const int64_t ldn = a.ldn;
    const int la = threadIdx.x / K;
    const T rc = T(a.r_cut);
    const T xs = T(2.0 / (a.r_cut - a.r_min));
    const T x0 = T(-(a.r_min + a.r_cut) / (a.r_cut - a.r_min));
    T vir[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) vir[k] = T(0);
    double fo[3] = {0.0, 0.0, 0.0};   // sum_j g_ij of this lane's pairs
    T *gout = static_cast<T *>(a.gbuf);
    int gstart = 0;
    // The next pair vector is loaded while the current one is used (after a
    // species' last pair the next species' first); the loads are unconditional
    // (past the last pair it is read again, in bounds and unused), so that the
    // wait for them leaves the gradient stores of the pair before in flight.
    // The reverse slot of the next pair likewise (its store waits for it).
    const auto in_list = [&](int p) { return p < a.max_nbrs ? p : a.max_nbrs - 1; };
    for (int t = 0; t < nt; ++t) {
        const int tc = tcount(c, t);
        T dc[R == 2 ? ND : 1];
        if constexpr (R == 2)
#pragma unroll
            for (int k = 0; k < ND; ++k) dc[k] = T(0);
        const int pnext = in_list(gstart + tc + sub);   // the next species' first pair
        // waited for here, once, so that the loop head does not wait for
        // every outstanding access (the stores included) on each pair
        __asm__ volatile("" ::"v"(next.x), "v"(next.y), "v"(next.z), "v"(nrv));
        for (int q = sub; q < tc; q += K) {
            const int p = gstart + q;
            const T x = T(next.x), y = T(next.y), z = T(next.z);
            const int rv = nrv;
            const int pn = q + K < tc ? p + K : (t + 1 < nt ? pnext : p);
            next = PairVector(a, c, pn);
            if constexpr (G) nrv = rslot[pn];
            constexpr bool F64 = sizeof(T) == sizeof(double);
            const T d2 = efs::norm2(x, y, z);
            T r, rinv;
            if constexpr (F64) root(d2, r, rinv);
            else r = sqrt(d2);
            T g0 = T(0), g1 = T(0), g2 = T(0);
            if (r < rc) {
                T f[NR], fp[NR], Tb[NPOLY];
                const T d = rc - r;
                const T cut = d * d;
                {
                    const T u = fma(r, xs, x0);
                    const T dcut = T(-2) * d;
                    T dT[NPOLY];
                    chebyshev<T, true>(u, Tb, dT);
#pragma unroll
                    for (int mu = 0; mu < NR; ++mu) {
                        const CoefRow<T> cm = coef_row(c_s, mu, c.zi, t, nt);
                        T s = T(0), sp = T(0);
#pragma unroll
                        for (int b = 0; b < NPOLY; ++b) {
                            s = fma(cm[b], Tb[b], s);
                            sp = fma(cm[b], dT[b], sp);
                        }
                        f[mu] = s * cut;
                        fp[mu] = fma(sp * xs, cut, s * dcut);
                    }
                }
                T radial_part = T(0);
                if constexpr (F64) {
                    const T v[3] = {x, y, z};
                    T q[6], g[3] = {T(0), T(0), T(0)};
                    quadratics(x, y, z, q);
                    add_all_mu<LV, R == 2>(s_dm, la, v, q, f, fp, Tb, cut, radial_part, g, dc,
                                           std::make_integer_sequence<int, NR>{});
                    g0 = g[0];
                    g1 = g[1];
                    g2 = g[2];
                } else {
                    T mono[20];
                    efs::monomials(x, y, z, mono);
                    T P[NR], Gx[NR], Gy[NR], Gz[NR];
#pragma unroll
                    for (int mu = 0; mu < NR; ++mu) P[mu] = Gx[mu] = Gy[mu] = Gz[mu] = T(0);
#pragma unroll
                    for (int k = 0; k < NC; ++k) {
                        const int mu = LV::comp_mu[k];
                        const T dmk = s_dm[k][la];
                        P[mu] = fma(dmk, mono[LV::comp_mono[k]], P[mu]);
                        if (LV::comp_dmonox[k] >= 0)
                            Gx[mu] = fma(dmk * T(LV::comp_dfacx[k]), mono[LV::comp_dmonox[k] < 0 ? 0 : LV::comp_dmonox[k]], Gx[mu]);
                        if (LV::comp_dmonoy[k] >= 0)
                            Gy[mu] = fma(dmk * T(LV::comp_dfacy[k]), mono[LV::comp_dmonoy[k] < 0 ? 0 : LV::comp_dmonoy[k]], Gy[mu]);
                        if (LV::comp_dmonoz[k] >= 0)
                            Gz[mu] = fma(dmk * T(LV::comp_dfacz[k]), mono[LV::comp_dmonoz[k] < 0 ? 0 : LV::comp_dmonoz[k]], Gz[mu]);
                    }
                    rinv = T(1) / r;
#pragma unroll
                    for (int mu = 0; mu < NR; ++mu) {
                        radial_part = fma(fp[mu], P[mu], radial_part);
                        g0 = fma(f[mu], Gx[mu], g0);
                        g1 = fma(f[mu], Gy[mu], g1);
                        g2 = fma(f[mu], Gz[mu], g2);
                    }
                }
                radial_part *= rinv;
                g0 = fma(radial_part, x, g0);
                g1 = fma(radial_part, y, g1);
                g2 = fma(radial_part, z, g2);
                // S_ab = -sum g_a r_b
                vir[0] -= g0 * x; vir[1] -= g0 * y; vir[2] -= g0 * z;
                vir[3] -= g1 * x; vir[4] -= g1 * y; vir[5] -= g1 * z;
                vir[6] -= g2 * x; vir[7] -= g2 * y; vir[8] -= g2 * z;
            }
            if constexpr (G) {
                const int64_t s3 = (int64_t)rv * 3;   // the reverse pair's slot
                gout[s3] = g0;
                gout[s3 + 1] = g1;
                gout[s3 + 2] = g2;
                fo[0] += double(g0);
                fo[1] += double(g1);
                fo[2] += double(g2);
            }
        }
        if (sub >= tc && t + 1 < nt) {   // no pair of this species on this lane: what it holds is not the next one's first
            next = PairVector(a, c, pnext);
            if constexpr (G) nrv = rslot[pnext];
        }
        if constexpr (R == 2) {
            int col[ND / K];
#pragma unroll
            for (int i = 0; i < ND / K; ++i) {
                const int k = sub * (ND / K) + i, mu = k / NPOLY, b = k % NPOLY;
                col[i] = s_col[((mu * nt + c.zi) * nt + t) * NPOLY + b];
            }
            efs::reduce_scatter<T, ND, K>(dc, sub);
            if (brow) {
#pragma unroll
                for (int i = 0; i < ND / K; ++i)
                    if (col[i] >= 0) brow[col[i] * ldn] = dc[i];
            }
        }
        gstart += tc;
    }
    if constexpr (G) {
#pragma unroll
        for (int o = K / 2; o > 0; o >>= 1)
#pragma unroll
            for (int d = 0; d < 3; ++d) fo[d] += __shfl_xor(fo[d], o, 64);
        if (c.live && sub == 0)
#pragma unroll
            for (int d = 0; d < 3; ++d) a.F[c.atom * 3 + d] = fo[d];
    }
    constexpr int NV = (9 + K - 1) / K * K;
    T vp[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) vp[k] = k < 9 ? vir[k] : T(0);
    efs::reduce_scatter<T, NV, K>(vp, sub);
    if (c.live && a.virial) {
#pragma unroll
        for (int i = 0; i < NV / K; ++i) {
            const int k = sub * (NV / K) + i;
            if (k < 9) a.virial[c.atom * 9 + k] = double(vp[i]);
        }
    }
}

// ---- kernel 4: the rest of b_i (Sec. II.C); LANES per atom ----------------
// FULL grade mode: the radial-coefficient part
//   dV_i/dc_{mu, z_i, z_j, beta} = sum_{j of species z_j} T_beta(r_ij) (R_cut - r_ij)^2 P_mu(r_ij)
// (P_mu as in kernel 3).  The rest (B_alpha, one-hot, zeros) comes from
// kernel 2.
template <typename T, int L, int K>
__device__ inline void efs_rows_body(const EfsArgs &a, int64_t blk, T (&s_dm)[Level<L>::NC][256 / K],
                                     int32_t *s_col) {
    static_assert(sizeof(T) == sizeof(double), "rows are FP64");
    using LV = Level<L>;
    constexpr int NC = LV::NC, NR = LV::NRAD, NL = LV::NLIN;
    const int nt = a.n_types;
    const int sub = threadIdx.x % K;
    const AtomCtx c = atom_ctx<K>(a, blk);
    const bool full_rows = a.grade_mode == GRADE_FULL;
    PairVector next(a, c, sub);
    if (full_rows) {
        // the kept columns of the c part, once per block in LDS: read from
        // global memory beside the row stores, each would wait for the store
        // before it (the two may alias)
        const DmLoad<T, LV, K> dm(a, c, sub, T(0));
        for (int k = threadIdx.x; k < NR * nt * nt * NPOLY; k += 256) s_col[k] = a.colmap[nt + NL + k];
        dm.store(c.live, sub, s_dm);
        __syncthreads();
    }
    const int la = threadIdx.x / K;
    // entry k of this neighborhood's row: brow[k * ldn] (column-major rows)
    double *brow = c.live ? a.brow + c.slot : nullptr;
    const int64_t ldn = a.ldn;
    const T rc = T(a.r_cut);
    const T xs = T(2.0 / (a.r_cut - a.r_min));
    const T x0 = T(-(a.r_min + a.r_cut) / (a.r_cut - a.r_min));
    if (full_rows) {
        int gstart = 0;
        for (int t = 0; t < nt; ++t) {
            constexpr int ND = NR * NPOLY;   // a multiple of K (NPOLY = 8)
            T dc[ND];
#pragma unroll
            for (int k = 0; k < ND; ++k) dc[k] = T(0);
            const int tc = tcount(c, t);
            if (t > 0 && (sub >= tcount(c, t - 1))) next = PairVector(a, c, gstart + sub);
            for (int q = sub; q < tc; q += K) {
                const int p = gstart + q;
                const T x = T(next.x), y = T(next.y), z = T(next.z);
                next = PairVector(a, c, q + K < tc ? p + K : (t + 1 < nt ? gstart + tc + sub : p));
                T r, rinv;
                root(efs::norm2(x, y, z), r, rinv);
                if (!(r < rc)) continue;
                const T u = fma(r, xs, x0);
                const T d = rc - r;
                const T cut = d * d;
                T Tb[NPOLY], dT[NPOLY];
                chebyshev<T, false>(u, Tb, dT);
                const T v[3] = {x, y, z};
                T qm[6];
                quadratics(x, y, z, qm);
                add_rows<LV>(s_dm, la, v, qm, Tb, cut, dc, std::make_integer_sequence<int, NR>{});
            }
            efs::reduce_scatter<T, ND, K>(dc, sub);
            if (brow) {
#pragma unroll
                for (int i = 0; i < ND / K; ++i) {
                    const int k = sub * (ND / K) + i, mu = k / NPOLY, b = k % NPOLY;
                    const int col = s_col[((mu * nt + c.zi) * nt + t) * NPOLY + b];
                    if (col >= 0) brow[col * ldn] = dc[i];
                }
            }
            gstart += tc;
        }
    }
}

// Kernels 3 and 4 in one launch: blocks [0, nblk) take kernel 3, blocks
// [nblk, 2 nblk) kernel 4 (when rows are wanted); both only read dE/dM.
// TF: arithmetic of the pair gradients; TD: type of dE/dM, and of the rows
// (rows exist only when TD is FP64: the FP64 form, or the mixed form whose
// contraction ran in FP64 because the grade needs FP64 rows).
// ROWS: with row blocks (a kernel of its own without: their registers would
// cost the gradients wavefronts).
template <typename TF, typename TD, int L, int K, bool ROWS>
__global__ __launch_bounds__(256) void efs_forces_rows(const EfsArgs a, int64_t nblk) {
    using LV = Level<L>;
    constexpr int NCF = LV::NRAD * MAX_TYPES * MAX_TYPES * NPOLY;
    constexpr size_t FBYTES = sizeof(TF) * (NCF + LV::NC * (256 / K));
    constexpr size_t RBYTES = sizeof(double) * LV::NC * (256 / K) + sizeof(int32_t) * NCF;
    static_assert(!ROWS || sizeof(TD) == sizeof(double), "rows are FP64");
    // one LDS area: a block takes either the gradient or the row part
    __shared__ __attribute__((aligned(16))) char smem[ROWS && RBYTES > FBYTES ? RBYTES : FBYTES];
    if (!ROWS || (int64_t)blockIdx.x < nblk) {
        TF *c_s = reinterpret_cast<TF *>(smem);
        auto &s_dm = *reinterpret_cast<TF (*)[LV::NC][256 / K]>(c_s + NCF);
        if (a.gbuf)
            efs_forces_body<TF, L, K, true, TD>(a, blockIdx.x, c_s, s_dm);
        else
            efs_forces_body<TF, L, K, false, TD>(a, blockIdx.x, c_s, s_dm);
        if (a.part) {   // uniform: the block's atoms are whole sum chunks (256 / K = 32, 64 or 128)
            constexpr int PER = 256 / K / SUM_CHUNK;
            static_assert(PER * SUM_CHUNK * K == 256, "chunks per block");
            for (int q = 0; q < PER; ++q) {
                const int64_t chunk = (int64_t)blockIdx.x * PER + q;
                __syncthreads();   // the block's virials are written; sp of the previous chunk is read
                if (chunk * SUM_CHUNK < a.n_atoms) chunk_partials(chunk, a.n_atoms, a.part_e, a.virial, a.part);
            }
        }
    } else if constexpr (ROWS) {
        auto &s_dm = *reinterpret_cast<double (*)[LV::NC][256 / K]>(smem);
        int32_t *s_col = reinterpret_cast<int32_t *>(smem + sizeof(double) * LV::NC * (256 / K));
        efs_rows_body<double, L, K>(a, (int64_t)blockIdx.x - nblk, s_dm, s_col);
    }
}

// FP64 form with forces and rows: kernels 3 and 4 in one pass over the pairs
// (R = 1 LINEAR, 2 FULL rows); no row blocks
template <typename T, int L, int K, int R>
__global__ __launch_bounds__(256) void efs_forces_fused(const EfsArgs a) {
    using LV = Level<L>;
    constexpr int NCF = LV::NRAD * MAX_TYPES * MAX_TYPES * NPOLY;
    __shared__ __attribute__((aligned(16))) char smem[sizeof(T) * (NCF + LV::NC * (256 / K)) + sizeof(int32_t) * NCF];
    T *c_s = reinterpret_cast<T *>(smem);
    auto &s_dm = *reinterpret_cast<T (*)[LV::NC][256 / K]>(c_s + NCF);
    int32_t *s_col = reinterpret_cast<int32_t *>(smem + sizeof(T) * (NCF + LV::NC * (256 / K)));
    efs_forces_body<T, L, K, true, T, R>(a, blockIdx.x, c_s, s_dm, s_col);
    if (a.part) {   // uniform: the block's atoms are whole sum chunks
        constexpr int PER = 256 / K / SUM_CHUNK;
        static_assert(PER * SUM_CHUNK * K == 256, "chunks per block");
        for (int q = 0; q < PER; ++q) {
            const int64_t chunk = (int64_t)blockIdx.x * PER + q;
            __syncthreads();
            if (chunk * SUM_CHUNK < a.n_atoms) chunk_partials(chunk, a.n_atoms, a.part_e, a.virial, a.part);
        }
    }
}

template <int L, typename T> int launch_mc_level_t(const EfsArgs &a);
template <int L, typename TF, typename TD> int launch_fr_level_t(const EfsArgs &a);

// instantiates the launchers of one level and one arithmetic type (each
// (level, type) pair is a translation unit of its own, generated at build
// time): the moments / contraction in TT (rows only when TT is FP64), the
// pair gradients in TT with dE/dM in TT, and for TT = float also with dE/dM
// in FP64 (the mixed form with FP64 rows)
#define MTP_EFS_MC_LEVEL_T(LEVEL, TT)                                                                    \
    /* moments and contraction, K lanes per neighborhood (K = 4, 8: one launch; K = 2: two) */         \
    template <typename T, int K, bool WB> static void launch_mc##LEVEL(const EfsArgs &a) {               \
        const unsigned grid = (unsigned)((a.n_atoms + 256 / K - 1) / (256 / K));                         \
        const unsigned grid1 = (unsigned)((a.n_atoms + 63) / 64);                                        \
        if constexpr (K == 4 && contract_waves<LEVEL>() == 4) {                                          \
            ProfScope ps("efs_moments", a.stream);                                                       \
            hipLaunchKernelGGL((efs_moments_contract<T, LEVEL, WB>), dim3(grid1), dim3(256), 0, a.stream, \
                               a);                                                                       \
        } else if constexpr (K == 8) {                                                                           \
            ProfScope ps("efs_moments", a.stream);                                                       \
            hipLaunchKernelGGL((efs_moments_contract8<T, LEVEL, WB>), dim3(grid1), dim3(512), 0,          \
                               a.stream, a);                                                             \
        } else {                                                                                         \
            {                                                                                            \
                ProfScope ps("efs_moments", a.stream);                                                   \
                hipLaunchKernelGGL((efs_moments<T, LEVEL, K>), dim3(grid), dim3(256), 0, a.stream, a);   \
            }                                                                                            \
            ProfScope ps("efs_contract", a.stream);                                                      \
            hipLaunchKernelGGL((efs_contract<T, LEVEL, WB>), dim3(grid1),                                \
                               dim3(64 * contract_waves<LEVEL>()), 0, a.stream, a);                      \
        }                                                                                                \
    }                                                                                                    \
    template <> int launch_mc_level_t<LEVEL, TT>(const EfsArgs &a) {                                     \
        if (a.n_atoms == 0) return 0;                                                                    \
        constexpr bool F64 = sizeof(TT) == sizeof(double);                                               \
        if (F64 && a.brow != nullptr) {                                                                  \
            switch (a.lanes_mc) {                                                                        \
                case 2: launch_mc##LEVEL<TT, 2, F64>(a); break;                                          \
                case 4: launch_mc##LEVEL<TT, 4, F64>(a); break;                                          \
                default: launch_mc##LEVEL<TT, 8, F64>(a); break;                                         \
            }                                                                                            \
        } else {                                                                                         \
            switch (a.lanes_mc) {                                                                        \
                case 2: launch_mc##LEVEL<TT, 2, false>(a); break;                                        \
                case 4: launch_mc##LEVEL<TT, 4, false>(a); break;                                        \
                default: launch_mc##LEVEL<TT, 8, false>(a); break;                                       \
            }                                                                                            \
        }                                                                                                \
        return (int)hipGetLastError();                                                                   \
    }

#define MTP_EFS_FR_LEVEL_T(LEVEL, TT)                                                                    \
    /* pair gradients and virial (+ the rest of the rows), K lanes per neighborhood */                   \
    template <typename TF, typename TD, int K> static void launch_fr##LEVEL(const EfsArgs &a) {          \
        const unsigned grid = (unsigned)((a.n_atoms + 256 / K - 1) / (256 / K));                         \
        const bool rows = sizeof(TD) == sizeof(double) && a.brow != nullptr;                             \
        ProfScope ps("efs_forces", a.stream);                                                            \
        if constexpr (sizeof(TF) == sizeof(double)) {                                                    \
            if (rows && a.gbuf) { /* FP64 with forces: rows in the same pass */                          \
                if (a.grade_mode == GRADE_FULL)                                                          \
                    hipLaunchKernelGGL((efs_forces_fused<TF, LEVEL, K, 2>), dim3(grid), dim3(256), 0,     \
                                       a.stream, a);                                                     \
                else                                                                                     \
                    hipLaunchKernelGGL((efs_forces_fused<TF, LEVEL, K, 1>), dim3(grid), dim3(256), 0,     \
                                       a.stream, a);                                                     \
                return;                                                                                  \
            }                                                                                            \
        }                                                                                                \
        if constexpr (sizeof(TD) == sizeof(double)) {                                                    \
            if (rows) {                                                                                  \
                hipLaunchKernelGGL((efs_forces_rows<TF, TD, LEVEL, K, true>), dim3(2 * grid), dim3(256),  \
                                   0, a.stream, a, (int64_t)grid);                                       \
                return;                                                                                  \
            }                                                                                            \
        }                                                                                                \
        hipLaunchKernelGGL((efs_forces_rows<TF, TD, LEVEL, K, false>), dim3(grid), dim3(256), 0,          \
                           a.stream, a, (int64_t)grid);                                                  \
    }                                                                                                    \
    template <typename TD> static int launch_fr_td##LEVEL(const EfsArgs &a) {                            \
        if (a.n_atoms == 0) return 0;                                                                    \
        switch (a.lanes) {                                                                               \
            case 2: launch_fr##LEVEL<TT, TD, 2>(a); break;                                               \
            case 4: launch_fr##LEVEL<TT, TD, 4>(a); break;                                               \
            default: launch_fr##LEVEL<TT, TD, 8>(a); break;                                              \
        }                                                                                                \
        return (int)hipGetLastError();                                                                   \
    }                                                                                                    \
    template <> int launch_fr_level_t<LEVEL, TT, TT>(const EfsArgs &a) { return launch_fr_td##LEVEL<TT>(a); } \
    MTP_EFS_HYBRID_##TT(LEVEL)

#define MTP_EFS_HYBRID_double(LEVEL)
#define MTP_EFS_HYBRID_float(LEVEL)                                                                      \
    template <> int launch_fr_level_t<LEVEL, float, double>(const EfsArgs &a) {                          \
        return launch_fr_td##LEVEL<double>(a);                                                           \
    }

}  // namespace mtp
