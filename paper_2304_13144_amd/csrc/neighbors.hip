// Cell-list neighbor build (neighborhoods of MLIP-3 paper Sec. II.A).
//
// Per configuration the cell is cut into n_k bins along each cell vector
// (n_k = floor(h_k / R_cut), h_k = height of the cell along axis k, coarsened
// so that a configuration never has more bins than atoms).  A bin is then at
// least R_cut high, and every neighbor of an atom lies within s_k =
// ceil(R_cut n_k / h_k) bins along axis k.  Periodic axes wrap bins and
// record the image shift; a bin visited twice through different wraps is a
// different image, so small cells (h_k < R_cut) come out right.
//
// Steps: geometry per configuration -> bin every atom (counting sort, then
// each bin sorted by atom index so the result is deterministic) -> the search:
// a block per bin tests the bin's atoms against the candidates of the 27 (or
// more) nearby bins, and places every pair in its list, grouped by neighbor
// species -> reverse-pair index for the atomic-free force gather.  Up to
// SMALL_ATOMS atoms everything before the search is one launch of one block.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.hpp"

namespace mtp {
namespace {

struct CfgGeo {
    double H[9], Hi[9];
    int n[3], s[3], pbc[3], pad;
    long long bin_off, nbins;
};

__device__ inline double height(const double *H, int k) {
    const double *u = H + 3 * ((k + 1) % 3), *v = H + 3 * ((k + 2) % 3), *w = H + 3 * k;
    double cx = u[1] * v[2] - u[2] * v[1], cy = u[2] * v[0] - u[0] * v[2], cz = u[0] * v[1] - u[1] * v[0];
    double vol = fabs(w[0] * cx + w[1] * cy + w[2] * cz);
    return vol / sqrt(cx * cx + cy * cy + cz * cz);
}

// Geometry of configuration c but for its bin offset; flags a degenerate cell
__device__ inline CfgGeo make_geo(int c, const int64_t *cfg_off, const double *cell, const uint8_t *pbc, double rc,
                                  int *flags) {
    CfgGeo g;
    for (int k = 0; k < 9; ++k) g.H[k] = cell[9 * c + k];
    const double *H = g.H;
    double a = H[0], b = H[1], cc = H[2], d = H[3], e = H[4], f = H[5], gg = H[6], h = H[7], kk = H[8];
    double det = a * (e * kk - f * h) - b * (d * kk - f * gg) + cc * (d * h - e * gg);
    if (!(fabs(det) > 1e-12)) {   // degenerate cell: flag it, keep every index in range
        atomicOr(&flags[3], 1);
        det = INFINITY;
    }
    g.Hi[0] = (e * kk - f * h) / det; g.Hi[1] = (cc * h - b * kk) / det; g.Hi[2] = (b * f - cc * e) / det;
    g.Hi[3] = (f * gg - d * kk) / det; g.Hi[4] = (a * kk - cc * gg) / det; g.Hi[5] = (cc * d - a * f) / det;
    g.Hi[6] = (d * h - e * gg) / det; g.Hi[7] = (b * gg - a * h) / det; g.Hi[8] = (a * e - b * d) / det;
    const long long natoms = cfg_off[c + 1] - cfg_off[c];
    double hk[3];
    for (int k = 0; k < 3; ++k) {
        hk[k] = height(H, k);
        g.pbc[k] = pbc ? (int)pbc[3 * c + k] : 1;
        int nk = (int)floor(hk[k] / rc);
        g.n[k] = nk < 1 ? 1 : (nk > 1024 ? 1024 : nk);
    }
    const long long cap = natoms > 1 ? natoms : 1;
    while ((long long)g.n[0] * g.n[1] * g.n[2] > cap) {
        // the first of the largest, picked without an index (the array stays in registers)
        const bool one = g.n[1] > g.n[0], two = g.n[2] > (one ? g.n[1] : g.n[0]);
        g.n[0] -= !one && !two;
        g.n[1] -= one && !two;
        g.n[2] -= two;
    }
    for (int k = 0; k < 3; ++k) {
        int s = (int)ceil(rc * g.n[k] / hk[k]);
        g.s[k] = s < 1 ? 1 : s;
    }
    g.pad = 0;
    g.bin_off = 0;
    g.nbins = (long long)g.n[0] * g.n[1] * g.n[2];
    return g;
}

// Exclusive scan of one value per thread over a block of 1024 threads (wave
// scans by shuffles, one LDS step across the 16 wavefronts); total: the sum.
constexpr int SCAN_T = 1024;
__device__ inline int32_t block_exclusive(int32_t v, int32_t *wsum, int32_t &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    __syncthreads();   // wsum of a call before is read
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < SCAN_T / 64; ++w) {
        before += w < wave ? wsum[w] : 0;
        total += wsum[w];
    }
    return before + inc - v;
}

// The configurations' geometry by one block, a thread per configuration; bin
// offsets are the running sum of the bin counts.  (One thread that walked all
// configurations took 1.7 us each.)
__device__ inline int32_t all_geometry(int n_cfg, const int64_t *cfg_off, const double *cell, const uint8_t *pbc, double rc,
                                       CfgGeo *geo, int *flags, int32_t *wsum) {
    if (threadIdx.x < 8) flags[threadIdx.x] = 0;
    __syncthreads();
    int32_t off = 0;
    for (int c0 = 0; c0 < n_cfg; c0 += SCAN_T) {
        const int c = c0 + threadIdx.x;
        CfgGeo g;
        if (c < n_cfg) g = make_geo(c, cfg_off, cell, pbc, rc, flags);
        int32_t tot;
        const int32_t ex = block_exclusive(c < n_cfg ? (int32_t)g.nbins : 0, wsum, tot);
        if (c < n_cfg) {
            g.bin_off = off + ex;
            geo[c] = g;
        }
        off += tot;
    }
    if (threadIdx.x == 0) flags[4] = off;   // bins in use (<= the host-side capacity n_atoms + n_cfg)
    return off;
}

// block 0: geometry and status words; the others clear the bin counters
__global__ __launch_bounds__(SCAN_T) void nbr_prepare(int n_cfg, const int64_t *cfg_off, const double *cell,
                                                      const uint8_t *pbc, double rc, CfgGeo *geo, int *flags,
                                                      int32_t *bin_count, int64_t bins) {
    __shared__ int32_t wsum[SCAN_T / 64];
    if (blockIdx.x == 0) {
        all_geometry(n_cfg, cfg_off, cell, pbc, rc, geo, flags, wsum);
        return;
    }
    for (int64_t i = (int64_t)(blockIdx.x - 1) * SCAN_T + threadIdx.x; i < bins; i += (int64_t)(gridDim.x - 1) * SCAN_T)
        bin_count[i] = 0;
}

// A position that is not finite (NaN, Inf) sets bit 16 of flags[3] and is
// binned at the origin of its cell (it then fails every distance test): the
// status check reports MTP_E_INVAL instead of an empty neighborhood.
struct Binned {
    int cfg, bin, w[3];
};
__device__ inline Binned bin_of(int64_t i, int n_cfg, const int64_t *cfg_off, double (&x)[3], const CfgGeo *geo,
                                int32_t *flags) {
    Binned B;
    // configuration of atom i: last c with cfg_off[c] <= i
    int lo = 0, hi = n_cfg - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) / 2;
        if (cfg_off[mid] <= i) lo = mid; else hi = mid - 1;
    }
    const CfgGeo &g = geo[lo];
    double y[3] = {x[0], x[1], x[2]};
    if (!(isfinite(y[0]) && isfinite(y[1]) && isfinite(y[2]))) {
        atomicOr(&flags[3], 16);
        y[0] = y[1] = y[2] = 0.0;
    }
    int b[3];
    for (int k = 0; k < 3; ++k) {
        double s = y[0] * g.Hi[k] + y[1] * g.Hi[3 + k] + y[2] * g.Hi[6 + k];
        if (g.pbc[k]) {
            double fw = floor(s);
            B.w[k] = (int)fw;
            s -= fw;
        } else {
            B.w[k] = 0;
        }
        int bk = (int)floor(s * g.n[k]);
        b[k] = bk < 0 ? 0 : (bk >= g.n[k] ? g.n[k] - 1 : bk);
    }
    B.cfg = lo;
    B.bin = (int)(g.bin_off + ((long long)b[2] * g.n[1] + b[1]) * g.n[0] + b[0]);
    return B;
}

// the atom's bin and, from the counter, a place in it (any order: sorted later)
__global__ void bin_kernel(int64_t n, int n_cfg, const int64_t *cfg_off, const double *pos, const CfgGeo *geo,
                           int32_t *atom_cfg, int32_t *atom_bin, int32_t *atom_wrap, int32_t *bin_count,
                           int32_t *atom_place, int32_t *flags) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double x[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
    const Binned B = bin_of(i, n_cfg, cfg_off, x, geo, flags);
    atom_cfg[i] = B.cfg;
#pragma unroll
    for (int k = 0; k < 3; ++k) atom_wrap[3 * i + k] = B.w[k];
    atom_bin[i] = B.bin;
    atom_place[i] = atomicAdd(&bin_count[B.bin], 1);
}

struct BinStart {
    const int32_t *loc;
    __device__ int32_t operator[](int64_t b) const { return loc[b]; }
};

// Room for every bin in use: a block scans its own 1024 counts and takes its
// part of the slots from the cursor flags[6].  Which part is a matter of
// order between blocks, and no list depends on it: a bin's slots are only
// ever reached through its start.  At 64,000 bins 4.8 us; one block's scan
// over all of them was a serial chain of 45 us.
__global__ __launch_bounds__(SCAN_T) void place_bins(const int32_t *count, int32_t *start, int32_t *flags) {
    __shared__ int32_t wsum[SCAN_T / 64];
    __shared__ int32_t base;
    const int64_t nbins = flags[4];
    for (int64_t b0 = (int64_t)blockIdx.x * SCAN_T; b0 < nbins; b0 += (int64_t)gridDim.x * SCAN_T) {
        const int64_t b = b0 + threadIdx.x;
        int32_t all;
        const int32_t ex = block_exclusive(b < nbins ? count[b] : 0, wsum, all);
        if (threadIdx.x == 0) base = atomicAdd(&flags[6], all);
        __syncthreads();
        if (b < nbins) start[b] = base + ex;
        __syncthreads();
    }
}

__global__ void fill_bins(int64_t n, const int32_t *atom_bin, const int32_t *atom_place, BinStart start,
                          int32_t *bin_atoms) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) bin_atoms[start[atom_bin[i]] + atom_place[i]] = (int32_t)i;
}

__device__ inline int pack_q(int x, int y, int z) { return (x + 512) | ((y + 512) << 10) | ((z + 512) << 20); }
// An atom's image number as it is packed: far ones (reported as too far from 255 on) end where the field still
// holds the sum with the wrap of any bin of a one-window search (at most 32: 64 bin offsets), which would otherwise
// carry into the next field or into the species above them.
__device__ inline int near_image(int w) { return w < -478 ? -478 : (w > 478 ? 478 : w); }

struct Stage {
    const double *pos;
    const int32_t *type, *atom_cfg, *atom_wrap;
    const CfgGeo *geo;
    int n_types;
    double *sx;     // [3 n] x_j - w_j.H
    int32_t *sw;    // [n] pack_q(-w_j) | species << 30 (0 where out of range: that is reported)
    int32_t *rank;  // [n] by atom: its place within its bin
};

// slot u of the bin order holds an atom at x, wrapped by w, of species t:
// wrapped position, packed -wrap and species
__device__ inline void stage_at(const Stage &S, int64_t u, const double (&x)[3], const int (&w)[3], int t,
                                const CfgGeo &g, bool &wide, bool &bad) {
#pragma unroll
    for (int k = 0; k < 3; ++k) S.sx[3 * u + k] = x[k] - (w[0] * g.H[k] + w[1] * g.H[3 + k] + w[2] * g.H[6 + k]);
    if (w[0] < -255 || w[0] > 255 || w[1] < -255 || w[1] > 255 || w[2] < -255 || w[2] > 255) wide = true;
    const bool out = t < 0 || t >= S.n_types;
    if (out) bad = true;   // reported as an error; 0 keeps later indexing in range
    S.sw[u] = pack_q(-near_image(w[0]), -near_image(w[1]), -near_image(w[2])) | (out ? 0 : t) << 30;
}
__device__ inline void stage_atom(const Stage &S, int64_t u, int64_t j, bool &wide, bool &bad) {
    const double x[3] = {S.pos[3 * j], S.pos[3 * j + 1], S.pos[3 * j + 2]};
    const int w[3] = {S.atom_wrap[3 * j], S.atom_wrap[3 * j + 1], S.atom_wrap[3 * j + 2]};
    stage_at(S, u, x, w, S.type[j], S.geo[S.atom_cfg[j]], wide, bad);
}

// The bin's atoms (in arbitrary order from the counters) are put in ascending
// index order, which makes every later step deterministic, and each is staged
// at its slot: ranks from all-pairs comparisons across G lanes for bins of up
// to G atoms, by one lane for larger ones.  lane: this lane's place in its group.
template <int G>
__device__ inline void sort_stage_bin(int32_t *a, int64_t start, int c, int lane, const Stage &S, bool &wide,
                                      bool &bad) {
    if (c <= G) {
        const int v = lane < c ? a[lane] : 0x7fffffff;
        int rank = 0;
        for (int k = 0; k < c; ++k) rank += __shfl(v, k, G) < v ? 1 : 0;
        if (lane < c) {
            a[rank] = v;
            S.rank[v] = rank;
            stage_atom(S, start + rank, v, wide, bad);
        }
    } else if (lane == 0) {
        for (int x = 1; x < c; ++x) {
            const int32_t v = a[x];
            int y = x - 1;
            while (y >= 0 && a[y] > v) {
                a[y + 1] = a[y];
                --y;
            }
            a[y + 1] = v;
        }
        for (int x = 0; x < c; ++x) {
            S.rank[a[x]] = x;
            stage_atom(S, start + x, a[x], wide, bad);
        }
    }
}

__device__ inline void report_stage(bool wide, bool bad, int lane, int32_t *flags) {
    const bool any_wide = __ballot(wide) != 0, any_bad = __ballot(bad) != 0;
    if (lane == 0 && (any_wide || any_bad)) atomicOr(&flags[3], (any_wide ? 2 : 0) | (any_bad ? 8 : 0));
}

// A wavefront takes four bins at a time, 16 lanes each; a bin of more than 16
// atoms makes its four go one after the other on all lanes.
__global__ __launch_bounds__(256) void sort_bins(int32_t *flags, BinStart start, const int32_t *count,
                                                 int32_t *bin_atoms, Stage S) {
    const int lane = threadIdx.x & 63;
    const int64_t nbins = flags[4];
    bool wide = false, bad = false;
    for (int64_t b = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 4; b < nbins; b += (int64_t)gridDim.x * 16) {
        const int64_t mine = b + (lane >> 4);
        const int c = mine < nbins ? count[mine] : 0;
        const int32_t sb = mine < nbins ? start[mine] : 0;
        if (__ballot(c > 16) == 0) {
            sort_stage_bin<16>(bin_atoms + sb, sb, c, lane & 15, S, wide, bad);
        } else {
            for (int q = 0; q < 4; ++q) {
                const int cq = __shfl(c, q * 16, 64);
                const int32_t sq = __shfl(sb, q * 16, 64);
                sort_stage_bin<64>(bin_atoms + sq, sq, cq, lane, S, wide, bad);
            }
        }
    }
    report_stage(wide, bad, lane, flags);
}

// Everything before the search in one block, for up to SMALL_ATOMS atoms in up
// to SMALL_CFGS configurations: the steps of the launches above, separated by
// barriers, with the geometry, the counters and the bins' atoms in LDS and
// each thread's atoms (two, four above 2,048) in its registers.  An atom's
// place in its bin is the number of lower indices among the bin's atoms.
// Launch-bound below the line: 6.2 us at 128 atoms and 7.0 at 864 against five
// launches of 4 to 5 us each; one compute unit's throughput and registers
// above it (42 us at 5,148 atoms, where the five take 19 us of kernels).  The
// whole build at 2,916 / 4,000 atoms: 26.5 / 30.8 us, in general launches
// 32.8 / 34.5.
constexpr int SMALL_ATOMS = 4096, SMALL_CFGS = 64;
template <int PER>
__global__ __launch_bounds__(SCAN_T) void bin_small(int n, int n_cfg, const int64_t *cfg_off, const double *cell,
                                                    const uint8_t *pbc, double rc, CfgGeo *geo_out, int32_t *flags,
                                                    int32_t *bin_count, int32_t *bin_start, int32_t *bin_atoms,
                                                    int32_t *atom_cfg, int32_t *atom_wrap, Stage S) {
    constexpr int MAX_ATOMS = PER * SCAN_T, SMALL_BINS = MAX_ATOMS + SMALL_CFGS;
    __shared__ CfgGeo geo[SMALL_CFGS];
    __shared__ int32_t cnt[SMALL_BINS], beg[SMALL_BINS], atoms[MAX_ATOMS];
    __shared__ int32_t wsum[SCAN_T / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    double x[PER][3];
    int t[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {   // in flight during the geometry
        const int i = tid + SCAN_T * q < n ? tid + SCAN_T * q : 0;
        x[q][0] = S.pos[3 * i];
        x[q][1] = S.pos[3 * i + 1];
        x[q][2] = S.pos[3 * i + 2];
        t[q] = S.type[i];
    }
    for (int b = tid; b < SMALL_BINS; b += SCAN_T) cnt[b] = 0;
    const int nbins = all_geometry(n_cfg, cfg_off, cell, pbc, rc, geo, flags, wsum);   // <= n + n_cfg <= SMALL_BINS
    __syncthreads();
    for (int k = tid; k < n_cfg * (int)(sizeof(CfgGeo) / 8); k += SCAN_T)
        reinterpret_cast<uint64_t *>(geo_out)[k] = reinterpret_cast<const uint64_t *>(geo)[k];
    Binned B[PER];
    int place[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = tid + SCAN_T * q;
        if (i < n) {
            B[q] = bin_of(i, n_cfg, cfg_off, x[q], geo, flags);
            place[q] = atomicAdd(&cnt[B[q].bin], 1);
            atom_cfg[i] = B[q].cfg;
#pragma unroll
            for (int k = 0; k < 3; ++k) atom_wrap[3 * i + k] = B[q].w[k];
        }
    }
    __syncthreads();
    int32_t carry = 0;
    for (int b0 = 0; b0 < nbins; b0 += SCAN_T) {
        const int b = b0 + tid, v = b < nbins ? cnt[b] : 0;
        int32_t all;
        const int32_t ex = carry + block_exclusive(v, wsum, all);
        if (b < nbins) {
            beg[b] = ex;
            bin_start[b] = ex;
            bin_count[b] = v;
        }
        carry += all;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (tid + SCAN_T * q < n) atoms[beg[B[q].bin] + place[q]] = tid + SCAN_T * q;
    __syncthreads();
    bool wide = false, bad = false;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = tid + SCAN_T * q;
        if (i < n) {
            const int s0 = beg[B[q].bin], c = cnt[B[q].bin];
            int r = 0;
            for (int k = 0; k < c; ++k) r += atoms[s0 + k] < i ? 1 : 0;
            S.rank[i] = r;
            bin_atoms[s0 + r] = i;
            stage_at(S, s0 + r, x[q], B[q].w, t[q], geo[B[q].cfg], wide, bad);
        }
    }
    report_stage(wide, bad, lane, flags);
}

__device__ inline int floordiv(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

// ---- pair search ------------------------------------------------------------
//
// One block of four wavefronts per bin (several blocks, each with its share of
// the atoms, where the system is too small to fill the chip).  The candidates
// of the bin (atoms of the surrounding bins, every periodic image that can be
// in range) are numbered by a wave-wide prefix sum over the bin offsets and
// staged in LDS, a window of PS_WIN at a time, each as y_j = x_j - w_j.H (atom
// j wrapped into the cell) and its bin offset, whose periodic wrap q gives the
// lattice vector q.H.  For an atom i of the bin r_ij = (y_j - y_i) + q.H,
// which is bitwise -r_ji (the opposite pair has offset -d and wrap -q), so the
// lists are exactly symmetric; the pair's shift is q - w_j + w_i.
//
// When the candidates fit one window (the usual case) a wavefront takes an
// atom at a time: a float32 sieve of all candidates whose margin is larger
// than its rounding (about 6 of 7 go), the survivors' numbers packed in LDS;
// then the float64 test of the 60 or so survivors, whose ballots per species
// give every pair its place in the list (grouped by species, candidate order
// inside a group, clamped to max_nbrs).  Otherwise each atom takes a counting
// sweep and a writing sweep over the windows.
//
// Bound by vector instructions (a float64 test of every candidate, bin
// arithmetic by integer division and shuffles where a lane read does: 420 per
// atom, 569 us at 524,288 BCC atoms with 58 neighbors; now 343 us, of which
// the 1 GB of lists take 200).  For few bins bound by the chain of loads
// instead: two or four blocks then share a bin, so that a wavefront has one or
// two atoms (128 atoms: 18 us in two launches -> 8.8 in one).
constexpr int PS_WIN = 512;
constexpr int PS_CC = PS_WIN / 64;

// lanes below this one whose bit of m is set
__device__ inline int rank_in(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ inline int field(int p, int k) { return ((p >> (10 * k)) & 1023) - 512; }

constexpr int NO_WRAP = 512 | 512 << 10 | 512 << 20;   // pack_q(0, 0, 0); x + pack_q(q) - NO_WRAP adds q to packed x
// the same where q may be of any size (cells far below the cut-off): the species above the fields is kept
__device__ inline int add_wrap(int sw, int q) {
    return (int)(((unsigned)sw & 0xc0000000u) | ((unsigned)(sw + (q - NO_WRAP)) & 0x3fffffffu));
}

// What the search needs of a bin's configuration, held while the bins are of
// the same one: division by n comes down to a product, and the lane's bin
// offset (of the group that starts at offset og) is not taken apart again.
struct Local {
    const CfgGeo *g;
    int cfg, n0, n1, n2, n_off, bin_off;
    double inv0, inv1;
    bool near;   // |offset| <= n on every axis: a wrap is -1, 0 or 1
};
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline Local local_of(const CfgGeo *geo, int cfg) {
    Local l;
    l.g = geo + cfg;
    l.cfg = cfg;
    l.n0 = uniform(l.g->n[0]), l.n1 = uniform(l.g->n[1]), l.n2 = uniform(l.g->n[2]);
    const int s0 = uniform(l.g->s[0]), s1 = uniform(l.g->s[1]), s2 = uniform(l.g->s[2]);
    l.n_off = (2 * s0 + 1) * (2 * s1 + 1) * (2 * s2 + 1);
    l.bin_off = uniform((int)l.g->bin_off);
    l.inv0 = 1.0 / l.n0;
    l.inv1 = 1.0 / l.n1;
    l.near = s0 <= l.n0 && s1 <= l.n1 && s2 <= l.n2;
    return l;
}
// floor(v / n) for 0 <= v < 2^30: (v + 1/2) / n is at least 1 / (2 n) from a whole number
__device__ inline int quotient(int v, double inv) { return (int)((v + 0.5) * inv); }

struct Offset {   // a bin offset
    int x, y, z;
};
__device__ inline Offset offset_of(const Local &l, int o) {
    const int s0 = l.g->s[0], s1 = l.g->s[1], ox = 2 * s0 + 1, oy = 2 * s1 + 1;
    return {o % ox - s0, (o / ox) % oy - s1, o / (ox * oy) - l.g->s[2]};
}

struct Around {   // the bins around one bin: this lane's bin offset
    int start, count, qp, excl, total;
};

__device__ inline int wrap_axis(int u, int n, bool periodic, bool near, int &q, bool &ok) {
    q = 0;
    if (!periodic) {
        ok = ok && u >= 0 && u < n;
        return u;
    }
    q = near ? (u >= n ? 1 : 0) - (u < 0 ? 1 : 0) : floordiv(u, n);
    return u - q * n;
}

__device__ inline Around bins_near(const Local &l, int bx, int by, int bz, const Offset &d, bool used,
                                   const BinStart &bin_start, const int32_t *bin_count) {
    Around A{0, 0, NO_WRAP, 0, 0};
    bool ok = used;
    int qx, qy, qz;
    const int ux = wrap_axis(bx + d.x, l.n0, l.g->pbc[0], l.near, qx, ok);
    const int uy = wrap_axis(by + d.y, l.n1, l.g->pbc[1], l.near, qy, ok);
    const int uz = wrap_axis(bz + d.z, l.n2, l.g->pbc[2], l.near, qz, ok);
    if (ok) {
        const int nb = l.bin_off + (uz * l.n1 + uy) * l.n0 + ux;
        A.start = bin_start[nb];
        A.count = bin_count[nb];
        A.qp = pack_q(qx, qy, qz);
    }
    return A;
}

// Sum over the lanes up to this one
__device__ inline int inclusive(int v) {
#define MTP_DPP_ADD(ctrl, rows) v += __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xf, false)
    MTP_DPP_ADD(0x111, 0xf);   // row_shr 1, 2, 4, 8
    MTP_DPP_ADD(0x112, 0xf);
    MTP_DPP_ADD(0x114, 0xf);
    MTP_DPP_ADD(0x118, 0xf);
    MTP_DPP_ADD(0x142, 0xa);   // last lane of a row of 16 to the next row
    MTP_DPP_ADD(0x143, 0xc);   // lane 31 to the upper half
#undef MTP_DPP_ADD
    return v;
}

__device__ inline Around number_candidates(Around A) {
    const int inc = inclusive(A.count);
    A.excl = inc - A.count;
    A.total = __builtin_amdgcn_readlane(inc, 63);
    return A;
}

struct Staged {
    const double *sx;
    const int32_t *sw, *bin_atoms;
};

struct Window {   // LDS: one window of candidates
    double x[PS_WIN], y[PS_WIN], z[PS_WIN];
    int jq[PS_WIN];   // j if the bin offset has no periodic wrap, else ~j (never equal to an atom index)
    int qt[PS_WIN];   // pack_q(q - w_j) | species << 30
    unsigned short lp[PS_WIN];   // bin offset (lane of the offset group) | place in its bin << 6
    double qh[64][3];            // q.H per bin offset of the group
};

// The same candidates in float32, r_j = y_j + q.H - origin; far: one of them
// has a coordinate past REACH cut-off radii.
constexpr float REACH = 64.0f;
struct Sieve {
    float x[PS_WIN], y[PS_WIN], z[PS_WIN];
    int far;
};

// Candidates w0 .. w0 + PS_WIN - 1 of an offset group into LDS; every wave
// of the block holds the same offset group A, and each stages its quarter.
__device__ inline void stage_window(Window &W, const Around &A, int w0, int wave, int lane, const CfgGeo &g,
                                    const Staged &S) {
    if (wave == 0) {
        const int qx = field(A.qp, 0), qy = field(A.qp, 1), qz = field(A.qp, 2);
#pragma unroll
        for (int k = 0; k < 3; ++k) W.qh[lane][k] = qx * g.H[k] + qy * g.H[3 + k] + qz * g.H[6 + k];
    }
    for (int e = wave * 64 + lane, e0 = wave * 64; e0 < PS_WIN && w0 + e0 < A.total; e += 256, e0 += 256) {
        const int v = w0 + e;
        int L = 0;   // last lane whose bins start at or before candidate v
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
            const int ex = __shfl(A.excl, L + step, 64);
            if (ex <= v) L += step;
        }
        const int st = __shfl(A.start, L, 64), pe = __shfl(A.excl, L, 64), q = __shfl(A.qp, L, 64);
        if (v < A.total && e < PS_WIN) {
            const int64_t u = st + v - pe;
            W.x[e] = S.sx[3 * u];
            W.y[e] = S.sx[3 * u + 1];
            W.z[e] = S.sx[3 * u + 2];
            const int j = S.bin_atoms[u];
            W.jq[e] = q == NO_WRAP ? j : ~j;
            W.qt[e] = add_wrap(S.sw[u], q);
            W.lp[e] = (unsigned short)(L | (int)(v - pe) << 6);
        }
    }
}

// The whole of a one-window offset group (n_off <= 64), with its float32 copy;
// the last 128 slots in use are filled up with candidates at infinity.  F.far:
// cleared, and all threads have seen it.
__device__ inline void stage_sieve(Window &W, Sieve &F, const Around &A, int n_off, int wave, int lane,
                                   const CfgGeo &g, const double (&o)[3], float reach, const Staged &S) {
    const bool wraps = __ballot(A.qp != NO_WRAP) != 0;   // wave-uniform; usually not
    if (wave == 0) {
        double q[3] = {0.0, 0.0, 0.0};
        if (wraps) {
            const int qx = field(A.qp, 0), qy = field(A.qp, 1), qz = field(A.qp, 2);
#pragma unroll
            for (int k = 0; k < 3; ++k) q[k] = qx * g.H[k] + qy * g.H[3 + k] + qz * g.H[6 + k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) W.qh[lane][k] = q[k];
    }
    const int top = n_off > 32 ? 32 : 16, from = A.start - A.excl;
    const int n = (A.total + 127) & ~127;
    for (int e = wave * 64 + lane; e - lane < n; e += 256) {
        int L = 0;   // last lane whose bins start at or before candidate e
        for (int step = top; step >= 1; step >>= 1) {
            const int ex = __shfl(A.excl, L + step, 64);
            if (ex <= e) L += step;
        }
        const int64_t u = __shfl(from, L, 64) + e;
        const int pe = __shfl(A.excl, L, 64);
        int q = NO_WRAP;
        if (wraps) q = __shfl(A.qp, L, 64);
        float f[3] = {INFINITY, 0.0f, 0.0f};
        if (e < A.total) {
            const double y[3] = {S.sx[3 * u], S.sx[3 * u + 1], S.sx[3 * u + 2]};
            const int j = S.bin_atoms[u];
            const int qt = S.sw[u] + (q - NO_WRAP);
            double d[3] = {y[0] - o[0], y[1] - o[1], y[2] - o[2]};
            if (wraps) {
                const int qx = field(q, 0), qy = field(q, 1), qz = field(q, 2);
#pragma unroll
                for (int k = 0; k < 3; ++k) d[k] += qx * g.H[k] + qy * g.H[3 + k] + qz * g.H[6 + k];
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) f[k] = (float)d[k];
            if (!(fmaxf(fmaxf(fabsf(f[0]), fabsf(f[1])), fabsf(f[2])) <= reach)) F.far = 1;
            W.x[e] = y[0];
            W.y[e] = y[1];
            W.z[e] = y[2];
            W.jq[e] = q == NO_WRAP ? j : ~j;
            W.qt[e] = qt;
            W.lp[e] = (unsigned short)(L | (e - pe) << 6);
        }
        F.x[e] = f[0];
        F.y[e] = f[1];
        F.z[e] = f[2];
    }
}

struct Centre {   // the atom whose neighborhood is built (wave-uniform)
    int i, wrap;   // wrap: added to a packed q - w_j gives the packed shift
    double y0, y1, y2;   // y_i
};

struct Flags {
    bool overlap = false, wide = false;
};

// Tests the window's candidates against atom i: bit cc of the returned mask
// is candidate 64 cc + lane; *tb gets its species (2 bits each).  The test
// 0 < |r| < R_cut is made as r.r <= d2max, d2max being the largest double
// whose (correctly rounded) square root is below R_cut: the same decision as
// sqrt(r.r) < R_cut, without the square root.
__device__ inline unsigned test_window(const Window &W, int n, const Centre &c, int lane, double d2max, unsigned &tb,
                                       Flags &fl) {
    unsigned in = 0;
    tb = 0;
    for (int cc = 0; cc * 64 < n; ++cc) {
        const int e = cc * 64 + lane;
        if (e >= n) break;
        const int o = W.lp[e] & 63;
        const double r0 = (W.x[e] - c.y0) + W.qh[o][0], r1 = (W.y[e] - c.y1) + W.qh[o][1],
                     r2 = (W.z[e] - c.y2) + W.qh[o][2];
        const double d2 = r0 * r0 + r1 * r1 + r2 * r2;
        bool ok = d2 <= d2max;
        ok = ok && W.jq[e] != c.i;   // the atom itself (same image)
        if (ok) {
            in |= 1u << cc;
            tb |= ((unsigned)W.qt[e] >> 30) << (2 * cc);
            if (d2 < 1e-12) fl.overlap = true;
        }
    }
    return in;
}

// One-window form, first part: the candidates that the float32 test does not
// rule out (NaN does not), their numbers into perm in ascending order; returns
// how many.  Two chunks of 64 at a time, so that their reads overlap.
__device__ inline int sieve(const Sieve &F, int n, float c0, float c1, float c2, float lim, int lane, short *perm) {
    int ns = 0;
    for (int e0 = 0; e0 < n; e0 += 128) {
        const int e = e0 + lane;
        const float a0 = F.x[e] - c0, a1 = F.y[e] - c1, a2 = F.z[e] - c2;
        const float b0 = F.x[e + 64] - c0, b1 = F.y[e + 64] - c1, b2 = F.z[e + 64] - c2;
        const bool ina = !(a0 * a0 + a1 * a1 + a2 * a2 > lim), inb = !(b0 * b0 + b1 * b1 + b2 * b2 > lim);
        const unsigned long long ma = __ballot(ina), mb = __ballot(inb);
        const int na = __popcll(ma);
        if (ina) perm[ns + rank_in(ma)] = (short)e;
        if (inb) perm[ns + na + rank_in(mb)] = (short)(e + 64);
        ns += na + __popcll(mb);
    }
    return ns;
}

// Second part: survivor a of the sieve, tested in float64.
struct Hit {
    double r0, r1, r2;
    int e, lp, jq, qt;
    unsigned t;
    bool ok;
};
template <int NT>
__device__ inline Hit test_survivor(const Window &W, const short *perm, int n, int a, int ns, const Centre &c,
                                    double d2max, Flags &fl) {
    Hit h;
    h.ok = false;
    h.t = 0;
    if (a < ns) {
        h.e = perm[a];
        h.lp = W.lp[h.e];
        h.jq = W.jq[h.e];
        h.qt = W.qt[h.e];
        const int o = h.lp & 63;
        h.r0 = (W.x[h.e] - c.y0) + W.qh[o][0];
        h.r1 = (W.y[h.e] - c.y1) + W.qh[o][1];
        h.r2 = (W.z[h.e] - c.y2) + W.qh[o][2];
        const double d2 = h.r0 * h.r0 + h.r1 * h.r1 + h.r2 * h.r2;
        if (NT > 1) h.t = (unsigned)h.qt >> 30;
        h.ok = d2 <= d2max && h.jq != c.i && h.e < n;   // not the atom itself (same image), no filler
        if (h.ok && d2 < 1e-12) fl.overlap = true;
    }
    return h;
}

// Where the pairs of one atom with the atoms of one nearby bin (offset o) of
// one species stand in its list: they are a run in ascending place within that
// bin, so a mask of the places that are present (the first RUN_BITS) and the
// list offset of the first give every pair's slot without a look at the list.
constexpr int RUN_BITS = 23;
constexpr int RUN_OFFS = 32;   // bin offsets with an entry: all 27 but in cells below the cut-off
constexpr unsigned RUN_NONE = 0xffffffffu;   // no entry (9 bits hold any one-window list offset)
template <int NT>
struct Runs {
    unsigned mask[NT][64], first[NT][64];
};

// per-species counts of the accepted candidates (wave-uniform)
__device__ inline void count_window(unsigned in, unsigned tb, int n, int n_types, int (&cnt)[MAX_TYPES]) {
    for (int cc = 0; cc * 64 < n; ++cc) {
        const bool a = (in >> cc) & 1u;
        const int t = (tb >> (2 * cc)) & 3;
#pragma unroll
        for (int s = 0; s < MAX_TYPES; ++s)
            if (s < n_types) cnt[s] += __popcll(__ballot(a && t == s));
    }
}

// Places the accepted candidates: list offset base[t] + run[t] + rank among
// this window's pairs of species t; kept if the rank is below cap[t] - run[t].
// perm_e / perm_k receive (candidate, list offset) for the kept ones; returns
// how many.  run[] advances by the window's counts.
__device__ inline int place_window(unsigned in, unsigned tb, int n, int n_types, int lane, int (&run)[MAX_TYPES],
                                   const int (&cap)[MAX_TYPES], const int (&base)[MAX_TYPES], short *perm_e,
                                   int *perm_k) {
    const unsigned long long below = (1ull << lane) - 1ull;
    int kept = 0;
    for (int cc = 0; cc * 64 < n; ++cc) {
        const bool a = (in >> cc) & 1u;
        const int t = (tb >> (2 * cc)) & 3;
#pragma unroll
        for (int s = 0; s < MAX_TYPES; ++s) {
            if (s >= n_types) continue;
            const unsigned long long mk = __ballot(a && t == s);
            const int k = run[s] + __popcll(mk & below);
            const bool keep = a && t == s && k < cap[s];
            const unsigned long long km = __ballot(keep);
            if (keep) {
                const int slot = kept + __popcll(km & below);
                perm_e[slot] = (short)(cc * 64 + lane);
                perm_k[slot] = base[s] + k;
            }
            kept += __popcll(km);
            run[s] += __popcll(mk);
        }
    }
    return kept;
}

// The packed shift p = 512 + shift per axis as the list's word without its top
// byte; flags a shift that int8 does not hold.
__device__ inline int shift_word(unsigned p, Flags &fl) {
    const unsigned a = (p & 1023) - 385u, b = ((p >> 10) & 1023) - 385u, c = ((p >> 20) & 1023) - 385u;
    if (max(max(a, b), c) > 254u) fl.wide = true;
    return (int)((p & 0xff) | ((p >> 2) & 0xff00) | ((p >> 4) & 0xff0000));
}

// consecutive lanes write consecutive kept pairs (multi-window path: the
// opposite bin offset is not recorded, 0xff)
__device__ inline void write_kept(const Window &W, const short *perm_e, const int *perm_k, int kept,
                                  const Centre &c, int lane, int max_nbrs, double *rout, int32_t *jout,
                                  int32_t *shout, Flags &fl) {
    for (int a = lane; a < kept; a += 64) {
        const int e = perm_e[a];
        const int64_t slot = (int64_t)c.i * max_nbrs + perm_k[a];
        const int qt = W.qt[e], jq = W.jq[e];
        const int o = W.lp[e] & 63;
        rout[3 * slot] = (W.x[e] - c.y0) + W.qh[o][0];
        rout[3 * slot + 1] = (W.y[e] - c.y1) + W.qh[o][1];
        rout[3 * slot + 2] = (W.z[e] - c.y2) + W.qh[o][2];
        jout[slot] = jq >= 0 ? jq : ~jq;
        shout[slot] = shift_word((unsigned)(qt + c.wrap), fl) | (0xff << 24);
    }
}

// pair h at list offset k of the rows rout, jout, shout
__device__ inline void write_hit(const Hit &h, const Centre &c, int k, int n_off, double *rout, int32_t *jout,
                                 int32_t *shout, Flags &fl) {
    rout[3 * k] = h.r0;
    rout[3 * k + 1] = h.r1;
    rout[3 * k + 2] = h.r2;
    jout[k] = h.jq ^ (h.jq >> 31);
    // top byte: the opposite bin offset (from j's bin to i's), for the reverse-pair index
    shout[k] = shift_word((unsigned)(h.qt + c.wrap), fl) | ((n_off - 1 - (h.lp & 63)) << 24);
}

// Per-species slots of one neighborhood: counts -> capacities (clamped to
// max_nbrs in species order) and list offsets.
__device__ inline void list_layout(const int (&cnt)[MAX_TYPES], int n_types, int max_nbrs, int (&cap)[MAX_TYPES],
                                   int (&base)[MAX_TYPES], int &tot) {
    int off = 0;
    tot = 0;
#pragma unroll
    for (int t = 0; t < MAX_TYPES; ++t) {
        cap[t] = 0;
        base[t] = off;
        if (t < n_types) {
            tot += cnt[t];
            const int room = max_nbrs - off;
            cap[t] = cnt[t] < room ? cnt[t] : room;
            off += cap[t];
        }
    }
}

__device__ inline int from_lane(int v, int k) { return __shfl(v, k, 64); }

__device__ inline double lane_value(double v, int k) {   // k: wave-uniform
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, k), hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double((long long)hi << 32 | (unsigned)lo);
}

__device__ inline void wave_sync() {   // LDS writes of this wavefront before, reads after
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One-window neighborhood of atom c by one wavefront; returns the number of
// neighbors, kept or not.  perm, T: this wavefront's own.
template <int NT>
__device__ inline int neighborhood(const Window &W, const Sieve &F, int n, int n_off, const Centre &c,
                                   const double (&o)[3], double d2max, float lim, int max_nbrs, int lane, short *perm,
                                   Runs<NT> &T, double *rout, int32_t *jout, int32_t *shout, int32_t *tcnt,
                                   unsigned *runs_out, Flags &fl) {
    const int ns = sieve(F, n, (float)(c.y0 - o[0]), (float)(c.y1 - o[1]), (float)(c.y2 - o[2]), lim, lane, perm);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        T.mask[t][lane] = 0;
        T.first[t][lane] = 511;
    }
    wave_sync();
    int cnt[MAX_TYPES] = {0, 0, 0, 0}, cap[MAX_TYPES], base[MAX_TYPES], run[MAX_TYPES] = {0, 0, 0, 0}, tot;
    if constexpr (NT > 1) {
        for (int a0 = 0; a0 < ns; a0 += 64) {
            const Hit h = test_survivor<NT>(W, perm, n, a0 + lane, ns, c, d2max, fl);
#pragma unroll
            for (int s = 0; s < NT; ++s) cnt[s] += __popcll(__ballot(h.ok && h.t == (unsigned)s));
        }
        list_layout(cnt, NT, max_nbrs, cap, base, tot);
    } else {
        cap[0] = max_nbrs;
        base[0] = 0;
    }
    const int64_t row = (int64_t)c.i * max_nbrs;   // wave-uniform
    for (int a0 = 0; a0 < ns; a0 += 64) {
        const Hit h = test_survivor<NT>(W, perm, n, a0 + lane, ns, c, d2max, fl);
        int k = 0;
        bool keep = false;
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            const bool of_s = NT == 1 ? h.ok : h.ok && h.t == (unsigned)s;
            const unsigned long long m = __ballot(of_s);
            if (of_s) {
                k = run[s] + rank_in(m);
                keep = k < cap[s];
                k += base[s];
            }
            run[s] += __popcll(m);
        }
        if (keep) {
            const int at = h.t * 64 + (h.lp & 63), place = h.lp >> 6;
            if (place < RUN_BITS) atomicOr(&T.mask[0][at], 1u << place);
            atomicMin(&T.first[0][at], (unsigned)k);
            write_hit(h, c, k, n_off, rout + 3 * row, jout + row, shout + row, fl);
        }
    }
    if constexpr (NT == 1) {
        tot = run[0];
        cap[0] = tot < max_nbrs ? tot : max_nbrs;
    }
    wave_sync();
    if (lane < n_off && lane < RUN_OFFS) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
            runs_out[((int64_t)c.i * NT + t) * RUN_OFFS + lane] = T.first[t][lane] << RUN_BITS | T.mask[t][lane];
    }
    wave_sync();
    if (lane < NT) {
        int v = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t == lane) v = cap[t];
        tcnt[(int64_t)c.i * NT + lane] = v;
    }
    return tot;
}

// A barrier that orders LDS only: a list's stores stay in flight across it
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// NARROW: every bin whose candidates fit one window; the others are appended
// to wide_list (count in flags[5]) for the WIDE launch.  BOTH: one launch for
// all bins (more registers and LDS a block: for systems that don't fill the
// chip).  2^share blocks share a bin's atoms.
constexpr int SEARCH_GRID = 8192;   // blocks at most (a bin each or several: the host knows only a bound on the bins)
enum SearchMode { NARROW, WIDE, BOTH };
template <SearchMode MODE, int NT>
__global__ __launch_bounds__(256, MODE == NARROW ? 5 : 2)
void pair_search(int n_cfg, int share, int max_nbrs, double rc, double d2max, const CfgGeo *geo, Staged S,
                 BinStart bin_start, const int32_t *bin_count, int32_t *tcnt, double *rout, int32_t *jout,
                 int32_t *shout, int32_t *flags, int32_t *wide_list, unsigned *runs_out) {
    __shared__ Window W;
    __shared__ Sieve F;
    __shared__ Runs<NT> runs[4];
    __shared__ short perm_e[4][PS_WIN];
    __shared__ int perm_k[4][MODE == NARROW ? 1 : PS_WIN];
    __shared__ int s_max[4], s_bits[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int n_types = NT;   // species loops unroll to the actual count
    const int items = (MODE == WIDE ? flags[5] : flags[4]) << share;
    Flags fl;
    int max_tot = 0;
    Local l;
    Offset d;
    l.cfg = -1;
    // What a bin needs before its candidates are known is loaded one bin ahead.
    struct Ahead {
        int bin, count, start, bx, by, bz;
        Local l;
        Around A;
    };
    auto ahead = [&](int it) {
        Ahead P;
        P.bin = MODE == WIDE ? uniform(wide_list[it >> share]) : it >> share;
        P.count = bin_count[P.bin];
        P.start = bin_start[P.bin];
        int lo = 0, hi = n_cfg - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (geo[mid].bin_off <= P.bin) lo = mid; else hi = mid - 1;
        }
        lo = uniform(lo);
        if (lo != l.cfg) {
            l = local_of(geo, lo);
            d = offset_of(l, lane);
        }
        P.l = l;
        const int local = P.bin - l.bin_off, col = quotient(local, l.inv0);
        P.bx = local - col * l.n0;
        P.bz = quotient(col, l.inv1);
        P.by = col - P.bz * l.n1;
        P.A = bins_near(l, P.bx, P.by, P.bz, d, lane < l.n_off, bin_start, bin_count);
        return P;
    };
    Ahead next;
    if ((int)blockIdx.x < items) next = ahead(blockIdx.x);
    for (int it = blockIdx.x; it < items; it += gridDim.x) {   // block-uniform
        const Ahead P = next;
        if (it + (int)gridDim.x < items) next = ahead(it + gridDim.x);
        const int part = it & ((1 << share) - 1);
        const int first = part * 4 + wave, step = 4 << share;   // this wavefront's atoms of the bin
        const int my_cnt = uniform(P.count), my_start = uniform(P.start), n_off = P.l.n_off;
        if (my_cnt == 0) continue;
        const CfgGeo &g = *P.l.g;
        const Around A0 = number_candidates(P.A);
        const bool one_window = n_off <= 64 && A0.total <= PS_WIN;
        if (MODE == NARROW && !one_window) {
            if (threadIdx.x == 0 && part == 0) wide_list[atomicAdd(&flags[5], 1)] = P.bin;
            continue;
        }
        const double o[3] = {S.sx[3 * (int64_t)my_start], S.sx[3 * (int64_t)my_start + 1],
                             S.sx[3 * (int64_t)my_start + 2]};
        float lim = 0.0f;
        if (MODE != WIDE && one_window) {
            lds_barrier();   // the previous bin's window is no longer read
            if (threadIdx.x == 0) F.far = 0;
            lds_barrier();
            stage_sieve(W, F, A0, n_off, wave, lane, g, o, REACH * (float)rc, S);
            lds_barrier();
            // A float32 coordinate is off by 2^-24 of its size, so a difference of two by at most 2^-22 REACH rc
            // per axis (its own rounding included); the second factor covers the roundings of the square and of
            // this line.  Coordinates past REACH rc (atoms far outside an open cell): nothing is ruled out.
            const float r = (float)rc * (1.0f + 0x1p-21f * REACH);
            lim = F.far ? INFINITY : r * r * (1.0f + 0x1p-20f);
        }
        for (int a_base = 0; a_base < my_cnt; a_base += 64 * step) {   // block-uniform
            // lane k holds atom a_base + first + step k of the bin
            const int ak = a_base + first + step * lane;
            int hold_i = 0, hold_w = NO_WRAP;
            double hold_x = 0.0, hold_y = 0.0, hold_z = 0.0;
            if (ak < my_cnt) {
                const int64_t u = (int64_t)my_start + ak;
                hold_i = S.bin_atoms[u];
                hold_w = S.sw[u];
                hold_x = S.sx[3 * u];
                hold_y = S.sx[3 * u + 1];
                hold_z = S.sx[3 * u + 2];
            }
            const int left = my_cnt - a_base - first > 0 ? (my_cnt - a_base - first + step - 1) / step : 0;
            const int na = left < 64 ? left : 64;
            auto centre = [&](int k) {   // k: wave-uniform
                Centre c;
                c.i = __builtin_amdgcn_readlane(hold_i, k);
                c.wrap = NO_WRAP - (__builtin_amdgcn_readlane(hold_w, k) & 0x3fffffff);
                c.y0 = lane_value(hold_x, k);
                c.y1 = lane_value(hold_y, k);
                c.y2 = lane_value(hold_z, k);
                return c;
            };
            if (MODE != WIDE && one_window) {
                for (int k = 0; k < na; ++k) {
                    const int tot = neighborhood<NT>(W, F, A0.total, n_off, centre(k), o, d2max, lim, max_nbrs, lane,
                                                     perm_e[wave], runs[wave], rout, jout, shout, tcnt, runs_out, fl);
                    max_tot = tot > max_tot ? tot : max_tot;
                }
            }
            if (MODE != NARROW && !(MODE == BOTH && one_window)) {
                // per held atom (lane k): counts, then capacities / offsets / placed so far
                int hc[MAX_TYPES] = {0, 0, 0, 0}, hcap[MAX_TYPES] = {0, 0, 0, 0}, hbase[MAX_TYPES] = {0, 0, 0, 0},
                    hrun[MAX_TYPES] = {0, 0, 0, 0};
                for (int pass = 0; pass < 2; ++pass) {
                    if (pass == 1) {
                        int tot;
                        list_layout(hc, n_types, max_nbrs, hcap, hbase, tot);
                        if (lane < na) max_tot = tot > max_tot ? tot : max_tot;
                    }
                    for (int og = 0; og < n_off; og += 64) {
                        const Around A = number_candidates(bins_near(P.l, P.bx, P.by, P.bz, offset_of(P.l, og + lane),
                                                                     og + lane < n_off, bin_start, bin_count));
                        for (int w0 = 0; w0 < A.total; w0 += PS_WIN) {
                            const int n = A.total - w0 < PS_WIN ? A.total - w0 : PS_WIN;
                            __syncthreads();
                            stage_window(W, A, w0, wave, lane, g, S);
                            __syncthreads();
                            for (int k = 0; k < na; ++k) {
                                const Centre c = centre(k);
                                unsigned tb;
                                const unsigned in = test_window(W, n, c, lane, d2max, tb, fl);
                                int cnt[MAX_TYPES] = {0, 0, 0, 0};
                                count_window(in, tb, n, n_types, cnt);
                                if (pass == 0) {
                                    if (lane == k)
                                        for (int t = 0; t < MAX_TYPES; ++t) hc[t] += cnt[t];
                                    continue;
                                }
                                int run[MAX_TYPES], cap[MAX_TYPES], base[MAX_TYPES];
#pragma unroll
                                for (int t = 0; t < MAX_TYPES; ++t) {
                                    run[t] = from_lane(hrun[t], k);
                                    cap[t] = from_lane(hcap[t], k);
                                    base[t] = from_lane(hbase[t], k);
                                }
                                const int kept = place_window(in, tb, n, n_types, lane, run, cap, base, perm_e[wave],
                                                              perm_k[wave]);
                                wave_sync();
                                write_kept(W, perm_e[wave], perm_k[wave], kept, c, lane, max_nbrs, rout, jout, shout,
                                           fl);
                                wave_sync();
                                if (lane == k)
                                    for (int t = 0; t < MAX_TYPES; ++t) hrun[t] = run[t];
                            }
                        }
                    }
                }
                if (lane < na)
                    for (int t = 0; t < n_types; ++t) tcnt[(int64_t)hold_i * n_types + t] = hcap[t];
                for (int k = 0; k < na; ++k)   // no runs for these atoms
                    for (int t = 0; t < n_types; ++t)
                        if (lane < RUN_OFFS)
                            runs_out[((int64_t)from_lane(hold_i, k) * n_types + t) * RUN_OFFS + lane] = RUN_NONE;
            }
        }
    }
    // Status words: one atomic per block (same-address atomics from every
    // atom would serialise in L2), and only when the stored value changes.
    const int bits = (__ballot(fl.overlap) ? 1 : 0) | (__ballot(fl.wide) ? 2 : 0);
    int wmax = max_tot;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) wmax = max(wmax, __shfl_xor(wmax, d, 64));
    if (lane == 0) {
        s_max[wave] = wmax;
        s_bits[wave] = bits;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int mt = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
        const int b = s_bits[0] | s_bits[1] | s_bits[2] | s_bits[3];
        if (mt > max_nbrs) atomicOr(&flags[0], 1);
        if (mt > __hip_atomic_load(&flags[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&flags[1], mt);
        if (b & 1) atomicOr(&flags[2], 1);
        if (b & 2) atomicOr(&flags[3], 2);
    }
}

__device__ inline int sx8(int v) { return (int)(signed char)(v & 0xff); }

// One thread per list slot: the slot of (j, i, -n) in j's list.  The top byte
// of a slot's shift word is the index of the opposite bin offset (from j's bin
// to i's); j's run for that offset and i's species holds a bit per place of
// i's bin, so the slot is the run's first plus the bits below i's.  Where the
// place has no bit the run is scanned, and without a run the whole group.
// Bound by the lists' traffic and the scattered word per pair: 143 us at
// 524,288 atoms with 58 neighbors each (a look into the list for every pair:
// 387 us).
__global__ __launch_bounds__(256) void reverse_pairs(unsigned slots, int n_types, int max_nbrs, const int32_t *type,
                                                     const int32_t *tcnt, const int32_t *jl, const int32_t *sh,
                                                     const int32_t *rank, const unsigned *runs, int32_t *rev,
                                                     int32_t *flags) {
    const unsigned slot = blockIdx.x * 256u + threadIdx.x;   // blocks of 256 threads
    if (slot >= slots) return;
    const unsigned i = slot / (unsigned)max_nbrs;
    const int p = (int)(slot - i * (unsigned)max_nbrs);
    // Each level of dependent loads is issued at once: the slot's own entry,
    // i's species, place and counts (the entry is stale and unused past the count) ...
    const int j = jl[slot];
    const int s = sh[slot];
    const int zi = type[i], place = rank[i];
    int tot = 0;
#pragma unroll
    for (int t = 0; t < MAX_TYPES; ++t) tot += t < n_types ? tcnt[(int64_t)i * n_types + t] : 0;
    __asm__ volatile("" ::"v"(j), "v"(s), "v"(zi), "v"(place));   // keeps the loads above the branch
    if (p >= tot) return;
    if (zi < 0 || zi >= n_types) {   // flagged when the atom was staged; the slot names itself (in bounds)
        rev[slot] = (int)slot;
        return;
    }
    const int orev = (s >> 24) & 0xff;
    // ... then j's run
    const unsigned w = orev < RUN_OFFS ? runs[((int64_t)j * n_types + zi) * RUN_OFFS + orev] : RUN_NONE;
    int found = -1;
    if (w != RUN_NONE && place < RUN_BITS) {
        if ((w >> place) & 1u)
            found = j * max_nbrs + (int)(w >> RUN_BITS) + __popc(w & ((1u << place) - 1u));
    } else {
        const int want = ((-sx8(s)) & 0xff) | ((-sx8(s >> 8)) & 0xff) << 8 | ((-sx8(s >> 16)) & 0xff) << 16;
        int start = 0, end = 0;
#pragma unroll
        for (int t = 0; t < MAX_TYPES; ++t) {
            const int c = t < n_types ? tcnt[(int64_t)j * n_types + t] : 0;
            if (t < zi) start += c;
            if (t <= zi) end += c;
        }
        if (w != RUN_NONE) start = (int)(w >> RUN_BITS);
        for (int q = start; q < end; ++q) {
            const int s2 = j * max_nbrs + q;
            const int j2 = jl[s2], sh2 = sh[s2];
            if ((j2 == (int)i) & ((sh2 & 0xffffff) == want)) {
                found = s2;
                break;
            }
        }
    }
    if (found < 0) {
        atomicOr(&flags[3], 4);
        found = (int)slot;   // keeps the gather in bounds; the status call reports the fault
    }
    rev[slot] = found;
}

}  // namespace

void build_neighbors(const mtp_model *m, const mtp_system *s, int max_nbrs, mtp_nbrs *nb, hipStream_t st) {
    const int64_t n = s->n_atoms;
    const int nt = m->n_types;
    nb->device = m->device;
    nb->n_atoms = n;
    nb->n_cfg = s->n_cfg;
    nb->max_nbrs = max_nbrs;
    nb->n_types = nt;
    nb->r_cut = m->r_cut;
    const int64_t P = n * max_nbrs;
    nb->r.ensure(sizeof(double) * 3 * (P > 0 ? P : 1));
    nb->j.ensure(sizeof(int32_t) * (P > 0 ? P : 1));
    nb->shift.ensure(sizeof(int32_t) * (P > 0 ? P : 1));
    nb->rev.ensure(sizeof(int32_t) * (P > 0 ? P : 1));
    nb->tcnt.ensure(sizeof(int32_t) * (n * nt > 0 ? n * nt : 1));
    nb->atom_cfg.ensure(sizeof(int32_t) * (n > 0 ? n : 1));
    nb->atom_bin.ensure(sizeof(int32_t) * (n > 0 ? n : 1));
    nb->atom_wrap.ensure(sizeof(int32_t) * 3 * (n > 0 ? n : 1));
    nb->cfg_geo.ensure(sizeof(CfgGeo) * s->n_cfg);
    const int64_t bins = n + s->n_cfg;   // upper bound: each configuration has at most max(1, N_c) bins
    nb->bin_count.ensure(sizeof(int32_t) * bins);
    nb->bin_start.ensure(sizeof(int32_t) * bins);
    nb->bin_cursor.ensure(sizeof(int32_t) * bins);
    nb->bin_atoms.ensure(sizeof(int32_t) * (n > 0 ? n : 1));
    nb->stage_x.ensure(sizeof(double) * 3 * (n > 0 ? n : 1));
    nb->stage_w.ensure(sizeof(int32_t) * (n > 0 ? n : 1));
    nb->rank.ensure(sizeof(int32_t) * (n > 0 ? n : 1));
    nb->runs.ensure(sizeof(uint32_t) * RUN_OFFS * (n * nt > 0 ? n * nt : 1));
    nb->flags.ensure(sizeof(StepRead));
    nb->bins_cap = bins;
    auto *geo = nb->cfg_geo.as<CfgGeo>();
    int32_t *flags = nb->flags.as<int32_t>();
    const int TB = 256;
    const BinStart bstart{nb->bin_start.as<int32_t>()};
    Stage sg{s->pos, s->type, nb->atom_cfg.as<int32_t>(), nb->atom_wrap.as<int32_t>(), geo, nt,
             nb->stage_x.as<double>(), nb->stage_w.as<int32_t>(), nb->rank.as<int32_t>()};
    const bool small = n > 0 && n <= SMALL_ATOMS && s->n_cfg <= SMALL_CFGS;
    if (small) {
        hipLaunchKernelGGL((n <= 2 * SCAN_T ? bin_small<2> : bin_small<4>), dim3(1), dim3(SCAN_T), 0, st, (int)n,
                           s->n_cfg, s->cfg_off, s->cell, s->pbc, m->r_cut, geo, flags, nb->bin_count.as<int32_t>(),
                           nb->bin_start.as<int32_t>(), nb->bin_atoms.as<int32_t>(), nb->atom_cfg.as<int32_t>(),
                           nb->atom_wrap.as<int32_t>(), sg);
    } else {
        hipLaunchKernelGGL(nbr_prepare, dim3((unsigned)std::min<int64_t>((bins + SCAN_T - 1) / SCAN_T, 512) + 1),
                           dim3(SCAN_T), 0, st, s->n_cfg, s->cfg_off, s->cell, s->pbc, m->r_cut, geo, flags,
                           nb->bin_count.as<int32_t>(), bins);
        if (n == 0) return;
        const dim3 ga((unsigned)((n + TB - 1) / TB));
        // bin_cursor: the atoms' places in their bins, then the list of bins for the WIDE launch
        hipLaunchKernelGGL(bin_kernel, ga, dim3(TB), 0, st, n, s->n_cfg, s->cfg_off, s->pos, geo,
                           nb->atom_cfg.as<int32_t>(), nb->atom_bin.as<int32_t>(), nb->atom_wrap.as<int32_t>(),
                           nb->bin_count.as<int32_t>(), nb->bin_cursor.as<int32_t>(), flags);
        hipLaunchKernelGGL(place_bins, dim3((unsigned)std::min<int64_t>((bins + SCAN_T - 1) / SCAN_T, 256)),
                           dim3(SCAN_T), 0, st, nb->bin_count.as<int32_t>(), nb->bin_start.as<int32_t>(), flags);
        hipLaunchKernelGGL(fill_bins, ga, dim3(TB), 0, st, n, nb->atom_bin.as<int32_t>(),
                           nb->bin_cursor.as<int32_t>(), bstart, nb->bin_atoms.as<int32_t>());
        hipLaunchKernelGGL(sort_bins, dim3((unsigned)std::min<int64_t>((bins + 15) / 16, 2048)), dim3(TB), 0, st, flags,
                           bstart, nb->bin_count.as<int32_t>(), nb->bin_atoms.as<int32_t>(), sg);
    }
    // largest d2 with sqrt(d2) < R_cut (IEEE square roots are correctly rounded, host and device alike)
    double d2max = m->r_cut * m->r_cut;
    while (d2max > 0 && std::sqrt(d2max) >= m->r_cut) d2max = std::nextafter(d2max, 0.0);
    while (std::sqrt(std::nextafter(d2max, INFINITY)) < m->r_cut) d2max = std::nextafter(d2max, INFINITY);
    const Staged staged{nb->stage_x.as<double>(), nb->stage_w.as<int32_t>(), nb->bin_atoms.as<int32_t>()};
    // 2^share blocks per bin.  More of them shorten the chain of atoms a wavefront takes and repeat the staging: of
    // the whole build, one / two / four blocks a bin measured 23.3 / 20.5 / 19.7 us at 864 FCC atoms, 22.6 / 20.3 /
    // 22.4 at 1,372, 26.5 / 29.5 / 34.2 at 2,916 and 51.4 / 58.8 / 72.5 at 16,384.
    const int share = n < 1000 ? 2 : (n <= 2048 ? 1 : 0);
    auto search = [&](auto mode, auto ntc) {
        constexpr SearchMode MODE = decltype(mode)::value;
        constexpr int NTC = decltype(ntc)::value;
        const dim3 grid((unsigned)std::min<int64_t>(bins << share, MODE == WIDE ? 512 : SEARCH_GRID));
        hipLaunchKernelGGL((pair_search<MODE, NTC>), grid, dim3(TB), 0, st, s->n_cfg, share, max_nbrs, m->r_cut, d2max,
                           geo, staged, bstart, nb->bin_count.as<int32_t>(), nb->tcnt.as<int32_t>(),
                           nb->r.as<double>(), nb->j.as<int32_t>(), nb->shift.as<int32_t>(), flags,
                           nb->bin_cursor.as<int32_t>(), nb->runs.as<uint32_t>());
    };
    auto all = [&](auto ntc) {
        if (small) {
            search(std::integral_constant<SearchMode, BOTH>{}, ntc);
        } else {
            search(std::integral_constant<SearchMode, NARROW>{}, ntc);
            search(std::integral_constant<SearchMode, WIDE>{}, ntc);
        }
    };
    switch (nt) {
        case 1: all(std::integral_constant<int, 1>{}); break;
        case 2: all(std::integral_constant<int, 2>{}); break;
        case 3: all(std::integral_constant<int, 3>{}); break;
        default: all(std::integral_constant<int, 4>{}); break;
    }
    hipLaunchKernelGGL(reverse_pairs, dim3((unsigned)((P + TB - 1) / TB)), dim3(TB), 0, st, (unsigned)P, nt, max_nbrs,
                       s->type, nb->tcnt.as<int32_t>(), nb->j.as<int32_t>(), nb->shift.as<int32_t>(),
                       nb->rank.as<int32_t>(), nb->runs.as<uint32_t>(), nb->rev.as<int32_t>(), flags);
    MTP_HIP(hipGetLastError());
}

}  // namespace mtp
