// Separable non-local projectors on MFMA.
//
//   V_nl psi_n = sum_a sum_i p_i^a E_i^a D[a][i][n],
//   D[a][i][n] = h^3 sum_{r in S_a} p_i^a(r) psi_n(r)
//
// The non-local pseudopotential and its projectors are the electron-ion
// term named in section "Magnetic response and gauge invariance in
// real-space grids"; the separable form with four real projectors per atom
// is this library's reading.  Both halves are dense contractions:
//
//   gather : D^T[cols x 4] = psi^T[cols x |S_a|] * P[|S_a| x 4]
//   scatter: Y[|S_a| x cols] += P[|S_a| x 4] * F[4 x cols],  F = c E D
//
// where cols are the 2*nst real columns (re and im of each orbital).  The
// batch is orbital-major: real column col of point r sits at
// (col / 2) * ldo + 2 r + col % 2 (in reals), ldo = 2 ldp.
// The gather runs on v_mfma_{f64,f32}_16x16x4: 16 columns on M, 4 support
// points on K and the 4 projectors on N (zero-padded to 16).  The scatter is
// bound by the points it reads and writes (8 multiply-adds per 32 bytes), so
// it goes by point, not by atom: every point of the union of all supports is
// updated once, by one thread per orbital, with all the projectors that cover
// it.
//
// MFMA operand layout (lane l of a wave of 64), measured on gfx950:
//   A[i][k] in lane i + 16k, B[k][j] in lane j + 16k;
//   accumulator element r of lane l holds D[i][j] with j = l % 16 and
//     i = l/16 + 4r      for v_mfma_f64_16x16x4f64,
//     i = 4(l/16) + r    for v_mfma_f32_16x16x4f32.
//
// Supports are padded to a multiple of 16 entries with p = 0 (and a valid
// index); padded entries contribute zero and are never written.  Atoms are
// coloured so that supports of one colour are disjoint; a point covered by
// several atoms adds them in colour order, so the result is deterministic
// without atomics.
#include "kb_gather.h"
#include "rsg_internal.h"

#include <algorithm>

namespace rsg {

namespace {

constexpr int SP = 32;                   // lanes of a scatter workgroup along the points
constexpr int SJ = kScatterPoints / SP;  // points per lane
constexpr int SA = 16;                   // atoms staged at a time

// F[i] = c E_i D[a][i][n], D = h3 * (the chunk partials added in order).
template <class Tc>
__device__ __forceinline__ typename cpx<Tc>::type scatter_coef(const Tc *__restrict__ D, const Tc *__restrict__ P,
                                                               int nchunk, Tc h3, const double *__restrict__ E,
                                                               int64_t ncols, int a, int i, int64_t n, double cre,
                                                               double cim) {
    const int64_t row = (int64_t)a * 4 + i;
    using C2 = typename cpx<Tc>::type;
    const C2 d = kb_value<Tc>(D, P, nchunk, h3, ncols, row, n);
    const double e = E[row];
    C2 f;
    f.x = (Tc)(e * (cre * (double)d.x - cim * (double)d.y));
    f.y = (Tc)(e * (cre * (double)d.y + cim * (double)d.x));
    return f;
}

// Scatter for one item (up to kScatterPoints points of one owner atom) and 8
// orbitals: lane e of SP takes points e and e + SP, so that a half-wave covers
// runs of consecutive points of one orbital.  The coefficients of the item's
// atoms (its owner and the atoms that overlap it there) are staged in LDS, SA
// atoms at a time.
// Latency bound on small systems, where the chunk sums and every colour were
// launches of their own: 2.0 + 2 x 3.6 us -> 5.0 us (2 atoms x 5 orbitals, 17 k
// points), 4.8 + 2 x 4.9 -> 7.2 us (3 x 7, 500 k); 16 atoms x 64 orbitals
// (3.05 M) 4.8 + 2 x 29.7 -> 49.9 us; 48 spheres 129 -> 110 us a stage.
// 32 points an item: 6.6, 65 and 142 us; 128: 9.2, 49 and 104 us.
template <class Tout, class Tc>
__device__ __forceinline__ void scatter_points(Tout *__restrict__ out, int64_t ldo, int64_t ncols, const int4 it, int ct,
                                               const ScatterTab &tab, const Tc *__restrict__ p,
                                               const double *__restrict__ E, const Tc *__restrict__ D,
                                               const Tc *__restrict__ P, int nchunk, Tc h3, double cre, double cim,
                                               const double *__restrict__ mask,
                                               typename cpx<Tc>::type (*sF)[4][8]) {
    using O2 = typename cpx<Tout>::type;
    const int t = threadIdx.x, o = t / SP;
    const int64_t nst = ncols >> 1, n = (int64_t)ct * 8 + o;
    O2 *const col = reinterpret_cast<O2 *>(out + (n < nst ? n : 0) * ldo);
    // the owner's contribution (the first of every point) is requested with
    // the point itself; only points under several atoms walk a list
    int pt[SJ], c[SJ], c1[SJ];
    Tc po[SJ][4];
#pragma unroll
    for (int j = 0; j < SJ; ++j) {
        const int e = (t & (SP - 1)) + j * SP;
        const bool live = e < it.y && n < nst;
        const int k = live ? it.x + e : it.x;
        pt[j] = live ? tab.pt[k] : -1;
        c[j] = tab.more[k];
        c1[j] = live ? tab.more[k + 1] : c[j];
#pragma unroll
        for (int i = 0; i < 4; ++i) po[j][i] = p[(int64_t)k * 4 + i];
    }
    O2 v[SJ];
    double m[SJ];
#pragma unroll
    for (int j = 0; j < SJ; ++j) {
        v[j] = O2{};
        m[j] = 1.0;
        if (pt[j] >= 0) {
            v[j] = col[pt[j]];
            if (mask) m[j] = mask[pt[j]];
        }
    }
    auto add = [&](O2 &y, double mk, const Tc (&pv)[4], int slot) {
        Tc re = 0, im = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            re += pv[i] * sF[slot][i][o].x;
            im += pv[i] * sF[slot][i][o].y;
        }
        const double ar = mask ? mk * (double)re : (double)re, ai = mask ? mk * (double)im : (double)im;
        y.x = (Tout)((double)y.x + ar);
        y.y = (Tout)((double)y.y + ai);
    };
    for (int b0 = 0; b0 < it.w; b0 += SA) {
        const int nb = min(SA, it.w - b0);
        for (int j = t; j < nb * 32; j += SP * 8) {
            const int64_t nn = (int64_t)ct * 8 + (j & 7);
            if (nn < nst)
                sF[j >> 5][(j >> 3) & 3][j & 7] = scatter_coef<Tc>(D, P, nchunk, h3, E, ncols, tab.atoms[it.z + b0 + (j >> 5)],
                                                                   (j >> 3) & 3, nn, cre, cim);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SJ; ++j) {
            if (b0 == 0) add(v[j], m[j], po[j], 0);
            for (; c[j] < c1[j]; ++c[j]) {
                const int q = tab.place[c[j]];
                if (q >= b0 + nb) break;
                Tc pv[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) pv[i] = p[(int64_t)c[j] * 4 + i];
                add(v[j], m[j], pv, q - b0);
            }
        }
        if (b0 + SA < it.w) __syncthreads();  // the next atoms overwrite the coefficients
    }
#pragma unroll
    for (int j = 0; j < SJ; ++j)
        if (pt[j] >= 0) col[pt[j]] = v[j];
}

// blockIdx.x = item, blockIdx.y = tile of 8 orbitals.
template <class Tout, class Tc>
__global__ void __launch_bounds__(SP * 8) k_kb_scatter(Tout *__restrict__ out, int64_t ldo, int64_t ncols,
                                                       ScatterTab tab, const Tc *__restrict__ p,
                                                       const double *__restrict__ E, const Tc *__restrict__ D,
                                                       const Tc *__restrict__ P, int nchunk, Tc h3, double cre,
                                                       double cim, const double *__restrict__ mask) {
    __shared__ typename cpx<Tc>::type sF[SA][4][8];
    scatter_points<Tout, Tc>(out, ldo, ncols, tab.items[blockIdx.x], blockIdx.y, tab, p, E, D, P, nchunk, h3, cre, cim,
                             mask, sF);
}

constexpr int GW = 16;  // waves of a gather workgroup in a launch of its own

// blockIdx.x = {atom, column tile, chunk}, as in the stencil's launch.
template <class Tin, class Tc>
__global__ void __launch_bounds__(GW * 64) k_kb_gather(const Tin *__restrict__ in, GatherArgs g) {
    __shared__ Tc red[kGatherSlots * 64];
    const int j = blockIdx.x, chunk = j % g.nchunk, q = j / g.nchunk, atom = q / g.nct;
    gather_tile<GW, Tin, Tc>(in, g.ldo, g.ncols, g.atoms[atom], atom, q - atom * g.nct, g.idx,
                             static_cast<const Tc *>(g.p), (Tc)g.h3, static_cast<Tc *>(g.D), red, chunk, g.nchunk,
                             static_cast<Tc *>(g.P));
}

// Batched forms over many systems (FP64): item {system, atom, column tile}
// for the gather, {system, scatter item, orbital tile} for the scatter.
__global__ void __launch_bounds__(GW * 64) k_kb_gather_batch(const KbSys *__restrict__ sys,
                                                             const int4 *__restrict__ items) {
    __shared__ double red[kGatherSlots * 64];
    const int4 it = items[blockIdx.x];
    const KbSys &s = sys[it.x];
    gather_tile<GW, double, double>(s.in, s.ldo, s.ncols, s.atoms[it.y], it.y, it.z, s.idx, s.p, s.h3, s.D,
                                    red, it.w, s.nchunk, s.P);
}

__global__ void __launch_bounds__(SP * 8) k_kb_scatter_batch(const KbSys *__restrict__ sys,
                                                             const int4 *__restrict__ items, double cre, double cim) {
    __shared__ double2 sF[SA][4][8];
    const int4 it = items[blockIdx.x];
    const KbSys &s = sys[it.x];
    scatter_points<double, double>(s.out, s.ldo, s.ncols, s.tab.items[it.y], it.z, s.tab, s.scatter_p, s.E, s.D, s.P, s.nchunk,
                                   s.h3, cre, cim, nullptr, sF);
}

}  // namespace

// Support chunks per (atom, column tile): enough workgroups to fill the chip
// when there are few atoms or few orbitals.  Of the smallest support every chunk
// keeps at least 8 groups (of 4 entries) for each of its kGatherSlots running
// sums: with fewer, a batch of many small systems ran tens of thousands of
// nearly empty gather workgroups.  The count depends on the system alone, so
// a system gives the same bits alone or in a batch.
int gather_chunks(const Ham &H, int64_t nst) {
    if (H.natoms == 0 || nst == 0) return 1;
    int64_t min_groups = INT64_MAX;
    for (int32_t a = 0; a < H.natoms; ++a) min_groups = std::min(min_groups, (H.kb_off[a + 1] - H.kb_off[a]) / 4);
    const int64_t tiles = (int64_t)H.natoms * ((2 * nst + 15) / 16);
    const int64_t want = (512 + tiles - 1) / tiles;
    const int64_t cap = std::max<int64_t>(1, min_groups / (8 * kGatherSlots));
    return (int)std::max<int64_t>(1, std::min<int64_t>(std::min(want, cap), 64));
}

size_t gather_partials_offset(const Ham &H, int64_t nst) {
    const size_t dbytes = (size_t)H.natoms * 4 * 2 * (size_t)nst * sizeof(double);
    return (dbytes + 255) / 256 * 256;
}

// D [natoms][4][2 nst] plus, when the support is split, the chunk partials
// [natoms][4][nchunk][2 nst] behind it (sized for FP64 in every path).
size_t kb_workspace_bytes(const Ham &H, int64_t nst) {
    const size_t d = (size_t)H.natoms * 4 * 2 * (size_t)nst * sizeof(double);
    const int nchunk = gather_chunks(H, nst);
    return nchunk > 1 ? 2 * ((d + 255) / 256 * 256) + (size_t)nchunk * d : d;
}

KbDot kb_dot(const Ham &H, int64_t nst, const void *D) {
    KbDot k;
    k.natoms = H.natoms;
    if (H.natoms == 0) return k;
    k.E = H.kb_E;
    k.D = (const double *)D;
    k.nchunk = gather_chunks(H, nst);
    k.P = k.nchunk > 1 ? (const double *)((const char *)D + gather_partials_offset(H, nst)) : nullptr;
    k.ncols = 2 * nst;
    k.h3 = H.g->h * H.g->h * H.g->h;
    return k;
}

GatherArgs gather_args(const Ham &H, int compute, int64_t nst, int64_t ldp, void *D) {
    GatherArgs g;
    if (!D || H.natoms == 0 || nst == 0) return g;
    g.atoms = H.gather_items;
    g.idx = H.kb_idx;
    g.p = compute == 0 ? (const void *)H.kb_p : (const void *)H.kb_p32;
    g.D = D;
    g.ncols = 2 * nst;
    g.ldo = 2 * ldp;
    g.nct = (int32_t)((g.ncols + 15) / 16);
    g.nchunk = gather_chunks(H, nst);
    // the partials start at the first 256-byte boundary after D (FP64 size)
    g.P = g.nchunk > 1 ? (void *)((char *)D + gather_partials_offset(H, nst)) : nullptr;
    g.nblk = H.natoms * g.nct * g.nchunk;
    g.h3 = H.g->h * H.g->h * H.g->h;
    return g;
}

int launch_kb_gather(const GatherArgs &g, const void *in, int in_t, int compute, hipStream_t s) {
    if (g.nblk == 0) return RSG_OK;
    if (compute == 0)
        k_kb_gather<double, double><<<(unsigned)g.nblk, GW * 64, 0, s>>>((const double *)in, g);
    else if (in_t == 0)
        k_kb_gather<double, float><<<(unsigned)g.nblk, GW * 64, 0, s>>>((const double *)in, g);
    else
        k_kb_gather<float, float><<<(unsigned)g.nblk, GW * 64, 0, s>>>((const float *)in, g);
    RSG_CHECK_HIP(hipGetLastError());
    return RSG_OK;
}

int launch_kb_scatter(const Ham &H, void *out, int out_t, int compute, int64_t nst, int64_t ldp,
                      const void *D, double cre, double cim, const double *mask, hipStream_t s) {
    if (H.natoms == 0 || nst == 0 || H.scatter_n == 0) return RSG_OK;
    const int64_t ncols = 2 * nst;
    const int nchunk = gather_chunks(H, nst);
    const double h3 = H.g->h * H.g->h * H.g->h;
    const void *P = nchunk > 1 ? (const void *)((const char *)D + gather_partials_offset(H, nst)) : nullptr;
    const dim3 grid((unsigned)H.scatter_n, (unsigned)((nst + 7) / 8));
    if (compute == 0) {
        if (out_t != 0) return RSG_EUNSUPPORTED;
        k_kb_scatter<double, double><<<grid, SP * 8, 0, s>>>((double *)out, 2 * ldp, ncols, H.scatter, H.scatter_p, H.kb_E,
                                                             (const double *)D, (const double *)P, nchunk, h3, cre,
                                                             cim, mask);
    } else if (out_t == 0) {
        k_kb_scatter<double, float><<<grid, SP * 8, 0, s>>>((double *)out, 2 * ldp, ncols, H.scatter, H.scatter_p32, H.kb_E,
                                                            (const float *)D, (const float *)P, nchunk, (float)h3, cre,
                                                            cim, mask);
    } else {
        k_kb_scatter<float, float><<<grid, SP * 8, 0, s>>>((float *)out, 2 * ldp, ncols, H.scatter, H.scatter_p32, H.kb_E,
                                                           (const float *)D, (const float *)P, nchunk, (float)h3, cre,
                                                           cim, mask);
    }
    RSG_CHECK_HIP(hipGetLastError());
    return RSG_OK;
}

// The scatter's tables (ScatterTab) from the padded supports and the atoms'
// colours: the points of the union of all supports grouped by the first atom
// in colour order that covers them, each with its atoms in colour order.
// atom_of: the atom of every entry.  mark: one value per slot, not negative at
// every covered one; holds ~(place of the slot's point) there on return.
void build_scatter(const std::vector<int32_t> &idx, const std::vector<int64_t> &off, const std::vector<int64_t> &len,
                   const std::vector<int> &colour, const std::vector<int32_t> &atom_of, std::vector<int32_t> &mark,
                   ScatterHost *t) {
    const int natoms = (int)len.size();
    std::vector<int> ord(natoms);
    for (int a = 0; a < natoms; ++a) ord[a] = a;
    std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) { return colour[a] < colour[b]; });
    int64_t nc = 0;
    for (const int64_t l : len) nc += l;
    t->pt.resize(nc);
    t->entry.resize(nc);
    t->more.assign(nc + 1, 0);
    size_t n = 0;  // points so far; more[u + 1] counts point u's atoms beyond its owner
    for (const int a : ord)
        for (int64_t k = 0; k < len[a]; ++k) {
            const int32_t e = (int32_t)(off[a] + k);
            int32_t &m = mark[idx[e]];
            if (m >= 0) {
                m = ~(int32_t)n;
                t->pt[n] = idx[e];
                t->entry[n++] = e;
            } else {
                ++t->more[~m + 1];
            }
        }
    t->pt.resize(n);
    t->more.resize(n + 1);
    t->more[0] = (int32_t)n;
    for (size_t u = 0; u < n; ++u) t->more[u + 1] += t->more[u];
    t->place.assign(nc, 0);
    if ((size_t)nc > n) {
        std::vector<int32_t> fill(t->more.begin(), t->more.end() - 1);
        for (const int a : ord)
            for (int64_t k = 0; k < len[a]; ++k) {
                const int32_t e = (int32_t)(off[a] + k), u = ~mark[idx[e]];
                if (t->entry[u] == e) continue;
                t->entry[fill[u]] = e;
                t->place[fill[u]++] = a;  // the atom for now
            }
    }
    std::vector<int> rank(natoms), seen(natoms, -1), list;
    for (int j = 0; j < natoms; ++j) rank[ord[j]] = j;
    for (size_t u = 0; u < n;) {
        const int owner = atom_of[t->entry[u]];
        size_t v = u + 1;
        while (v < n && v - u < (size_t)kScatterPoints && atom_of[t->entry[v]] == owner) ++v;
        list.assign(1, owner);  // the item's atoms in colour order, the owner first
        seen[owner] = (int)t->items.size();
        for (int32_t c = t->more[u]; c < t->more[v]; ++c) {
            const int a = t->place[c];
            if (seen[a] != (int)t->items.size()) {
                seen[a] = (int)t->items.size();
                list.push_back(a);
            }
        }
        std::sort(list.begin() + 1, list.end(), [&](int a, int b) { return rank[a] < rank[b]; });
        for (int32_t c = t->more[u]; c < t->more[v]; ++c)
            t->place[c] = (int32_t)(std::find(list.begin(), list.end(), t->place[c]) - list.begin());
        t->items.push_back(make_int4((int)u, (int)(v - u), (int)t->atoms.size(), (int)list.size()));
        t->atoms.insert(t->atoms.end(), list.begin(), list.end());
        u = v;
    }
}

int launch_kb_gather_batch(const KbSys *sys, const int4 *items, int32_t nitems, hipStream_t s) {
    if (nitems == 0) return RSG_OK;
    k_kb_gather_batch<<<(unsigned)nitems, GW * 64, 0, s>>>(sys, items);
    RSG_CHECK_HIP(hipGetLastError());
    return RSG_OK;
}

int launch_kb_scatter_batch(const KbSys *sys, const int4 *items, int32_t nitems, double cre, double cim,
                            hipStream_t s) {
    if (nitems == 0) return RSG_OK;
    k_kb_scatter_batch<<<(unsigned)nitems, SP * 8, 0, s>>>(sys, items, cre, cim);
    RSG_CHECK_HIP(hipGetLastError());
    return RSG_OK;
}

}  // namespace rsg
