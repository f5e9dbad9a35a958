// Kinetic + local-potential part of H applied to an orbital batch, with the
// Taylor-stage epilogue fused in.
//
//   (H psi)(r) = kin/h^2 sum_axes sum_{m=-4..4} c_|m| psi(r + m h e_axis)
//              + (V(r) + E x_axis(r)) psi(r)
//
// c_0..c_4 = -205/72, 8/5, -1/5, 8/315, -1/560 (8th-order centred second
// derivative); orbitals vanish outside the box.  High-order finite
// differences are the discretisation of the section "Introduction"; the
// order is this library's choice.  The separable projectors are added by the
// projector kernels after this one.
//
// Data layout: an orbital batch is orbital-major, [nst][ldp] complex:
// orbital n holds its values at n*ldp + i for compact point i (z-major, y,
// x), so every orbital is one contiguous field and every grid row of it is
// contiguous.  Mapping onto CDNA4:
//   - one workgroup owns a TX x TY tile of (x, y) columns of one orbital and
//     marches along z over the tile's z-extent (or a chunk of it);
//   - a thread owns one column and keeps its complex value on the planes
//     z-4..z+4 in registers (z taps), plus the planes in flight;
//   - the current plane, with a 4-point x/y halo, is staged in LDS for the
//     x and y taps (two plane buffers used in turn, so one barrier per plane
//     suffices); the halo comes from the neighbouring tiles through L2;
//   - x runs fastest over the threads, so a wave's loads are runs of TX
//     consecutive 16-byte values;
//   - loads of later planes are issued before the current plane is computed
//     (software pipeline, depth PD);
//   - workgroup ids are remapped so that each XCD (own L2) receives a
//     contiguous range of the launch order.
// A tile per workgroup covers many more points than a point-major layout
// with the orbitals of a point side by side would allow in the same
// registers, so far fewer halo values are read per output.
//
// The kernels come in two sets that differ only in the store policy of the
// stage output (NTS: non-temporal stores for outputs much larger than the
// caches); each set is instantiated in a source file of its own.
#pragma once

#include "kb_gather.h"
#include "rsg_internal.h"
#include "stencil_common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace rsg {
namespace sk {

// Sums a stage gathers on the way.
enum { SUM_NONE = 0, SUM_PAIR = 1, SUM_TDOT = 2, SUM_HDOT = 3, SUM_ONLY = 4 };


// Halo assignment of a TX x TY tile (fixed for the whole march): halo value
// j is a y-halo point for j < 8 TX (4 rows above, 4 below, x fastest) and an
// x-halo point otherwise (4 left and 4 right of each tile row).
template <int TX, int TY, int NT, int HPT>
struct Halo {
    int l[HPT], x[HPT], y[HPT];
    bool ok[HPT];
    __device__ __forceinline__ Halo(int t, int4 it) {
        constexpr int NHP = 8 * TX + 8 * TY, LX = TX + 8;
#pragma unroll
        for (int k = 0; k < HPT; ++k) {
            const int j = t + k * NT;
            int lxl, lyl;
            if (j < 8 * TX) {
                const int yh = j / TX;
                lxl = j % TX + 4;
                lyl = yh < 4 ? yh : TY + yh;
            } else {
                const int q = j - 8 * TX;
                const int cc = q % 8;
                lyl = q / 8 + 4;
                lxl = cc < 4 ? cc : TX + cc;
            }
            ok[k] = j < NHP;
            if (!ok[k]) lxl = lyl = 0;
            l[k] = lyl * LX + lxl;
            x[k] = it.x * TX + lxl - 4;
            y[k] = it.y * TY + lyl - 4;
        }
    }
};

// x_axis along the march: bound to the thread's column for axis 0 (xa), to
// the row or plane for axis 1 and 2 (hz = h there, else 0; at() takes that
// row or plane), zero without a field axis, and the field E (zero without an
// axis), so that a step needs no test of the axis.
struct FieldTerm {
    double xa, hz, off, E;
    __device__ __forceinline__ FieldTerm(const KParams &a, int x) {
        xa = a.axis == 0 ? a.h * ((double)x - a.off_axis) : 0.0;
        hz = a.axis >= 1 ? a.h : 0.0;
        off = a.off_axis;
        E = a.axis < 0 ? 0.0 : (a.field_dev ? *a.field_dev : a.field);
    }
    __device__ __forceinline__ double at(int i) const { return fma(hz, (double)i - off, xa); }
};

// The per-point epilogue shared by both marches: H value from the Laplacian
// taps, then the stage combination (times the absorber mask m_c when MASK),
// stored at the point's code (zero at a dead slot, dropped outside the box).
// SUM_PAIR (a first-type FP64 stage of the discrete adjoint): b_c
// holds the pair operand u at the point, and pacc gathers conj(in) x_axis u
// (zero wherever the point is outside the box, since both loads read zero
// there).  SUM_TDOT, SUM_HDOT (H applications): pacc gathers in H in without
// and with conjugation of the first factor, over the box points; SUM_ONLY
// does the second and stores nothing.
template <bool NTS, class Tc, class Tout, int MODE, bool FIRST, bool MASK, bool CS, int SUM = 0>
__device__ __forceinline__ void finish(const KParams &a, typename CT<Tc>::c2 q0, Tc lr, Tc li, Tc v_c,
                                       Tc vi_c, double2 b_c, double m_c, const FieldTerm &f, int yz,
                                       unsigned code, __amdgpu_buffer_rsrc_t rout, double2 &pacc) {
    const double xc = f.at(yz);
    const Tc vloc = v_c + (Tc)(f.E * xc);
    if constexpr (SUM == SUM_PAIR) {
        pacc.x += xc * ((double)q0.x * b_c.x + (double)q0.y * b_c.y);
        pacc.y += xc * ((double)q0.x * b_c.y - (double)q0.y * b_c.x);
    }
    const Tc kin_h2 = (Tc)a.kin_h2;
    Tc hr, hi;
    if constexpr (CS) {
        // complex kinetic prefactor and complex local potential
        const Tc ki = (Tc)a.kin_h2_im;
        hr = kin_h2 * lr - ki * li + vloc * q0.x - vi_c * q0.y;
        hi = kin_h2 * li + ki * lr + vloc * q0.y + vi_c * q0.x;
    } else {
        hr = kin_h2 * lr + vloc * q0.x;
        hi = kin_h2 * li + vloc * q0.y;
    }
    const bool zero = (int)code < 0;
    const unsigned o = coff<Tout>(code & ~CODE_DEAD);
    if (MODE == 0) {
        const double sr = zero ? 0.0 : (double)hr, si = zero ? 0.0 : (double)hi;
        if constexpr (SUM == SUM_TDOT) {
            pacc.x += q0.x * sr - q0.y * si;
            pacc.y += q0.x * si + q0.y * sr;
        } else if constexpr (SUM == SUM_HDOT || SUM == SUM_ONLY) {
            pacc.x += q0.x * sr + q0.y * si;
            pacc.y += q0.x * si - q0.y * sr;
        }
        if constexpr (SUM != SUM_ONLY) store_c<NTS>(rout, o, (Tout *)nullptr, sr, si);
    } else {
        const double2 bb = FIRST ? make_double2((double)q0.x, (double)q0.y) : b_c;
        double r = bb.x + (a.cre * (double)hr - a.cim * (double)hi);
        double i = bb.y + (a.cre * (double)hi + a.cim * (double)hr);
        if (MASK) {
            r *= m_c;
            i *= m_c;
        }
        store_c<NTS>(rout, o, (Tout *)nullptr, zero ? 0.0 : r, zero ? 0.0 : i);
    }
}

// A stage that carries another operand per point (a base, a mask, an adjoint
// pair).
constexpr bool stage_heavy(int mode, bool first, int sum) { return mode == 1 && (!first || sum == SUM_PAIR); }

// Constants of the pipelined march: depth D, ring lengths, and the LDS ring
// of row entries (segments of P planes, the unroll period).
template <int TX, int TY, int D, int CY, bool HEAVY>
struct Ring {
    static_assert(D >= 1 && D <= 2, "pipeline depth 1..2");
    static constexpr int NT = TX * TY / CY;                       // threads
    static constexpr int HPT = (8 * TX + 8 * TY + NT - 1) / NT;  // halo values per thread
    static constexpr int Q = D == 1 ? 10 : 12;                   // own-column ring, >= 9 + D
    static constexpr int HA = HPT <= CY && !HEAVY ? 4 + D : D;   // planes ahead at which the halo is loaded
    static constexpr int VD = D + 1;                             // V / base ring slots
    static constexpr int P = clcm(clcm(clcm(clcm(Q, D), VD), 2), HA);
    static constexpr int RY = TY + 8;                            // rows of a plane, halo included
    static constexpr int SEG = HA == 4 + D ? 2 : 3;              // live segments of row entries
    static constexpr int RPT = (P * RY + NT - 1) / NT;           // row entries a thread loads per segment
    static constexpr int ROWS = SEG * P * RY;                    // int4 in LDS
};

// Software-pipelined march, depth D = 1..2, over the item's planes zs, zs +
// dir, ... (dir = +1 upward, -1 downward; the stencil is symmetric in z).
// At step k (output plane z = zs + dir k) a thread
//   - issues the data loads of plane k+4+D (own column), of the halo of plane
//     k+HA and of V and base at plane k+D,
//   - computes plane k from data that arrived during earlier steps.
// HA = 4+D when each thread carries one halo value per column (the halo of a
// plane is then loaded in the same step as the plane's own columns, by this
// and by the neighbouring workgroups, while the lines are in L2), else HA = D;
// the FP64 stages with another operand take HA = D too (16 registers, the
// difference between 2 and 3 waves per SIMD at 16 x 16).
// All rings are indexed by compile-time constants after unrolling the step
// loop by a common period, so no register is moved while its load is in
// flight.  FIRST: base == in, whose value at the point is the centre tap.
//
// Row entries come from LDS: the workgroup keeps the entries of its TY + 8
// rows for one unroll period of planes ahead, loaded together once per
// period.  Loaded by every thread for the next step, they sat in the vector
// memory queue between the data loads; that queue completes in order, so
// waiting for a row entry also waited for the data loads issued a step
// before it, which cut the pipeline to one step whatever D said.  The ring
// also takes two loads and about 40 of 118 vector instructions (table
// addresses, range tests, offsets) out of every step, and 16-24 registers,
// so depth-1 FP64 tiles run 3 waves per SIMD instead of 2.  Measured: a
// Taylor stage of the 3.05 M-point sphere with 64 orbitals 1.88 -> 1.79 ms
// (32 x 16, depth 2) and 1.81 -> 1.65 ms with the best tile of each form;
// 96^3 cube, 8 orbitals 77 -> 64 us; 48 uneven spheres 2.6 -> 1.8 ms.
template <bool NTS, int TX, int TY, int D, int CY, class Tin, class Tc, class Tout, int MODE, bool FIRST, bool MASK,
          bool CS, int SUM>
__device__ __forceinline__ void march_ring(const KParams &a, const int4 it, const int n,
                                           typename CT<Tc>::c2 *tile, int4 *rowl, double2 &pacc) {
    using C2 = typename CT<Tc>::c2;
    using R = Ring<TX, TY, D, CY, std::is_same<Tc, double>::value && stage_heavy(MODE, FIRST, SUM)>;
    constexpr int NT = R::NT, LX = TX + 8, HPT = R::HPT, Q = R::Q, HA = R::HA, HQ = R::HA, VD = R::VD, P = R::P;
    constexpr int RY = R::RY, SEG = R::SEG, RPT = R::RPT;
    constexpr int PLANE = (TY + 8) * LX;       // one plane buffer; tile holds two
    const int t = threadIdx.x, lx = t % TX, ly = t / TX * CY;
    const int x = it.x * TX + lx, y = it.y * TY + ly;
    const int64_t np = a.np;
    const auto rin = rsrc(static_cast<const Tin *>(a.in) + (int64_t)n * a.ldp, np * (int64_t)sizeof(Tin));
    // the base operand (later stages), or the pair operand of an adjoint stage
    const auto rbase = rsrc(static_cast<const double2 *>(SUM == SUM_PAIR ? a.pair_y : a.base) + (int64_t)n * a.ldp, np * 16);
    const auto rout = rsrc(static_cast<Tout *>(a.out) + (int64_t)n * a.ldp, np * (int64_t)sizeof(Tout));
    const auto rv = rsrc(a.V, np * (int64_t)sizeof(Tc));
    const auto rm = rsrc(MASK ? a.mask : a.V, MASK ? np * 8 : 0);
    const auto rvi = rsrc(CS ? a.Vim : a.V, CS && a.Vim ? np * 8 : 0);
    const Halo<TX, TY, NT, HPT> hl(t, it);

    auto fetch = [&](unsigned c) -> C2 { return load_c<Tc, Tin>(rin, coff<Tin>(c)); };
    auto fetch_v = [&](unsigned c) -> Tc { return BL<Tc>::ld(rv, coff<Tc>(c)); };
    auto fetch_b = [&](unsigned c) -> double2 {
        if (MODE != 1 || (FIRST && SUM != SUM_PAIR)) return make_double2(0.0, 0.0);
        return BL<double2>::ld(rbase, coff<double2>(c));
    };
    auto fetch_m = [&](unsigned c) -> double { return MASK ? BL<double>::ld(rm, coff<double>(c)) : 1.0; };
    auto fetch_vi = [&](unsigned c) -> Tc { return CS ? (Tc)BL<double>::ld(rvi, coff<double>(c)) : (Tc)0; };

    const int zs = it.z, dir = it.w > it.z ? 1 : -1;
    const int nk = (it.w - it.z) * dir;  // planes to compute

    // Row entries of segment b (planes bP + 4 + D ... bP + P + 3 + D of the
    // march, b = -1 the prologue's), one per thread and pass; rows outside
    // the tight box and planes past the last one read (nk + 3) are empty.
    int2 seg[RPT];
    auto seg_load = [&](int b) {
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int e = t + j * NT, pl = e / RY, r = e - pl * RY;
            const int k = b * P + 4 + D + pl;
            const int yy = it.y * TY + r - 4, zz = zs + dir * k;
            const bool v = (unsigned)yy < (unsigned)a.ny && (unsigned)zz < (unsigned)a.nz && k < nk + 4 && pl < P;
            // the rows of a full box need no table (FP64: the choice would
            // take the first FP32 stage from 128 to 130 registers, 4 waves to
            // 3: a mixed step of 500 k points x 32 orbitals 583 -> 602 us)
            if (std::is_same<Tc, double>::value && a.row_slots)
                seg[j] = v ? make_int2((zz * a.ny + yy) * a.row_slots, a.row_len << 16) : make_int2(0, 0);
            else
                seg[j] = a.rows[v ? zz * a.ny + yy : a.ny * a.nz];
        }
    };
    auto seg_store = [&](int slot) {
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int e = t + j * NT;
            if (P * RY % NT == 0 || e < P * RY) rowl[slot * (P * RY) + e] = row_entry(seg[j], a.align);
        }
    };
    // prologue: planes k = -4 .. 3+D into ring slots 0 .. Q-2 (slot of plane
    // k is k + 4), halo of planes 0 .. HA-1, V/base of planes 0 .. D-1
    seg_load(-1);
    seg_store(SEG - 1);
    seg_load(0);
    seg_store(0);
    int hrow[HPT];  // row of each halo value within a plane's entries
#pragma unroll
    for (int j = 0; j < HPT; ++j) hrow[j] = hl.l[j] / LX;
    __syncthreads();
    const int4 *const pro = rowl + (SEG - 1) * (P * RY) + (P - 4 - D) * RY;  // entries of plane 0
    C2 cv[CY][Q];
    unsigned oid[CY][Q];
#pragma unroll
    for (int c = 0; c < CY; ++c) {
#pragma unroll
        for (int j = 0; j < Q - 1; ++j) {
            oid[c][j] = code_in_row(pro[(j - 4) * RY + ly + 4 + c], x);
            cv[c][j] = fetch(oid[c][j]);
        }
        cv[c][Q - 1] = C2{(Tc)0, (Tc)0};
        oid[c][Q - 1] = CODE_OUT;
    }
    C2 hal[HQ][HPT];
#pragma unroll
    for (int d = 0; d < HQ; ++d)
#pragma unroll
        for (int j = 0; j < HPT; ++j) hal[d][j] = fetch(halo_code(pro[d * RY + hrow[j]], hl.x[j], hl.ok[j] && d < nk));
    Tc vr[CY][VD], vir[CY][VD];
    double2 br[CY][VD];
    double mr[CY][VD];
#pragma unroll
    for (int c = 0; c < CY; ++c) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            vr[c][d] = fetch_v(oid[c][4 + d]);
            vir[c][d] = fetch_vi(oid[c][4 + d]);
            br[c][d] = fetch_b(oid[c][4 + d]);
            mr[c][d] = fetch_m(oid[c][4 + d]);
        }
        vr[c][D] = (Tc)0;
        vir[c][D] = (Tc)0;
        br[c][D] = make_double2(0.0, 0.0);
        mr[c][D] = 0.0;
    }

    const FieldTerm ft(a, x);
    const int own = (ly + 4) * LX + lx + 4;
    int slot = 0;  // LDS segment of the current period

    for (int kb = 0, b = 0; kb < nk; kb += P, ++b) {
        const int next = slot + 1 == SEG ? 0 : slot + 1, prev = slot == 0 ? SEG - 1 : slot - 1;
        const int4 *const rs = rowl + slot * (P * RY), *const rp = rowl + prev * (P * RY);
#pragma unroll
        for (int s = 0; s < P; ++s) {
            const int k = kb + s;
            if (k >= nk) break;
            const int z = zs + dir * k;
            const int sh = s % HQ;
            const int shl = (s + HA) % HQ;              // halo slot of plane k + HA
            const int sv = s % VD, svn = (s + D) % VD;  // V/base: read slot, load slot
            // ring slot of plane k + m
#define SLOT(m) ((s + (m) + 4 + Q) % Q)
            C2 *const pl = tile + (s % 2) * PLANE;  // plane buffer of this step
#pragma unroll
            for (int c = 0; c < CY; ++c) pl[own + c * LX] = cv[c][SLOT(0)];
#pragma unroll
            for (int j = 0; j < HPT; ++j)
                if (hl.ok[j]) pl[hl.l[j]] = hal[sh][j];
            // next period's row entries: requested at the period's start,
            // stored D + 2 steps later, when they have arrived with the data
            // loads around them
            if (s == 0) seg_load(b + 1);
            if (s == D + 2) seg_store(next);
            unsigned code_c[CY];
            Tc v_c[CY], vi_c[CY];
            double2 b_c[CY];
            double m_c[CY];
#pragma unroll
            for (int c = 0; c < CY; ++c) {
                code_c[c] = oid[c][SLOT(0)];
                v_c[c] = vr[c][sv];
                vi_c[c] = vir[c][sv];
                b_c[c] = br[c][sv];
                m_c[c] = mr[c][sv];
            }
            __syncthreads();
            {
#pragma unroll
                for (int c = 0; c < CY; ++c) {
                    const unsigned cf = code_in_row(rs[s * RY + ly + 4 + c], x);
                    oid[c][SLOT(4 + D)] = cf;
                    cv[c][SLOT(4 + D)] = fetch(cf);
                }
                const bool hlive = k + HA < nk;
                constexpr int back = 4 + D - HA;  // the halo's plane lies this far behind the own column's
#pragma unroll
                for (int j = 0; j < HPT; ++j) {
                    const int4 e = s >= back ? rs[(s - back) * RY + hrow[j]] : rp[(P + s - back) * RY + hrow[j]];
                    hal[shl][j] = fetch(halo_code(e, hl.x[j], hl.ok[j] && hlive));
                }
#pragma unroll
                for (int c = 0; c < CY; ++c) {
                    const unsigned cd = k + D < nk ? oid[c][SLOT(D)] : CODE_OUT;
                    vr[c][svn] = fetch_v(cd);
                    vir[c][svn] = fetch_vi(cd);
                    br[c][svn] = fetch_b(cd);
                    mr[c][svn] = fetch_m(cd);
                }
            }
            // rows y - 4 .. y + CY + 3 of this column: the thread's own rows
            // from registers, the others from the plane
            C2 yr[CY + 8];
#pragma unroll
            for (int r = 0; r < CY + 8; ++r)
                yr[r] = r >= 4 && r < 4 + CY ? cv[r >= 4 && r < 4 + CY ? r - 4 : 0][SLOT(0)] : pl[own + (r - 4) * LX];
#pragma unroll
            for (int c = 0; c < CY; ++c) {
                const C2 q0 = cv[c][SLOT(0)];
                const C2 *const row = pl + own + c * LX;
                Tc lr, li;
                {
                    const C2 xm1 = row[-1], xp1 = row[1], xm2 = row[-2], xp2 = row[2];
                    const C2 xm3 = row[-3], xp3 = row[3], xm4 = row[-4], xp4 = row[4];
                    const C2 ym1 = yr[c + 3], yp1 = yr[c + 5], ym2 = yr[c + 2], yp2 = yr[c + 6];
                    const C2 ym3 = yr[c + 1], yp3 = yr[c + 7], ym4 = yr[c], yp4 = yr[c + 8];
                    const C2 zm1 = cv[c][SLOT(-1)], zp1 = cv[c][SLOT(1)], zm2 = cv[c][SLOT(-2)], zp2 = cv[c][SLOT(2)];
                    const C2 zm3 = cv[c][SLOT(-3)], zp3 = cv[c][SLOT(3)], zm4 = cv[c][SLOT(-4)], zp4 = cv[c][SLOT(4)];
                    lr = (Tc)3 * FD<Tc>::c0 * q0.x + FD<Tc>::c1 * ((xm1.x + xp1.x) + (ym1.x + yp1.x) + (zm1.x + zp1.x)) +
                         FD<Tc>::c2 * ((xm2.x + xp2.x) + (ym2.x + yp2.x) + (zm2.x + zp2.x)) +
                         FD<Tc>::c3 * ((xm3.x + xp3.x) + (ym3.x + yp3.x) + (zm3.x + zp3.x)) +
                         FD<Tc>::c4 * ((xm4.x + xp4.x) + (ym4.x + yp4.x) + (zm4.x + zp4.x));
                    li = (Tc)3 * FD<Tc>::c0 * q0.y + FD<Tc>::c1 * ((xm1.y + xp1.y) + (ym1.y + yp1.y) + (zm1.y + zp1.y)) +
                         FD<Tc>::c2 * ((xm2.y + xp2.y) + (ym2.y + yp2.y) + (zm2.y + zp2.y)) +
                         FD<Tc>::c3 * ((xm3.y + xp3.y) + (ym3.y + yp3.y) + (zm3.y + zp3.y)) +
                         FD<Tc>::c4 * ((xm4.y + xp4.y) + (ym4.y + yp4.y) + (zm4.y + zp4.y));
                }
                finish<NTS, Tc, Tout, MODE, FIRST, MASK, CS, SUM>(a, q0, lr, li, v_c[c], vi_c[c], b_c[c], m_c[c], ft,
                                                                   a.axis == 1 ? y + c : z, code_c[c], rout, pacc);
            }
#undef SLOT
            // no barrier here: the next step writes the other plane buffer,
            // and every wave has finished reading it once all have passed
            // this step's barrier
        }
        slot = next;
    }
}

// Lean march (depth 1, few registers): the own-column queue q[9] rotates in
// registers and every load of plane k+1 (own column k+5, halo, V, base) is
// issued one step ahead; a step starts by waiting for the previous step's
// loads.  Planes run zs, zs + dir, ... as in the pipelined march.
template <bool NTS, int TX, int TY, class Tin, class Tc, class Tout, int MODE, bool FIRST, bool MASK, bool CS,
          int SUM>
__device__ __forceinline__ void march_lean(const KParams &a, const int4 it, const int n,
                                           typename CT<Tc>::c2 *tile, double2 &pacc) {
    using C2 = typename CT<Tc>::c2;
    constexpr int NT = TX * TY, LX = TX + 8;
    constexpr int HPT = (8 * TX + 8 * TY + NT - 1) / NT;
    constexpr int PLANE = (TY + 8) * LX;  // one plane buffer; tile holds two
    const int t = threadIdx.x, lx = t % TX, ly = t / TX;
    const int x = it.x * TX + lx, y = it.y * TY + ly;
    const int64_t np = a.np;
    const auto rin = rsrc(static_cast<const Tin *>(a.in) + (int64_t)n * a.ldp, np * (int64_t)sizeof(Tin));
    // the base operand (later stages), or the pair operand of an adjoint stage
    const auto rbase = rsrc(static_cast<const double2 *>(SUM == SUM_PAIR ? a.pair_y : a.base) + (int64_t)n * a.ldp, np * 16);
    const auto rout = rsrc(static_cast<Tout *>(a.out) + (int64_t)n * a.ldp, np * (int64_t)sizeof(Tout));
    const auto rv = rsrc(a.V, np * (int64_t)sizeof(Tc));
    const auto rm = rsrc(MASK ? a.mask : a.V, MASK ? np * 8 : 0);
    const auto rvi = rsrc(CS ? a.Vim : a.V, CS && a.Vim ? np * 8 : 0);
    const Halo<TX, TY, NT, HPT> hl(t, it);

    auto fetch = [&](int idx, bool ok) -> C2 { return load_c<Tc, Tin>(rin, ok ? boff<Tin>(idx) : OOB); };
    auto fetch_v = [&](int idx) -> Tc { return BL<Tc>::ld(rv, boff<Tc>(idx)); };
    auto fetch_b = [&](int idx) -> double2 {
        if (MODE != 1 || (FIRST && SUM != SUM_PAIR)) return make_double2(0.0, 0.0);
        return BL<double2>::ld(rbase, boff<double2>(idx));
    };
    auto fetch_m = [&](int idx) -> double { return MASK ? BL<double>::ld(rm, boff<double>(idx)) : 1.0; };
    auto fetch_vi = [&](int idx) -> Tc { return CS ? (Tc)BL<double>::ld(rvi, boff<double>(idx)) : (Tc)0; };

    const int zs = it.z, dir = it.w > it.z ? 1 : -1;
    const int nk = (it.w - it.z) * dir;
    // every row entry of the prologue is requested before any is used (one
    // round trip, not one per entry)
    int2 rq[9];  // planes zs - 4 .. zs + 4
#pragma unroll
    for (int j = 0; j < 9; ++j) rq[j] = row_of(a, y, zs + dir * (j - 4));
    int2 rh0[HPT];
#pragma unroll
    for (int j = 0; j < HPT; ++j) rh0[j] = row_of(a, hl.y[j], zs);
    int2 rf = row_of(a, y, zs + dir * 5);  // rows for the loads of the first step
    int2 ro = rq[5];                       // plane zs + 1
    int2 rh[HPT];
#pragma unroll
    for (int j = 0; j < HPT; ++j) rh[j] = row_of(a, hl.y[j], zs + dir);
    C2 q[9];
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = fetch(idx_in_row(rq[j], x), true);
    int idx_c = slot_in_row(rq[4], x, a.align);
    C2 nxt = fetch(idx_in_row(rq[8], x), true);
    C2 hv[HPT];
#pragma unroll
    for (int j = 0; j < HPT; ++j) hv[j] = fetch(idx_in_row(rh0[j], hl.x[j]), hl.ok[j]);
    Tc v_c = fetch_v(idx_c);
    Tc vi_c = fetch_vi(idx_c);
    double2 b_c = fetch_b(idx_c);
    double m_c = fetch_m(idx_c);

    const FieldTerm ft(a, x);
    const int own = (ly + 4) * LX + lx + 4;

    for (int k = 0; k < nk; ++k) {
        const int z = zs + dir * k;
        C2 *const pl = tile + (k & 1) * PLANE;  // plane buffer of this step
        q[8] = nxt;
        pl[own] = q[4];
#pragma unroll
        for (int j = 0; j < HPT; ++j)
            if (hl.ok[j]) pl[hl.l[j]] = hv[j];
        __syncthreads();
        // row entries for the next step, then this step's loads (plane k+1)
        const int2 rf_n = row_of(a, y, z + dir * 6), ro_n = row_of(a, y, z + dir * 2);
        int2 rh_n[HPT];
#pragma unroll
        for (int j = 0; j < HPT; ++j) rh_n[j] = row_of(a, hl.y[j], z + dir * 2);
        const bool live = k + 1 < nk;
        nxt = fetch(live ? idx_in_row(rf, x) : -1, true);
#pragma unroll
        for (int j = 0; j < HPT; ++j) hv[j] = fetch(idx_in_row(rh[j], hl.x[j]), hl.ok[j] && live);
        const int idx_n = live ? slot_in_row(ro, x, a.align) : -1;
        const Tc v_n = fetch_v(idx_n);
        const Tc vi_n = fetch_vi(idx_n);
        const double2 b_n = fetch_b(idx_n);
        const double m_n = fetch_m(idx_n);
        rf = rf_n;
        ro = ro_n;
#pragma unroll
        for (int j = 0; j < HPT; ++j) rh[j] = rh_n[j];

        const C2 q0 = q[4];
        Tc lr, li;
        {
            const C2 xm1 = pl[own - 1], xp1 = pl[own + 1], xm2 = pl[own - 2], xp2 = pl[own + 2];
            const C2 xm3 = pl[own - 3], xp3 = pl[own + 3], xm4 = pl[own - 4], xp4 = pl[own + 4];
            const C2 ym1 = pl[own - LX], yp1 = pl[own + LX], ym2 = pl[own - 2 * LX], yp2 = pl[own + 2 * LX];
            const C2 ym3 = pl[own - 3 * LX], yp3 = pl[own + 3 * LX], ym4 = pl[own - 4 * LX], yp4 = pl[own + 4 * LX];
            lr = (Tc)3 * FD<Tc>::c0 * q0.x + FD<Tc>::c1 * ((xm1.x + xp1.x) + (ym1.x + yp1.x) + (q[3].x + q[5].x)) +
                 FD<Tc>::c2 * ((xm2.x + xp2.x) + (ym2.x + yp2.x) + (q[2].x + q[6].x)) +
                 FD<Tc>::c3 * ((xm3.x + xp3.x) + (ym3.x + yp3.x) + (q[1].x + q[7].x)) +
                 FD<Tc>::c4 * ((xm4.x + xp4.x) + (ym4.x + yp4.x) + (q[0].x + q[8].x));
            li = (Tc)3 * FD<Tc>::c0 * q0.y + FD<Tc>::c1 * ((xm1.y + xp1.y) + (ym1.y + yp1.y) + (q[3].y + q[5].y)) +
                 FD<Tc>::c2 * ((xm2.y + xp2.y) + (ym2.y + yp2.y) + (q[2].y + q[6].y)) +
                 FD<Tc>::c3 * ((xm3.y + xp3.y) + (ym3.y + yp3.y) + (q[1].y + q[7].y)) +
                 FD<Tc>::c4 * ((xm4.y + xp4.y) + (ym4.y + yp4.y) + (q[0].y + q[8].y));
        }
        finish<NTS, Tc, Tout, MODE, FIRST, MASK, CS, SUM>(a, q0, lr, li, v_c, vi_c, b_c, m_c, ft, a.axis == 1 ? y : z, code_of(idx_c),
                                                       rout, pacc);
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = q[j + 1];
        idx_c = idx_n;
        v_c = v_n;
        vi_c = vi_n;
        b_c = b_n;
        m_c = m_n;
    }
}

// Columns per thread (in y) of a tile: two in the FP64 depth-1 march of the
// widest tiles.  The thread's two rows share 8 of their 16 y taps and the
// halo and address registers, so the 32 x 16 tile needs 256 threads of 242
// VGPRs and two of them are resident per compute unit, 1024 columns in
// flight instead of 768 (16 x 16 tiles) with half the x halo per column.
// Stages that carry another operand (stage_heavy) would spill in that form;
// they keep one column per thread at 32 x 16, and fit at 32 x 32 (512
// threads, one halo value each).  Measured per stage:
// 3.05 M-point sphere x 64 orbitals 1.65 (16 x 16) and 1.71 ms (32 x 16, one
// column) -> 1.59 ms (32 x 16, two), 96^3 cube x 8 57 -> 52 us (32 x 32; a
// candidate of the tuner, no default).
constexpr int tile_cy(int TX, int TY, int D, bool fp64, bool heavy) {
    return fp64 && D == 1 && (TX * TY == 1024 || (TX * TY == 512 && TX == 32 && !heavy)) ? 2 : 1;
}
template <int TX, int TY, int D, class Tc, int MODE, bool FIRST, int SUM>
constexpr int stage_cy() {
    return tile_cy(TX, TY, D, std::is_same<Tc, double>::value, stage_heavy(MODE, FIRST, SUM));
}
// LDS row entries of a march (the lean one needs none).
template <int TX, int TY, int D, int CY, bool HEAVY>
constexpr int march_rows() {
    if constexpr (D == 0)
        return 1;
    else
        return Ring<TX, TY, D, CY, HEAVY>::ROWS;
}

template <bool NTS, int TX, int TY, int D, class Tin, class Tc, class Tout, int MODE, bool FIRST, bool MASK, bool CS,
          int SUM = 0>
__device__ __forceinline__ void march(const KParams &a, const int4 it, const int n, typename CT<Tc>::c2 *tile,
                                      int4 *rowl, double2 &pacc) {
    if constexpr (D == 0)
        march_lean<NTS, TX, TY, Tin, Tc, Tout, MODE, FIRST, MASK, CS, SUM>(a, it, n, tile, pacc);
    else
        march_ring<NTS, TX, TY, D, stage_cy<TX, TY, D, Tc, MODE, FIRST, SUM>(), Tin, Tc, Tout, MODE, FIRST, MASK, CS,
                   SUM>(a, it, n, tile, rowl, pacc);
}

// Sum of v over the workgroup (xor shuffles within each wave, then the wave
// totals in wave order through LDS); thread 0 gets the result.  The caller's
// LDS buffer must be free: a barrier precedes its reuse.
template <int NT>
__device__ __forceinline__ double2 wg_sum(double2 v, double2 *lds) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        v.x += __shfl_xor(v.x, off);
        v.y += __shfl_xor(v.y, off);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double2 s = make_double2(0.0, 0.0);
    if (threadIdx.x == 0)
        for (int w = 0; w < (NT + 63) / 64; ++w) {
            s.x += lds[w].x;
            s.y += lds[w].y;
        }
    return s;
}

template <bool NTS, int TX, int TY, int D, class Tin, class Tc, class Tout, int MODE, bool FIRST, bool MASK = false,
          bool CS = false, int SUM = 0>
__global__ void __launch_bounds__((TX * TY / stage_cy<TX, TY, D, Tc, MODE, FIRST, SUM>()), 2)
    k_stencil(KParams a, GatherArgs g) {
    __shared__ typename CT<Tc>::c2 tile[2 * (TY + 8) * (TX + 8)];  // two plane buffers
    __shared__ int4 rowl[march_rows<TX, TY, D, stage_cy<TX, TY, D, Tc, MODE, FIRST, SUM>(),
                                    std::is_same<Tc, double>::value && stage_heavy(MODE, FIRST, SUM)>()];
    constexpr int NW = TX * TY / stage_cy<TX, TY, D, Tc, MODE, FIRST, SUM>() / 64;
    using Real = decltype(Tin{}.x);
    if ((unsigned)((int)blockIdx.x - g.at) < (unsigned)g.nblk) {
        // the projector gather of the same input, with the plane buffer as
        // its LDS: the first workgroups of a launch that is resident at once,
        // the last of a larger one.  A launch of its own before the stencil
        // cost 6-7 us on small and middle systems and 20 us on 16 atoms x 64
        // orbitals, all latency; here it hides under the marches (masked step
        // of 500 k points x 7 orbitals x 3 atoms 272 -> 245 us).  Short
        // marches in tiles of one or two waves don't hide it: there it stays
        // a launch of its own and nblk is 0.
        static_assert(sizeof(tile) >= kGatherSlots * 64 * sizeof(Tc), "gather sums fit the plane buffer");
        const int j = (int)blockIdx.x - g.at, chunk = j % g.nchunk, q = j / g.nchunk, atom = q / g.nct;
        gather_tile<NW, Real, Tc>(static_cast<const Real *>(a.in), g.ldo, g.ncols, g.atoms[atom], atom, q - atom * g.nct,
                                  g.idx, static_cast<const Tc *>(g.p), (Tc)g.h3, static_cast<Tc *>(g.D),
                                  reinterpret_cast<Tc *>(tile), chunk, g.nchunk, static_cast<Tc *>(g.P));
        return;
    }
    const int blk = xcd_remap((int)blockIdx.x - (g.at == 0 ? g.nblk : 0), (int)gridDim.x - g.nblk);
    int n, item;
    block_item(a, blk, &n, &item);
    // uniform by construction; saying so keeps the buffer resources in
    // scalar registers (no per-lane loop around each buffer instruction)
    n = __builtin_amdgcn_readfirstlane(n);
    item = __builtin_amdgcn_readfirstlane(item);
    double2 pacc = make_double2(0.0, 0.0);
    int4 it;
    if (a.ntx) {  // dense plan
        const int c = item / (a.ntx * a.nty), k = item - c * a.ntx * a.nty, ty = k / a.ntx;
        it = make_int4(k - ty * a.ntx, ty, c * a.ZC, min(a.nz, (c + 1) * a.ZC));
    } else {
        it = a.items[item];
    }
    march<NTS, TX, TY, D, Tin, Tc, Tout, MODE, FIRST, MASK, CS, SUM>(a, it, n, tile, rowl, pacc);
    if constexpr (SUM != 0) {
        // this workgroup's part of the sum, at a fixed place (so the final
        // sum has a fixed order): its place in the launch order for the pair
        // sum over all orbitals, {orbital, item} for the per-orbital sums
        const double2 s = wg_sum<TX * TY / stage_cy<TX, TY, D, Tc, MODE, FIRST, SUM>()>(pacc, reinterpret_cast<double2 *>(tile));
        if (threadIdx.x == 0)
            reinterpret_cast<double2 *>(a.pair_out)[SUM == SUM_PAIR ? blk : (int64_t)n * a.nitems + item] = s;
    }
}

// Persistent form over many independent systems (FP64).  The item list
// {tile, system, orbital} is cut into kBatchQueues contiguous segments of
// about equal work, one per XCD: a workgroup takes the next item of its own
// XCD's segment (workgroup b runs on XCD b mod 8) from that segment's
// counter as soon as it is free, so the items in flight on one XCD are
// neighbours in the list (neighbouring tiles of one system and orbital,
// which then share halo lines in that XCD's L2) however long each march is.
// A workgroup whose segment is used up takes items from the following
// segments in turn.  Each system's parameters come from sysp[system].
// ctr[q] counts the items taken from segment q, ctr[kBatchQueues] the
// workgroups done; the last workgroup out sets them all back to zero for
// the next launch (every workgroup has found every segment used up before
// it counts itself done, so no item is taken after the reset).
// Every stage of a product-form step is its own base (a first-type stage).
template <bool NTS, int TX, int TY, int D>
__global__ void __launch_bounds__((TX * TY / tile_cy(TX, TY, D, true, false)),
                                  TX == 16 && TY == 16 && D == 1 ? 3 : 2)
    k_stencil_batch(const KParams *__restrict__ sysp, const BatchItem *__restrict__ items,
                    const int32_t *__restrict__ seg, double cre, double cim, int32_t *ctr) {
    __shared__ double2 tile[2 * (TY + 8) * (TX + 8)];  // two plane buffers
    __shared__ int4 rowl[march_rows<TX, TY, D, tile_cy(TX, TY, D, true, false), false>()];
    __shared__ int32_t next;
    const int home = blockIdx.x % kBatchQueues;
    for (int j = 0; j < kBatchQueues; ++j) {
        const int q = (home + j) % kBatchQueues;
        const int32_t s0 = seg[q], s1 = seg[q + 1];
        for (;;) {
            if (threadIdx.x == 0) next = s0 + atomicAdd(&ctr[q], 1);
            __syncthreads();
            const int w = __builtin_amdgcn_readfirstlane(next);
            __syncthreads();  // every thread has read next before it is written again
            if (w >= s1) break;
            const BatchItem bi = items[w];
            KParams a = sysp[__builtin_amdgcn_readfirstlane(bi.sys)];
            a.cre = cre;
            a.cim = cim;
            a.row_slots = 0;  // rows from the table: the choice would cost registers here
            double2 unused = make_double2(0.0, 0.0);
            march<NTS, TX, TY, D, double2, double, double2, 1, true, false, false>(
                a, bi.tile, __builtin_amdgcn_readfirstlane(bi.ob), tile, rowl, unused);
            __syncthreads();  // the next item reuses the plane buffer
        }
    }
    if (threadIdx.x == 0) {
        __threadfence();  // this workgroup's last takes precede its count below
        if (atomicAdd(&ctr[kBatchQueues], 1) == (int)gridDim.x - 1) {
            for (int q = 0; q <= kBatchQueues; ++q) atomicExch(&ctr[q], 0);
        }
    }
}

// Complex-scaled Hamiltonians use the depth-1 pipelined march; other tile
// shapes are mapped to these (see launch_stencil).
template <bool NTS, int TX, int TY, int D>
int launch_fp64_cs(const StageArgs &a, const KParams &p, const GatherArgs &g, int nb, hipStream_t s) {
    constexpr int N1 = TX * TY / tile_cy(TX, TY, D, true, false), N2 = TX * TY / tile_cy(TX, TY, D, true, true);
    if (a.in_t != 0 || a.out_t != 0 || a.mask || a.pair_y) return RSG_EUNSUPPORTED;
    if (a.mode == 0 && a.dot == DOT_T)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 0, false, false, true, SUM_TDOT><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.mode == 0 && a.dot == DOT_ONLY)
        k_stencil<false, TX, TY, D, double2, double, double2, 0, false, false, true, SUM_ONLY><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.dot)
        return RSG_EUNSUPPORTED;
    else if (a.mode == 0)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 0, false, false, true><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.first)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 1, true, false, true><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else
        k_stencil<NTS, TX, TY, D, double2, double, double2, 1, false, false, true><<<nb + g.nblk, N2, 0, s>>>(p, g);
    return RSG_OK;
}

template <bool NTS, int TX, int TY, int D>
int launch_fp64(const StageArgs &a, const KParams &p, const GatherArgs &g, int nb, hipStream_t s) {
    constexpr int N1 = TX * TY / tile_cy(TX, TY, D, true, false), N2 = TX * TY / tile_cy(TX, TY, D, true, true);
    if (a.in_t != 0 || a.out_t != 0) return RSG_EUNSUPPORTED;
    if (a.pair_y && !(a.mode == 1 && a.first && !a.mask)) return RSG_EUNSUPPORTED;
    if (a.mode == 0 && a.dot == DOT_T)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 0, false, false, false, SUM_TDOT><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.mode == 0 && a.dot == DOT_H)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 0, false, false, false, SUM_HDOT><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.mode == 0 && a.dot == DOT_ONLY)
        k_stencil<false, TX, TY, D, double2, double, double2, 0, false, false, false, SUM_ONLY><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.dot)
        return RSG_EUNSUPPORTED;
    else if (a.mode == 0)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 0, false><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.pair_y)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 1, true, false, false, SUM_PAIR><<<nb + g.nblk, N2, 0, s>>>(p, g);
    else if (a.first)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 1, true><<<nb + g.nblk, N1, 0, s>>>(p, g);
    else if (a.mask)
        k_stencil<NTS, TX, TY, D, double2, double, double2, 1, false, true><<<nb + g.nblk, N2, 0, s>>>(p, g);
    else
        k_stencil<NTS, TX, TY, D, double2, double, double2, 1, false><<<nb + g.nblk, N2, 0, s>>>(p, g);
    return RSG_OK;
}

// Mixed path: FP32 arithmetic; the first stage reads complex128 psi and
// writes complex64, the middle stages complex64 to complex64 (each its own
// base), the last complex64 to complex128 with the complex128 base psi.
template <bool NTS, int TX, int TY, int D>
int launch_fp32(const StageArgs &a, const KParams &p, const GatherArgs &g, int nb, hipStream_t s) {
    constexpr int NT = TX * TY;
    if (a.mode != 1 || a.pair_y || a.dot) return RSG_EUNSUPPORTED;
    if (a.in_t == 0 && a.out_t == 1 && a.first)
        k_stencil<NTS, TX, TY, D, double2, float, float2, 1, true><<<nb + g.nblk, NT, 0, s>>>(p, g);
    else if (a.in_t == 1 && a.out_t == 1 && a.first)
        k_stencil<NTS, TX, TY, D, float2, float, float2, 1, true><<<nb + g.nblk, NT, 0, s>>>(p, g);
    else if (a.in_t == 1 && a.out_t == 0 && !a.first && a.mask)
        k_stencil<NTS, TX, TY, D, float2, float, double2, 1, false, true><<<nb + g.nblk, NT, 0, s>>>(p, g);
    else if (a.in_t == 1 && a.out_t == 0 && !a.first)
        k_stencil<NTS, TX, TY, D, float2, float, double2, 1, false><<<nb + g.nblk, NT, 0, s>>>(p, g);
    else
        return RSG_EUNSUPPORTED;
    return RSG_OK;
}

// grid < 0: return the number of resident workgroups of this kernel on the
// device (occupancy query, not allowed during graph capture); grid > 0:
// launch with that many persistent workgroups.
template <bool NTS, int TX, int TY, int D>
int launch_batch_inst(const KParams *sysp, const BatchItem *items, const int32_t *seg, int32_t nitems, double cre,
                      double cim, int32_t *ctr, int grid, hipStream_t s) {
    constexpr int NT = TX * TY / tile_cy(TX, TY, D, true, false);
    auto kern = k_stencil_batch<NTS, TX, TY, D>;
    if (grid < 0) {
        int per_cu = 0, dev = 0;
        hipDeviceProp_t prop;
        RSG_CHECK_HIP(hipGetDevice(&dev));
        RSG_CHECK_HIP(hipGetDeviceProperties(&prop, dev));
        RSG_CHECK_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, NT, 0));
        return std::max(1, per_cu) * prop.multiProcessorCount;
    }
    kern<<<(int)std::min<int64_t>(nitems, grid), NT, 0, s>>>(sysp, items, seg, cre, cim, ctr);
    return RSG_OK;
}

}  // namespace sk

// Tile shapes compiled into the library, {TX, TY, depth}: depth 1..2 is the
// pipelined march, depth 0 the lean one.  (Deeper pipelines and 1024-thread
// tiles are not compiled: their rings spill past the register limit.)
#define RSG_FP64_SHAPES(X) \
    X(8, 8, 1) X(8, 8, 2) X(16, 8, 1) X(16, 8, 2) X(32, 8, 1) X(32, 8, 2) X(16, 16, 1) \
    X(16, 16, 2) X(32, 16, 1) X(32, 16, 2) X(64, 8, 1) X(64, 8, 2) X(32, 16, 0) \
    X(32, 32, 1)
#define RSG_FP32_SHAPES(X) X(16, 8, 1) X(32, 8, 1) X(32, 8, 2) X(32, 16, 1) X(32, 16, 2) X(64, 8, 2)
#define RSG_CS_SHAPES(X) X(8, 8, 1) X(16, 8, 1) X(32, 8, 1) X(16, 16, 1) X(32, 16, 1)

// One stencil stage over nb workgroups with the compiled kernel for the
// tile shape and the stage's types (RSG_EUNSUPPORTED if there is none).
template <bool NTS>
int stencil_dispatch(const StageArgs &a, const KParams &p, const GatherArgs &g, const TileShape &shape, bool cs, int nb,
                     hipStream_t s) {
    int rc = RSG_EUNSUPPORTED;
    bool found = false;
#define RSG_TRY(X_, Y_, D_, FN)                                         \
    if (!found && shape.TX == X_ && shape.TY == Y_ && shape.PD == D_) { \
        found = true;                                                   \
        rc = sk::FN<NTS, X_, Y_, D_>(a, p, g, nb, s);                   \
    }
#define RSG_TRY64(X_, Y_, D_) RSG_TRY(X_, Y_, D_, launch_fp64)
#define RSG_TRY32(X_, Y_, D_) RSG_TRY(X_, Y_, D_, launch_fp32)
#define RSG_TRYCS(X_, Y_, D_) RSG_TRY(X_, Y_, D_, launch_fp64_cs)
    if (shape.B == 1) {
        if (cs) {
            RSG_CS_SHAPES(RSG_TRYCS)
        } else if (a.compute == 0) {
            RSG_FP64_SHAPES(RSG_TRY64)
        } else {
            RSG_FP32_SHAPES(RSG_TRY32)
        }
    }
#undef RSG_TRY64
#undef RSG_TRY32
#undef RSG_TRYCS
#undef RSG_TRY
    return rc;
}

// The persistent batched kernel for the tile shape: grid < 0 returns its
// resident workgroups on the device, grid > 0 launches it with that many
// (RSG_EUNSUPPORTED if the shape is not compiled).
template <bool NTS>
int batch_dispatch(const TileShape &shape, const KParams *sysp, const BatchItem *items, const int32_t *seg,
                   int32_t nitems, double cre, double cim, int32_t *ctr, int grid, hipStream_t s) {
    int rc = RSG_EUNSUPPORTED;
    bool found = false;
#define RSG_TRY_B(X_, Y_, D_)                                                                             \
    if (!found && shape.TX == X_ && shape.TY == Y_ && shape.PD == D_) {                                   \
        found = true;                                                                                     \
        rc = sk::launch_batch_inst<NTS, X_, Y_, D_>(sysp, items, seg, nitems, cre, cim, ctr, grid, s);    \
    }
    if (shape.B == 1) { RSG_FP64_SHAPES(RSG_TRY_B) }
#undef RSG_TRY_B
    return rc;
}

// instantiated in stencil_inst.hip (false) and stencil_inst_nt.hip (true)
#define RSG_STENCIL_INST(EXT, NTS_)                                                                           \
    EXT template int stencil_dispatch<NTS_>(const StageArgs &, const KParams &, const GatherArgs &,            \
                                            const TileShape &, bool, int, hipStream_t);                       \
    EXT template int batch_dispatch<NTS_>(const TileShape &, const KParams *, const BatchItem *,               \
                                          const int32_t *, int32_t, double, double, int32_t *, int, hipStream_t);
RSG_STENCIL_INST(extern, false)
RSG_STENCIL_INST(extern, true)

}  // namespace rsg
