// Host side of the stencil stage: the tile shapes compiled into the library,
// the default shape for a grid, the kernel parameters of a stage and the
// launch (kernels and their dispatch over tile shapes in stencil_kernels.h).
// A stage whose output is at least kNtStoreBytes runs the kernel set with
// non-temporal output stores: such an output is not read again before it
// has left every cache, and streaming it past L2 leaves L2 to the input
// planes and halo lines that neighbouring tiles still read.
#include "stencil_kernels.h"

namespace rsg {

std::vector<TileShape> tile_candidates(int compute) {
    std::vector<TileShape> v;
#define RSG_ADD(X_, Y_, D_)                \
    {                                      \
        TileShape sh{1, X_, Y_, 0};        \
        sh.PD = D_;                        \
        v.push_back(sh);                   \
    }
    if (compute == 0) {
        RSG_FP64_SHAPES(RSG_ADD)
    } else {
        RSG_FP32_SHAPES(RSG_ADD)
    }
#undef RSG_ADD
    return v;
}

// Tile and z-chunk of a launch nobody tuned, by its points times orbitals.
// A tile wants to be wide (halo lines per column: 32 x 8 1.5, 16 x 16 1.5,
// 32 x 16 1.0) but a launch also wants enough workgroups: below 4 M values
// the widest tiles leave compute units idle or pay for empty columns, and
// z is cut so that about `items` workgroups start (768: the 256 units x 3
// resident 32 x 8 workgroups, one round) with no chunk shorter than `zmin`
// planes (each chunk re-reads 8 planes, which such batches find in
// cache).  Chunks are cut equal, at the same planes for every tile (ZM = 2),
// and two orbitals of a tile run side by side (BO = 2, V shared).
// The lines come from timing every compiled tile with chunks of 1..96 planes
// on 207 FP64 and 214 mixed systems (spheres 27 to 181 points across and
// cubes of 20^3 to 120^3, 1..64 orbitals, both storages), below 2 M values in
// captured graphs, so that the host does not hide in the figures.  Time over
// that system's best, geometric mean, FP64: this table 1.01-1.08 by size (worst
// system 1.25), the fixed 32 x 16 / 32 x 8 / 16 x 8 choice before it 1.03-1.26
// (at 4-8 M values 16 x 8 tiles over the whole z-range 1.26); mixed 1.01-1.06
// against 1.02-1.39.
namespace {
struct ShapeRule {
    double below;  // points x orbitals
    int TX, TY, PD, items, zmin;
    double fill;  // share of a sphere's tile columns x chunks that hold points, as counted towards items
};
constexpr ShapeRule kRules64[] = {
    {1e5, 32, 8, 1, 768, 1, 1.0},    // latency: as many short marches as fit at once
    {2.5e5, 32, 8, 1, 768, 2, 1.0},
    {1e6, 32, 8, 1, 768, 4, 0.75},
    {4e6, 32, 8, 1, 1536, 6, 1.0},   // two rounds
    {1e7, 16, 16, 1, 4096, 12, 1.0}, // 3 workgroups a unit, still cache resident
    {4e7, 32, 16, 1, 6144, 32, 1.0}, // memory bound: least halo per column
    {1e300, 32, 16, 1, 8192, 48, 1.0},
};
// FP32 below 1 M values: 16 x 8 tiles time alike (1.05), but their workgroups
// are 128 threads and the projector gather that rides in the launch takes
// twice as long on two waves (38^3 x 7, one atom, a step 93 us against 66).
constexpr ShapeRule kRules32[] = {
    {1e5, 32, 8, 1, 768, 1, 1.0},
    {2.5e5, 32, 8, 1, 768, 2, 1.0},
    {1e6, 32, 8, 1, 1024, 2, 0.75},
    {4e6, 16, 8, 1, 3072, 8, 1.0},
    {1e7, 16, 8, 1, 6144, 8, 1.0},
    {4e7, 32, 8, 2, 8192, 24, 1.0},
    {1e300, 32, 16, 1, 4096, 64, 1.0},
};
}  // namespace

TileShape default_shape(const Grid &g, int64_t nst, int compute) {
    const double orbitals = (double)std::max<int64_t>(nst, 1), work = (double)g.npts * orbitals;
    const ShapeRule *r = compute == 0 ? kRules64 : kRules32;
    while (work >= r->below) ++r;
    TileShape sh{1, r->TX, r->TY, 0};
    sh.PD = r->PD;
    sh.BO = 2;
    const double tiles = (double)((g.n[0] + r->TX - 1) / r->TX) * ((g.n[1] + r->TY - 1) / r->TY) * orbitals *
                         (g.shape == RSG_BOX_SPHERE ? r->fill : 1.0);
    const double zc = std::max<double>(r->zmin, g.n[2] * tiles / r->items);
    const int chunks = std::max(1, (int)std::lround(g.n[2] / zc));
    sh.ZC = (g.n[2] + chunks - 1) / chunks;
    sh.ZM = chunks > 1 ? 2 : 0;
    return sh;
}

TileShape Ham::tile_for(int64_t nst, int compute) const {
    auto it = tiles.find(std::make_pair(nst, compute));
    if (it != tiles.end()) return it->second;
    return default_shape(*g, nst, compute);
}

KParams make_params(const Ham &H, const StageArgs &a, const TileShape &shape, const TilePlan *plan) {
    const Grid &g = *H.g;
    KParams p;
    p.in = a.in;
    p.base = a.base;
    p.out = a.out;
    p.items = plan ? plan->items : nullptr;
    p.rows = g.rows;
    p.zeros = g.zeros;
    p.V = a.compute == 0 ? (const void *)H.V : (const void *)H.V32;
    p.field_dev = a.field_dev;
    p.mask = a.mask;
    p.pair_y = a.pair_y;
    p.pair_out = a.pair_out;
    p.nst = a.nst;
    p.ldp = a.ldp;
    p.np = g.np;
    p.Vim = H.vim;
    if (H.cs_theta != 0) {
        // kin e^{-2 i theta}
        p.kin_h2 = H.kin * std::cos(2.0 * H.cs_theta) / (g.h * g.h);
        p.kin_h2_im = -H.kin * std::sin(2.0 * H.cs_theta) / (g.h * g.h);
    } else {
        p.kin_h2 = H.kin / (g.h * g.h);
        p.kin_h2_im = 0.0;
    }
    p.field = a.field;
    p.h = g.h;
    // box centre along the field axis (one scalar, so that a register copy
    // of these parameters needs no indexed private-memory array)
    p.off_axis = H.axis >= 0 ? 0.5 * (double)(g.n[H.axis] - 1) : 0.0;
    p.cre = a.cre;
    p.cim = a.cim;
    p.nitems = plan ? plan->nitems : 0;
    p.block_order = shape.BO;
    p.ny = g.n[1];
    p.nz = g.n[2];
    p.axis = H.axis;
    p.align = g.align;
    p.ntx = plan ? plan->ntx : 0;
    p.nty = plan ? plan->nty : 0;
    p.ZC = plan ? plan->ZC : 0;
    const bool box = g.shape == RSG_BOX_CUBE;
    p.row_slots = box ? (g.n[0] + g.align - 1) / g.align * g.align : 0;
    p.row_len = box ? g.n[0] : 0;
    return p;
}

TileShape launch_shape(const Ham &H, const TileShape &tile) {
    TileShape shape = tile;
    if (H.complex_scaled()) {
        bool have = false;
#define RSG_CS_HAVE(X_, Y_, D_) have = have || (shape.TX == X_ && shape.TY == Y_);
        RSG_CS_SHAPES(RSG_CS_HAVE)
#undef RSG_CS_HAVE
        shape.PD = 1;
        if (!have) {
            shape.TX = 16;
            shape.TY = 8;
        }
    }
    if (shape.ZC <= 0) shape.ZC = H.g->n[2];
    return shape;
}

int64_t stencil_blocks(const Ham &H, int64_t nst, int compute, hipStream_t s) {
    int err = RSG_OK;
    const TilePlan *plan = H.g->plan(launch_shape(H, H.tile_for(nst, compute)), s, &err);
    if (!plan) return err;
    return (int64_t)plan->nitems * nst;
}

int launch_stencil(const Ham &H, const StageArgs &a, const TileShape &tile, hipStream_t s) {
    const Grid &g = *H.g;
    int err = RSG_OK;
    const bool cs = H.complex_scaled();
    if (cs && a.compute != 0) {
        set_error("stencil: a complex-scaled Hamiltonian needs the FP64 path");
        return RSG_EUNSUPPORTED;
    }
    const TileShape shape = launch_shape(H, tile);
    const TilePlan *plan = const_cast<Grid &>(g).plan(shape, s, &err);
    if (!plan) return err;
    if (plan->nitems == 0 || a.nst == 0) return RSG_OK;
    if (g.np >= (int64_t)(OOB / 16)) {
        set_error("stencil: grids of 2^27 points or more are not supported");
        return RSG_EUNSUPPORTED;
    }
    const KParams p = make_params(H, a, shape, plan);
    const int64_t nb64 = (int64_t)plan->nitems * a.nst;
    if (nb64 > INT32_MAX) {
        set_error("stencil launch too large");
        return RSG_EUNSUPPORTED;
    }
    const int nb = (int)nb64;
    // an output that no cache level holds is streamed past L2
    const bool nt = (double)a.nst * (double)g.np * (a.out_t == 0 ? 16.0 : 8.0) >= kNtStoreBytes;
    // the projector gather's workgroups: first in a launch that is resident at
    // once (they take as long as a short march), last in a larger one, where
    // they fill compute units that the last marches leave idle
    GatherArgs ga = gather_args(H, a.compute, a.nst, a.ldp, a.D);
    ga.at = nb > 4096 ? nb : 0;
    if ((int64_t)nb + ga.nblk > INT32_MAX) {
        set_error("stencil launch too large");
        return RSG_EUNSUPPORTED;
    }
    timing_before(s);
    const int rc =
        nt ? stencil_dispatch<true>(a, p, ga, shape, cs, nb, s) : stencil_dispatch<false>(a, p, ga, shape, cs, nb, s);
    timing_after(s);
    if (rc == RSG_EUNSUPPORTED) {
        set_error("stencil: unsupported tile %dx%dx%d depth %d for this precision", shape.B, shape.TX,
                  shape.TY, shape.PD);
        return rc;
    }
    RSG_CHECK_HIP(hipGetLastError());
    return RSG_OK;
}

int stencil_batch_grid(const TileShape &shape, bool first, bool nt) {
    return nt ? batch_dispatch<true>(shape, first, nullptr, nullptr, nullptr, 0, 0.0, 0.0, nullptr, -1, nullptr)
              : batch_dispatch<false>(shape, first, nullptr, nullptr, nullptr, 0, 0.0, 0.0, nullptr, -1, nullptr);
}

int launch_stencil_batch(const TileShape &shape, int mode, bool first, bool nt, const KParams *sysp,
                         const BatchItem *items, const int32_t *seg, int32_t nitems, double cre, double cim,
                         int32_t *ctr, int grid, hipStream_t s) {
    if (nitems == 0) return RSG_OK;
    if (mode != 1) {
        set_error("batched stencil: only Horner stages are batched");
        return RSG_EUNSUPPORTED;
    }
    if (grid <= 0 || !ctr || !seg) {
        set_error("batched stencil: need a persistent grid size > 0, work counters and segment bounds");
        return RSG_EINVAL;
    }
    timing_before(s);
    const int rc = nt ? batch_dispatch<true>(shape, first, sysp, items, seg, nitems, cre, cim, ctr, grid, s)
                      : batch_dispatch<false>(shape, first, sysp, items, seg, nitems, cre, cim, ctr, grid, s);
    timing_after(s);
    if (rc != RSG_OK) {
        if (rc == RSG_EUNSUPPORTED)
            set_error("batched stencil: unsupported tile %dx%dx%d depth %d", shape.B, shape.TX, shape.TY, shape.PD);
        return rc;
    }
    RSG_CHECK_HIP(hipGetLastError());
    return RSG_OK;
}

}  // namespace rsg
