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
// the widest tiles leave compute units idle or pay for empty columns, and z is
// cut into as many equal chunks, at the same planes for every tile (ZM = 2), as
// start at most `items` workgroups and hold at least `zmin` planes (each chunk
// re-reads 8 planes, which such batches find in cache).  There the workgroups
// are counted as the plan lists them: the best chunk of a small launch is
// the shortest whose workgroups are all resident at once (3 of 256 threads or 6
// of 128 on each of 256 units: 768, 1536), and one more round costs up to 1.2
// times as long.  Larger launches take several rounds anyway; they count every
// tile of the box in every chunk and round the number of chunks.
// All tiles of an orbital run before the next orbital's (BO = 1) in these:
// a pair of orbitals side by side reads V half as often, which batches that stay in
// cache do not feel, but spreads an orbital's halos over more XCDs (45 points
// across x 3 orbitals, 32 x 8: 6.97 us a stage in pairs, 6.2 without).
// The lines come from timing every compiled tile, chunks of 1..64 planes and
// both orders on 372 FP64 and 302 mixed systems of 1e4 to 3.5e7 values (spheres 27
// to 149 points across, cubes of 20^3 to 118^3, 1..64 orbitals, both storages, with
// and without projectors) in captured graphs.
namespace {
struct ShapeRule {
    double below;  // points x orbitals
    int TX, TY, PD, items, zmin, BO;
    bool counted;  // items: the plan's, else every tile of the box
};
constexpr ShapeRule kRules64[] = {
    {1e6, 32, 8, 1, 768, 1, 1, true},     // one round
    {2e6, 32, 8, 1, 1536, 6, 1, true},
    {4e6, 32, 8, 1, 2048, 8, 1, true},
    {1e7, 16, 16, 1, 4096, 12, 2, false},  // 3 workgroups a unit, still cache resident
    {4e7, 32, 16, 1, 6144, 32, 2, false},  // memory bound: least halo per column
    {1e300, 32, 16, 1, 8192, 48, 2, false},
};
// Spheres without projectors: 16-wide tiles leave fewer columns of the rim
// empty (45 points across x 13 orbitals 12.9 us a stage, 14.8 in 32 x 8; boxes
// take 1.04 times as long in 16 x 8).
constexpr ShapeRule kSphere64[] = {
    {2.5e5, 32, 8, 1, 768, 1, 1, true},
    {1e6, 16, 8, 1, 1536, 3, 1, true},
    {2e6, 16, 8, 1, 3072, 4, 1, true},
    {4e6, 16, 8, 1, 4096, 4, 1, true},
    {1e7, 16, 16, 1, 4096, 12, 2, false},
    {4e7, 32, 16, 1, 6144, 32, 2, false},
    {1e300, 32, 16, 1, 8192, 48, 2, false},
};
constexpr ShapeRule kRules32[] = {
    {1e5, 32, 8, 1, 512, 1, 1, true},
    {2.5e5, 16, 8, 1, 1024, 1, 1, true},
    {1e6, 16, 8, 1, 2048, 3, 1, true},
    {2e6, 16, 8, 1, 2048, 4, 1, true},
    {1e7, 16, 8, 1, 4096, 8, 1, true},
    {4e7, 32, 8, 2, 8192, 24, 2, false},
    {1e300, 32, 16, 1, 4096, 64, 2, false},
};
// With projectors their gather rides in the launch with the tile's own threads,
// and on the two waves of a 16 x 8 tile it takes twice as long (FP32, 41^3 x 18
// orbitals, two atoms: a stage 25.8 us against 21.3), so that these take wider
// tiles and longer chunks.
constexpr ShapeRule kRules32p[] = {
    {2.5e5, 32, 8, 1, 512, 1, 1, true},
    {1e6, 32, 8, 1, 768, 4, 1, true},
    {2e6, 32, 8, 1, 2048, 4, 1, true},
    {4e6, 32, 8, 2, 2048, 6, 1, true},
    {1e7, 32, 8, 2, 3072, 8, 1, true},
    {4e7, 32, 8, 2, 8192, 24, 2, false},
    {1e300, 32, 16, 1, 4096, 64, 2, false},
};

TileShape shape_by_rule(const Grid &g, int64_t nst, int compute, bool projectors) {
    const int nz = g.n[2];
    const double orbitals = (double)std::max<int64_t>(nst, 1), work = (double)g.npts * orbitals;
    const ShapeRule *r = compute != 0 ? (projectors ? kRules32p : kRules32)
                         : g.shape == RSG_BOX_SPHERE && !projectors ? kSphere64
                                                                    : kRules64;
    while (work >= r->below) ++r;
    TileShape sh{1, r->TX, r->TY, nz};
    sh.PD = r->PD;
    sh.BO = r->BO;
    if (r->counted) {
        const TileExtents &e = g.extents(r->TX, r->TY);
        // (a tile has at most one item a chunk: so many chunks fit uncounted)
        const int sure = (int)std::min<double>(nz, r->items / (orbitals * (double)e.zlo.size()));
        for (int chunks = 1; chunks <= nz; ++chunks) {
            const int zc = (nz + chunks - 1) / chunks;
            int64_t items = 0;
            for (size_t k = 0; chunks > sure && k < e.zlo.size(); ++k)
                if (e.zhi[k] >= e.zlo[k]) items += e.zhi[k] / zc - e.zlo[k] / zc + 1;
            if (zc < r->zmin || (double)items * orbitals > r->items) break;
            sh.ZC = zc;
        }
    } else {
        const double tiles = (double)((g.n[0] + r->TX - 1) / r->TX) * ((g.n[1] + r->TY - 1) / r->TY) * orbitals;
        const double zc = std::max<double>(r->zmin, nz * tiles / r->items);
        const int chunks = std::max(1, (int)std::lround(nz / zc));
        sh.ZC = (nz + chunks - 1) / chunks;
    }
    sh.ZM = sh.ZC < nz ? 2 : 0;
    return sh;
}
}  // namespace

TileShape default_shape(const Grid &g, int64_t nst, int compute, bool projectors) {
    const auto key = std::make_tuple(nst, compute, projectors);
    try {
        {
            std::lock_guard<std::mutex> lk(g.lazy_mu);
            const auto it = g.defaults.find(key);
            if (it != g.defaults.end()) return it->second;
        }
        const TileShape sh = shape_by_rule(g, nst, compute, projectors);
        std::lock_guard<std::mutex> lk(g.lazy_mu);
        return g.defaults[key] = sh;
    } catch (const std::bad_alloc &) {
        return TileShape{1, 32, 8, g.n[2]};
    }
}

TileShape Ham::tile_for(int64_t nst, int compute) const {
    auto it = tiles.find(std::make_pair(nst, compute));
    if (it != tiles.end()) return it->second;
    return default_shape(*g, nst, compute, natoms > 0);
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

// Whether the projector gather rides in the launch of a tile: a workgroup of few
// waves takes long for its part (19 us on two, 32 on one, for two atoms of 1,200
// points), which hides only behind marches that last as long.  23^3 x 2 orbitals, a
// stage in 8 x 8 tiles with chunks of 2 planes: 32.4 us riding, 14.6 with a gather
// launch of 16 waves before it, with chunks of 8 17.2; 16 x 8 with 2 planes 19.7 and
// 14.4.  With marches of 49 planes and more riding leads in 8 x 8 (34.3 and 40.6
// us), of 23 and more in 16 x 8 (19.4 and 24.8).
bool gather_rides(const TileShape &s) { return s.TX * s.TY >= 256 || s.TX * s.TY * s.ZC >= 2048; }

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
    if (!gather_rides(shape) && a.in_t <= a.compute) {
        const int rc = launch_kb_gather(ga, a.in, a.in_t, a.compute, s);
        if (rc) return rc;
        ga = GatherArgs{};
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

int stencil_batch_grid(const TileShape &shape, bool nt) {
    return nt ? batch_dispatch<true>(shape, nullptr, nullptr, nullptr, 0, 0.0, 0.0, nullptr, -1, nullptr)
              : batch_dispatch<false>(shape, nullptr, nullptr, nullptr, 0, 0.0, 0.0, nullptr, -1, nullptr);
}

int launch_stencil_batch(const TileShape &shape, bool nt, const KParams *sysp, const BatchItem *items,
                         const int32_t *seg, int32_t nitems, double cre, double cim, int32_t *ctr, int grid,
                         hipStream_t s) {
    if (nitems == 0) return RSG_OK;
    if (grid <= 0 || !ctr || !seg) {
        set_error("batched stencil: need a persistent grid size > 0, work counters and segment bounds");
        return RSG_EINVAL;
    }
    timing_before(s);
    const int rc = nt ? batch_dispatch<true>(shape, sysp, items, seg, nitems, cre, cim, ctr, grid, s)
                      : batch_dispatch<false>(shape, sysp, items, seg, nitems, cre, cim, ctr, grid, s);
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
