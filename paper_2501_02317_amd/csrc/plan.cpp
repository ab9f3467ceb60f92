#include "plan.h"

#include <algorithm>
#include <cmath>
#include <tuple>

#include "hydro.h"

namespace hydro {

Tile default_tile(const Geo& g, int precision, int mode) {
    Tile t;
    if (mode == MODE_VL2_PRED_C || mode == MODE_VL2_CORR_C) {
        // the one tile of the refined mesh's van Leer stages
        t.tx = g.ndim == 3 ? 32 : 64;
        t.ty = g.ndim == 3 ? 8 : 1;
    } else if (g.ndim == 3) {
        // From a sweep at 256^3: 32 x 16 halves the share of halo cells and
        // extra faces where the occupancy allows it; 32 x 8 where a larger
        // work-group would cost occupancy (the FP64 kernels).  16 x 16 is 5-7 %
        // behind in the mixed kernels on a mesh that each fills (256^3 339 +
        // 444 against 362 + 476 us a step) and even in FP64 (a step of 128^3,
        // 192^3, 256^3 and 384^3 within 2 %, both integrators: 256^3 535 + 648
        // against 541 + 646); it takes over where it pads less: 48^3 mixed 28
        // against 31 us a step, 101 x 75 x 50 FP64 57 against 65 us.
        const bool narrow = precision == 0;
        auto padded = [&](int tx, int ty) {
            return (double)((g.n[0] + tx - 1) / tx * tx) * ((g.n[1] + ty - 1) / ty * ty);
        };
        t.tx = 32;
        t.ty = narrow ? 8 : 16;
        if (1.04 * padded(16, 16) < padded(t.tx, t.ty)) t.tx = t.ty = 16;
    } else if (g.ndim == 2) {
        // the row width with the least padding, each row segment's halo and
        // extra face counted as 24 cells (they take a wave of the work-group
        // about a third of a plane): 256 for wide rows, 128 for rows of 384
        t.tx = 256;
        t.ty = 1;
        auto cost = [&](int tx) { return (double)((g.n[0] + tx - 1) / tx) * (tx + 24); };
        for (int tx = 128; tx >= 64; tx /= 2)
            if (cost(tx) < cost(t.tx)) t.tx = tx;
    } else {
        t.tx = 64;
        t.ty = 1;
    }
    // chunk length chosen at launch (auto_kz)
    t.kz = g.ndim == 1 ? 1 : 0;
    return t;
}

bool tile_supported(int ndim, const Tile& t) {
    if (t.kz < 0 || (t.kz == 0 && ndim == 1)) return false;
    if (ndim == 3)
        return (t.tx == 32 && t.ty == 8) || (t.tx == 64 && t.ty == 8) || (t.tx == 16 && t.ty == 16) ||
               (t.tx == 32 && t.ty == 16);
    return t.ty == 1 && (t.tx == 64 || t.tx == 128 || t.tx == 256);
}

int tile_candidates(const Geo& g, Tile* out, int max) {
    static const int shapes3[4][2] = {{32, 8}, {64, 8}, {16, 16}, {32, 16}};
    static const int shapes12[4][2] = {{64, 1}, {128, 1}, {256, 1}, {0, 0}};
    static const int kzs[5] = {0, 8, 16, 32, 64};  // 0: automatic
    const int(*shapes)[2] = g.ndim == 3 ? shapes3 : shapes12;
    int n = 0;
    for (int s = 0; s < (g.ndim == 3 ? 4 : 3); ++s) {
        // in 1-D and 2-D a row wider than twice the mesh only idles threads
        if (g.ndim < 3 && s > 0 && shapes[s][0] >= 2 * g.n[0]) continue;
        for (int q = 0; q < (g.ndim == 1 ? 1 : 5); ++q) {
            const int kz = g.ndim == 1 ? 1 : kzs[q];
            if (q > 1 && kzs[q - 1] >= g.n[2]) break;  // same chunks as the previous kz
            if (n < max) {
                out[n].tx = shapes[s][0];
                out[n].ty = shapes[s][1];
                out[n].kz = kz;
            }
            ++n;
        }
    }
    return n;
}

int balanced_kz(int n2, int kz) {
    kz = kz < 1 ? 1 : (kz > n2 ? n2 : kz);
    const int chunks = (n2 + kz - 1) / kz;
    return (n2 + chunks - 1) / chunks;
}

// The chunk length that a launch over the columns m[0 .. n) takes least time
// with, by a model of the march: a work-group spends kz planes and a lead of
// about two planes more (three in 2-D: the start of the z pipeline), and a
// plane takes 1 + (w - 1)/3 with 4 w waves resident on the CU.  Fitted to
// sweeps of both precisions and integrators from 32^3 to 160^3 and 64^2 to
// 4096 x 1024: a plane's time is 2.6 us with four waves on a CU and 4.1 us
// with twelve (mixed 3-D), so small meshes want a work-group per plane or two
// (48^3 mixed: a step 102 us in chunks of 16, 28 us in chunks of 1-2; 256^2
// FP64 89 and 21 us), and a last round of a few work-groups costs as much as a
// full one (160^3 mixed: 316 us with 800 work-groups on 768 places, 225 us
// with 700) -- unless each XCD has a block of its own, whose columns' shorter
// last chunks come last and two deep beside the others (in eight blocks, with
// the rule and without: 192^3 mixed a step 350 and 362 us, van Leer 292 and
// 301 us -- 576 work-groups in chunks of 28 and 12 on 512 places, or 432 equal
// ones; 160^3 FP64 311 and 320 us; 224^3 mixed and 192^3 and 256^3 FP64 even).
int auto_kz(int ndim, const Slots& sl, const MarchCols* m, int n, double* time) {
    if (time) *time = 0.0;
    if (ndim == 1) return 1;
    int most = 1;
    for (int i = 0; i < n; ++i) most = m[i].n2 > most ? m[i].n2 : most;
    most = most > kMaxAutoKz ? kMaxAutoKz : most;
    if (sl.cus < 1 || sl.per_cu < 1) return most < 32 ? most : 32;
    const double lead = ndim == 3 ? 2.0 : 3.0;
    const long long slots = (long long)sl.cus * sl.per_cu;
    auto plane = [&](long long wgs) {
        const double w = (double)((wgs + sl.cus - 1) / sl.cus) * sl.waves / 4.0;
        return w > 1.0 ? 1.0 + (w - 1.0) / 3.0 : 1.0;
    };
    const bool xcd = n == 1 && m[0].per_xcd;
    int best = most;
    double least = -1.0;
    for (int kz = most, next; kz >= 1; kz = next) {
        // with the same chunks per column the shortest length is the best (the
        // last chunk alone may still matter to per_xcd)
        int same = xcd ? kz : 1;
        long long wgs = 0;
        for (int i = 0; i < n; ++i) {
            const int chunks = (m[i].n2 + kz - 1) / kz, shortest = (m[i].n2 + chunks - 1) / chunks;
            wgs += m[i].cols * chunks;
            same = shortest > same ? shortest : same;
        }
        kz = same;
        next = kz - 1;
        const long long full = wgs / slots, rest = wgs % slots;
        double t = (kz + lead) * (full * plane(slots) + (rest ? plane(rest) : 0.0));
        if (xcd && full == 1 && rest > 0 && 2 * slots + m[0].cols >= 2 * wgs) {
            const int last = m[0].n2 - (m[0].n2 - 1) / kz * kz;
            t = std::fmin(t, plane(slots) * std::fmax(kz + lead, 2.0 * (last + lead)));
        }
        if (least < 0.0 || t <= least) {
            least = t;
            best = kz;
        }
    }
    if (time) *time = least;
    return best;
}

void plan_tiles(const Geo& g, const Tile& t, int& tiles_x, int& tiles_y, int& chunks_z, int& kz) {
    tiles_x = (g.n[0] + t.tx - 1) / t.tx;
    tiles_y = (g.n[1] + t.ty - 1) / t.ty;
    kz = t.kz < 1 ? 1 : (t.kz > g.n[2] ? g.n[2] : t.kz);
    chunks_z = (g.n[2] + kz - 1) / kz;
}

// ------------------------------------------------------------------ batches

namespace {

// Tile rules of the batch autotuner for members of one or two dimensions:
// a row width for every such member (0: the member's own) and a chunk length
// (-1: the member's own, 0: the automatic one of its group).  Rule 0
// keeps every member's tile.  3-D members keep their tiles.
struct BatchRule {
    int tx, kz;
};
constexpr BatchRule kBatchRules[] = {{0, -1}, {64, -1}, {128, -1}, {256, -1}, {0, 16},   {64, 16},
                                     {128, 16}, {0, 32}, {64, 32},   {128, 32},  {0, 64},  {64, 64}};
static_assert(sizeof(kBatchRules) / sizeof(kBatchRules[0]) == kNumBatchRules, "rules");

// The columns of members idx[0 .. n) in tile t, and the automatic chunk length
// and modelled time of a launch over them (a launch of its own counts two
// planes; a tile's halo and extra faces as in default_tile).
int batch_kz(const std::vector<int>& idx, const std::vector<PlanMember>& m, const Tile& t, Residency residency,
             double* time = nullptr) {
    std::vector<MarchCols> cols;  // of one length each
    for (int i : idx) {
        const Geo& g = m[i].geo;
        int tx, ty, cz, kz;
        plan_tiles(g, t, tx, ty, cz, kz);
        size_t k = 0;
        while (k < cols.size() && cols[k].n2 != g.n[2]) ++k;
        if (k == cols.size()) cols.push_back({0, g.n[2], false});
        cols[k].cols += (long long)tx * ty;
    }
    const PlanMember& h = m[idx[0]];
    const int mode = h.integrator == HYDRO_VL2 ? MODE_VL2_CORR : MODE_STAGE2;
    const Slots sl = residency(h.geo.ndim, h.precision, mode, t);
    const int kz = auto_kz(h.geo.ndim, sl, cols.data(), (int)cols.size(), time);
    if (time) {
        const double wide = h.geo.ndim == 3 ? (t.tx * t.ty > 256 ? 1.0 : 1.08) : 1.0 + 24.0 / t.tx;
        *time = 2.0 + *time * wide;
    }
    return kz;
}

// One tile for the members (of one ndim, precision and integrator) that have
// the default ones, where their launches' modelled times add up to more than
// that of one launch with it: a group's last work-groups leave the chip idle,
// and a stage of 16-30 us is a good part launch (48 ragged 2-D meshes alone:
// 7.27 ms in three groups, 5.95 ms in one of width 128, 6.08 of 64).
void share_tile(const std::vector<int>& idx, const std::vector<PlanMember>& m, Residency residency,
                std::vector<Tile>& tiles) {
    if (idx.empty()) return;
    if (m[idx[0]].geo.ndim == 1) return;
    std::vector<Tile> kinds;
    std::vector<std::vector<int>> of;
    for (int i : idx) {
        size_t k = 0;
        while (k < kinds.size() && (kinds[k].tx != tiles[i].tx || kinds[k].ty != tiles[i].ty)) ++k;
        if (k == kinds.size()) {
            kinds.push_back(tiles[i]);
            of.push_back({});
        }
        of[k].push_back(i);
    }
    if (kinds.size() < 2) return;
    double own = 0.0;
    for (size_t k = 0; k < kinds.size(); ++k) {
        double t = 0.0;
        batch_kz(of[k], m, kinds[k], residency, &t);
        own += t;
    }
    int best = -1;
    for (size_t k = 0; k < kinds.size(); ++k) {
        double t = 0.0;
        batch_kz(idx, m, kinds[k], residency, &t);
        if (t < own) {
            own = t;
            best = (int)k;
        }
    }
    if (best >= 0)
        for (int i : idx) tiles[i] = kinds[best];
}

}  // namespace

Tile rule_tile(const PlanMember& m, int rule) {
    Tile t = m.tile;
    if (m.geo.ndim == 3 || rule <= 0 || rule >= kNumBatchRules) return t;
    if (kBatchRules[rule].tx > 0) t.tx = kBatchRules[rule].tx;
    if (kBatchRules[rule].kz >= 0) t.kz = kBatchRules[rule].kz;
    return t;
}

// Members grouped by (ndim, precision, tile): each group's descriptors and
// work-groups are contiguous in their tables, members in the caller's order
// within a group.  Member i runs tile rule_tile(m[i], rule); members of the
// default tiles may share one (share_tile) where the rule keeps their tiles:
// under every rule in 3-D, so that what a rule leaves is what was timed under
// it.
bool plan_layout(const std::vector<PlanMember>& m, int rule, Residency residency, BatchLayout& L) {
    const int n = (int)m.size();
    std::vector<int> order(n);
    std::vector<Tile> tiles(n);
    for (int i = 0; i < n; ++i) tiles[i] = rule_tile(m[i], rule);
    for (int c = 0; c < 16; ++c) {
        std::vector<int> same;
        for (int i = 0; i < n; ++i)
            if ((rule == 0 || m[i].geo.ndim == 3) && !m[i].tile_set &&
                c == 4 * m[i].geo.ndim + 2 * (m[i].precision == HYDRO_MIXED) + (m[i].integrator == HYDRO_VL2))
                same.push_back(i);
        share_tile(same, m, residency, tiles);
    }
    L.tiling.resize(n);
    for (int i = 0; i < n; ++i) {
        MemberTiling& d = L.tiling[i];
        plan_tiles(m[i].geo, tiles[i], d.tiles_x, d.tiles_y, d.chunks_z, d.kz);
        order[i] = i;
    }
    auto key = [&](int i) {
        return std::make_tuple(m[i].geo.ndim, m[i].precision, m[i].integrator, tiles[i].tx, tiles[i].ty);
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return key(a) < key(b); });
    // automatic chunk lengths: one per group, for the columns of all its members
    for (int i0 = 0, i1 = 0; i0 < n; i0 = i1) {
        std::vector<int> aut;
        for (i1 = i0; i1 < n && key(order[i1]) == key(order[i0]); ++i1)
            if (tiles[order[i1]].kz == 0) aut.push_back(order[i1]);
        if (aut.empty()) continue;
        const int kz = batch_kz(aut, m, tiles[aut[0]], residency);
        for (int i : aut) {
            MemberTiling& d = L.tiling[i];
            const int n2 = m[i].geo.n[2];
            d.kz = balanced_kz(n2, kz);
            d.chunks_z = (n2 + d.kz - 1) / d.kz;
        }
    }
    for (int idx = 0; idx < n; ++idx) {
        const int i = order[idx];
        if (L.groups.empty() || key(order[idx - 1]) != key(i)) {
            BatchGroup g;
            g.ndim = m[i].geo.ndim;
            g.precision = m[i].precision;
            g.integrator = m[i].integrator;
            g.tile = tiles[i];
            g.blk_off = L.nblk;
            g.nblk = 0;
            g.mem_off = idx;
            g.nmem = 0;
            g.cells = 0.0;
            L.groups.push_back(g);
        }
        const MemberTiling& d = L.tiling[i];
        const long long nb = (long long)d.tiles_x * d.tiles_y * d.chunks_z;
        if (nb > (1ll << 28) || L.nblk + nb > (1ll << 30)) return false;
        L.nblk += (int)nb;
        L.groups.back().nmem += 1;
        L.groups.back().cells += (double)m[i].geo.ncells;
        L.groups.back().nblk += (int)nb;
    }
    L.order = order;
    return true;
}

}  // namespace hydro
