// Host-side planning: tiles, chunk lengths and the layout of a batch.  Plain
// C++ without device code or HIP types, so it is built and checked on its own.
#pragma once

#include <vector>

namespace hydro {

// Geometry in kernel axes.  Kernel axis 0 is x.  For 3-D, kernel axes
// (0, 1, 2) are (x, y, z); for 2-D, kernel axis 2 (the marching axis)
// is the physical y axis and kernel axis 1 has extent 1; for 1-D only
// kernel axis 0 is active.  The cell index (k * n1 + j) * n0 + i is the
// physical storage index in every case.
//
// A mesh may be split into blocks[0] x blocks[1] x blocks[2] blocks of equal
// extents (kernel axes); n and ncells are those of one block.  Fields are
// stored block after block, [block][comp][cell of the block], with block
// index b0 + blocks[0] (b1 + blocks[1] b2).  The boundary codes are those of
// the whole mesh: a side of a block inside the mesh, or on a periodic axis,
// reads its ghosts from the neighbouring block (a c-boundary); one block on a
// periodic axis is its own neighbour.
struct Geo {
    int ndim;
    int n[3];
    int blocks[3];
    double dx[3];
    double inv_dx[3];
    int bc[3][2];
    double gamma;
    double cfl;
    long long ncells;
};

struct Tile {
    int tx, ty, kz;
};

// Stage kernels: the Heun stages (and the stage right-hand side), and the
// van Leer predictor and corrector (Sec. 3.3).  The _C forms keep the
// predicted state conserved in FP64 (a refined mesh, whose level-jump passes
// read conserved stage inputs): the predictor writes U* = U^n + (dt/2) L_1(U^n)
// and the corrector reads U* as its stencil input.  MODE_STAGE2_R is the Heun
// stage 2 of a refined mesh (as MODE_VL2_CORR_C the corrector of one): the
// cells corrected after it take no part in its CFL rate.
enum StageMode : int {
    MODE_RHS = 0,
    MODE_STAGE1 = 1,
    MODE_STAGE2 = 2,
    MODE_VL2_PRED = 3,
    MODE_VL2_CORR = 4,
    MODE_VL2_PRED_C = 5,
    MODE_VL2_CORR_C = 6,
    MODE_STAGE2_R = 7
};

// The automatic chunk length (Tile::kz == 0), 1 .. kMaxAutoKz planes, of a
// launch over the columns m[0 .. n) (each marches over n2 planes) by a kernel
// of the given residency; and the length that gives a column the same number
// of chunks in the most equal parts.
constexpr int kMaxAutoKz = 128;
struct Slots {
    int cus, per_cu;  // CUs of the device, work-groups of the kernel resident on each
    int waves;        // waves of a work-group
};
struct MarchCols {
    long long cols;
    int n2;
    bool per_xcd;  // the launch covers eight blocks of a split mesh: one to each XCD
};
// *time (if given): the launch's modelled time, in planes of a work-group that
// has a CU to itself.
int auto_kz(int ndim, const Slots& sl, const MarchCols* m, int n, double* time = nullptr);
int balanced_kz(int n2, int kz);

// The tiling of a mesh (or of one block) by a tile (kz == 0 counts as 1: the
// caller resolves the automatic length).
void plan_tiles(const Geo& g, const Tile& t, int& tiles_x, int& tiles_y, int& chunks_z, int& kz);

// Default tile for a mesh (kernel axes) and precision.
Tile default_tile(const Geo& g, int precision, int mode);
// Whether the stage kernel is compiled for this tile shape.
bool tile_supported(int ndim, const Tile& t);
// Tiles the autotuner tries for a mesh (at most max written); returns how
// many there are.
int tile_candidates(const Geo& g, Tile* out, int max);

// ------------------------------------------------------------------ batches

// What the plan of a batch needs to know of a member.
struct PlanMember {
    Geo geo;
    int precision, integrator;
    Tile tile;      // of stage 1: a batch uses it for both stages
    bool tile_set;  // by the caller or an autotuner (else the default)
};

struct BatchGroup {
    int ndim, precision, integrator;
    Tile tile;
    int blk_off, nblk;
    int mem_off, nmem;  // the group's descriptors: [mem_off, mem_off + nmem) of the descriptor table
    double cells;       // cells of its members
};

struct MemberTiling {
    int tiles_x, tiles_y, chunks_z, kz;
};

struct BatchLayout {
    std::vector<int> order;           // order[k]: the member of descriptor k
    std::vector<MemberTiling> tiling;  // per member (caller's order)
    std::vector<BatchGroup> groups;
    int nblk = 0;                      // work-groups of all groups
};

// Tells what the device holds at once of a stage kernel (stage_residency).
typedef Slots (*Residency)(int ndim, int precision, int mode, const Tile& t);

// The batch autotuner's rules are 0 .. kNumBatchRules - 1; rule 0 keeps every
// member's tile.  rule_tile: a member's tile under a rule.
constexpr int kNumBatchRules = 12;
Tile rule_tile(const PlanMember& m, int rule);
// The layout under a rule; false if it has too many work-groups.
bool plan_layout(const std::vector<PlanMember>& m, int rule, Residency residency, BatchLayout& L);

}  // namespace hydro
