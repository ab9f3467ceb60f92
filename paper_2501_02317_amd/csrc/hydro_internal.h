// Internal interface between the host runtime (runtime.hip) and the device
// kernels (kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.h"

namespace hydro {

constexpr int kMaxComp = 5;

// Device control block, one per mesh, in the caller's workspace: this
// structure, at kCtrlNext the step control that a step's first stage leaves
// for its second (StepCtl), and at kCtrlSlots two sets of kRateSlots
// accumulators of the CFL rate, each in a cache line of its own (an atomic
// maximum to one address takes 11.5 ns of every work-group on the device: 1024
// of them were 12 us of a stage).
//
// The rate of the current state is still in set `par` of the slots while
// pend is not kPendNone; then dt_raw (and after a step t, steps and done) are
// those of before it.  Outside such a state set `par` is zero; a first stage
// clears the set that its step will use, a control launch both.
struct Ctrl {
    double dt_raw;                  // cfl / (max CFL rate) of the current state
    double t;                       // simulation time
    unsigned int pend;              // what the rate in the slots is still to be used for (kPend...)
    unsigned int par;               // the set of slots in use
    unsigned int flags;             // sticky error flags
    unsigned int dt_valid;          // dt_raw belongs to the current state
    unsigned long long steps;       // completed steps
    double sums[2 * kMaxComp];      // totals: (sum, compensation) per component
    double t_end;                   // run limit in time (0: none)
    unsigned long long max_steps;   // run limit in steps (0: none)
    unsigned int done;              // a limit is reached: device-dt stages skip this mesh
    unsigned int pend_flags;        // error flags of the state that a pending rate belongs to
    double pad[6];
};
static_assert(sizeof(Ctrl) == 192, "control block layout");

constexpr unsigned int kPendNone = 0;  // nothing pending
constexpr unsigned int kPendStep = 1;  // a device-dt step: advance t and steps, then the next dt
constexpr unsigned int kPendRate = 2;  // the rate of a state: its dt only

struct StepCtl {
    double dt, dt_raw, t;
    unsigned long long steps;
    unsigned int done, par;
};

constexpr int kRateSlots = 32;
constexpr size_t kRateStride = 16;  // in doubles: one cache line
constexpr size_t kCtrlNext = 256, kCtrlSlots = 512;
constexpr size_t kCtrlBytes = kCtrlSlots + 2 * kRateSlots * kRateStride * sizeof(double);

__host__ __device__ inline StepCtl* ctrl_next(Ctrl* c) {
    return reinterpret_cast<StepCtl*>(reinterpret_cast<char*>(c) + kCtrlNext);
}
// Slot i of set par: the bits of a non-negative double, which order as integers.
__host__ __device__ inline unsigned long long* rate_slot(Ctrl* c, unsigned int par, unsigned int i) {
    return reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(c) + kCtrlSlots) +
           (par * kRateSlots + i) * kRateStride;
}

enum : unsigned int { FLAG_NONPHYSICAL = 1u };

enum CtrlOp : int {
    CTRL_INIT = 0,           // t = a0, steps = 0, flags = 0, dt invalid, nothing pending, no limits
    CTRL_FINALIZE = 1,       // use the pending rate, if any: dt_raw = cfl / rate, dt valid (after a step: t, steps, done)
    CTRL_FINALIZE_STEP = 2,  // the same for a step whose rate is in the slots unannounced
    CTRL_ADVANCE_T = 3,      // t += a0 (host dt), dt invalid
    CTRL_SET_LIMITS = 4,     // t_end = a0, max_steps = a1 (relative to the steps done), done
    CTRL_DROP_RATE = 5,      // nothing pending
};

// Refinement levels 0 .. kMaxLevels - 1; a refined block is named by the code
// level * 2^kLevelShift + its index on that level's block grid.
constexpr int kMaxLevels = 4;
constexpr int kLevelShift = 26;

// First block of each level 1 .. kMaxLevels - 1 in a refined mesh's leaf
// order (a level with no leaves starts where the next one does; unrefined
// meshes: every entry at the block count).
struct LevelStarts {
    int s[kMaxLevels - 1];
};

struct StageArgs {
    const double* in;    // stencil source: U^n (stage 1 / rhs) or U1 (stage 2)
    const double* base;  // U^n for the stage-2 combine (may alias out)
    double* out;         // U1, U^{n+1} (in place over base) or the increment
    Ctrl* ctrl;
    Geo geo;
    double dt_host;      // dt when use_device_dt == 0
    int use_device_dt;   // dt from ctrl (clamped to its t_end); skip the mesh when done
    int want_dt;         // stage 2: accumulate the next CFL candidate
    // the step keeps its own books: the first stage takes the pending rate
    // and leaves the step's control, the second leaves the next rate pending
    // (with want_dt; else nothing).  0: the caller's control launches do
    int chain;
    int tiles_x, tiles_y, chunks_z, kz;  // per block
    int blk0, nblk;      // the launch covers blocks blk0 .. blk0 + nblk - 1
    int conc;            // blocks whose stage work runs at once (automatic chunk length)
    // static refinement: per block 6 side codes (else null: the uniform
    // block grid of geo), and the ghost slots of the sides at level jumps
    const int* side;
    const double* gbuf;
    long long gcs;       // component stride within a ghost slot (slot = ncomp * gcs)
    // refined: the levels of the blocks (geo holds level 0's cell widths), and
    // the number of restriction slots (0 .. nres - 1): the cells next to those
    // sides are corrected after the stage, which takes their rate then
    LevelStarts starts;
    int nres;
};

// Side codes of a refined mesh's blocks, [block][kernel axis][low, high]:
// >= 0 the block of the same level across the side; kSidePhys a face of the
// mesh (its boundary rule); kSideSlot0 - q the ghost slot q, which holds the
// two ghost layers of the side, [comp][layer][t_hi][t_lo] over the side's two
// transverse kernel axes (t_lo the lower), layer 0 next to the face.
constexpr int kSidePhys = -1;
constexpr int kSideSlot0 = -2;

// One ghost slot: the side (ax, s) of block `leaf` at a level jump.
// kind 0 (restriction; leaf is coarse): src[o] is the fine block on the face
// at transverse child offsets o (bit 0: t_lo, bit 1: t_hi).  kind 1
// (prolongation; leaf is fine): src[0] is the coarse block, child[] the
// leaf's offsets (0/1) per kernel axis within its parent.  lev: the leaf's
// refinement level (its cell widths are level 0's times 2^-lev).
struct GhostTask {
    int leaf, ax, s, kind;
    int src[4];
    int child[3];
    int slot;
    int lev;
};

// One member of a batch: the stage kernels build StageArgs from it.
struct MeshDesc {
    double* U;
    double* U1;
    Ctrl* ctrl;
    Geo geo;
    int tiles_x, tiles_y, chunks_z, kz;
};

// What the device holds at once of a stage kernel (zero if the runtime cannot
// tell).
Slots stage_residency(int ndim, int precision, int mode, const Tile& t);

// The chunk length of a launch: the tile's, or the automatic one for the blocks
// whose work runs at once (this launch's, or those of the launches on the
// other streams as well).  The model takes 0.3-5 us of the host, so a handle
// keeps the answer.
int stage_kz(int precision, int mode, const Tile& tile, const StageArgs& a);
hipError_t launch_stage(int precision, int mode, const Tile& tile, StageArgs a, hipStream_t s);
// The same launch described (kernel, grid, block, arguments) instead of
// enqueued, for a caller that adds it to a graph as a kernel node.
struct StageLaunch {
    const void* func;
    dim3 grid, block;
    StageArgs args;
};
// Launch context of the stage dispatch: a single mesh (args) or a batch group
// (descriptor table); with rec, a single-mesh launch is described there
// instead of enqueued; with slots, nothing is launched and the kernel's
// residency is written there.
struct LaunchCtx {
    const StageArgs* a;
    const MeshDesc* d;
    const int2* blk;
    int nblk;
    StageLaunch* rec;
    Slots* slots;
};
hipError_t launch_stage_1d_fp64(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s);
hipError_t launch_stage_1d_mixed(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s);
hipError_t launch_stage_2d_fp64(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s);
hipError_t launch_stage_2d_mixed(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s);
hipError_t launch_stage_3d_fp64(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s);
hipError_t launch_stage_3d_mixed(int mode, const Tile& t, const LaunchCtx& L, hipStream_t s);

hipError_t plan_stage_launch(int precision, int mode, const Tile& tile, StageArgs a, StageLaunch* out);
// One stage over every mesh of a group sharing ndim, precision and tile:
// blk[i] = (member, work-group within the member), nblk entries.
hipError_t launch_stage_batch(int ndim, int precision, int mode, const Tile& tile, const MeshDesc* d,
                              const int2* blk, int nblk, hipStream_t s);
// nsteps device-dt steps of an unsplit 1-D mesh of at most kRun1dMost cells in
// one work-group: the pending rate, if any, is used, and nothing is left
// pending.  Two stage launches take 9.7-10.5 us a step at any such size; the
// one work-group takes 2.7 us at 256 cells, 7.4 us at 1024 (FP64; mixed 2.3
// and 5.3 us), and with two cells a thread would take 13 us at 2048.
constexpr int kRun1dMost = 1024;
hipError_t launch_run_1d_fp64(int vl2, const Geo& g, double* U, Ctrl* ctrl, int nsteps, hipStream_t s);
hipError_t launch_run_1d_mixed(int vl2, const Geo& g, double* U, Ctrl* ctrl, int nsteps, hipStream_t s);
// (done, flags, steps) of members [0, n) of a descriptor table into out[3 i ..].
hipError_t launch_status_gather(const MeshDesc* d, int n, unsigned long long* out, hipStream_t s);
// CTRL_FINALIZE for members [0, n) of a descriptor table.
hipError_t launch_ctrl_batch(const MeshDesc* d, int n, hipStream_t s);
hipError_t launch_ctrl(Ctrl* c, int op, double a0, double a1, double cfl, hipStream_t s);
hipError_t launch_totals(const Geo& g, const double* U, double* partials, int nparts, Ctrl* ctrl,
                         hipStream_t s);
// The same reduction, written as out[c] = dV (sum + compensation) on the
// device (partials: 2 ncomp nparts doubles of scratch).
hipError_t launch_totals_out(const Geo& g, const double* U, double* partials, int nparts, double* out, double dV,
                             hipStream_t s);
// Conserved variables U (block layout) of the primitive state W, in the mesh
// layout (mesh_layout != 0) or the block layout (in place when W == U), with
// the CFL rate of U left pending.  Blocks of level L take g0's cell widths
// times 2^-L.
hipError_t launch_prim_to_cons(const Geo& g0, const LevelStarts& starts, int nblk, const double* W, double* U,
                               int mesh_layout, Ctrl* ctrl, hipStream_t s);
// Copy a field between the mesh layout [comp][k][j][i] (mesh) and the block
// layout (blk): to_blocks != 0 reads mesh and writes blk, else the reverse.
hipError_t launch_relayout(const Geo& g, double* mesh, double* blk, int to_blocks, hipStream_t s);
hipError_t launch_padded_prim(const Geo& g, int precision, const double* U, double* Wpad, Ctrl* ctrl,
                              hipStream_t s);
hipError_t launch_riemann(int precision, int ntan, double gamma, long long n, const double* WL,
                          const double* WR, double* F, hipStream_t s);

// Static refinement passes over the ghost slots tasks[0, n) (all of one
// kind): restriction or prolongation of the stage input U into gbuf
// (conserved FP64 values); and, after a stage from in to out, the fine-flux
// corrections of the coarse cells next to every level jump (the nres
// restriction slots): factor * lam * (coarse flux - mean of the fine fluxes)
// added to out, a cell next to jumps on several axes in axis order (first:
// fluxes of piecewise-constant states, as in the van Leer predictor), with
// want_dt also the CFL rate of the corrected cells.  g holds a block's extents
// and level 0's cell widths; the step's length is the one its first stage left
// (StageArgs::chain).
hipError_t launch_smr_restrict(const Geo& g, const double* U, double* gbuf, long long gcs, const GhostTask* tasks,
                               int n, Ctrl* ctrl, hipStream_t s);
hipError_t launch_smr_prolong(const Geo& g, const double* U, const int* side, double* gbuf, long long gcs,
                              const GhostTask* tasks, int n, Ctrl* ctrl, hipStream_t s);
hipError_t launch_smr_correct(int precision, int first, const Geo& g, const double* in, double* out, double factor,
                              int use_device_dt, double dt_host, const int* side, const double* gbuf, long long gcs,
                              const GhostTask* tasks, int nres, int want_dt, Ctrl* ctrl, hipStream_t s);
// CFL rate of the nblk blocks of U, left pending; a block of level L (from the
// level starts) has g0's cell widths times 2^-L.
hipError_t launch_dt_levels(const Geo& g0, const LevelStarts& starts, int nblk, const double* U, Ctrl* ctrl,
                            hipStream_t s);

// Number of totals partials the runtime reserves.
constexpr int kTotalsParts = 1024;
// Blocks of one mesh: each needs one totals partial at least.
constexpr int kMaxBlocks = kTotalsParts;

__host__ __device__ inline int geo_nblk(const Geo& g) { return g.blocks[0] * g.blocks[1] * g.blocks[2]; }

}  // namespace hydro
