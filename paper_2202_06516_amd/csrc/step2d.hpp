// step2d.hpp -- one time step of a D2Q9 lattice in a single launch.
//
// The split step is five or six launches per step (density, two fills, mu,
// collision, finalize) that pass rho and mu through memory and read every
// population twice.  k_step2d does the step of a tile of nodes in one
// workgroup: it forms rho of the tile and of the halo the stencils of Eq. 7
// and Eq. 12 reach (from the populations, which the neighbouring tiles read as
// well: those reads are cache hits), fills the solid layers of Eq. 14 inside
// the halo, forms mu, all in LDS, and collides the tile's nodes from the
// populations it kept in registers.  Each node's arithmetic is that of the
// split path's bodies, expression by expression, so both paths give the same
// bits; rho and mu of the step never reach memory (on measure steps the field
// that the crossing search reads is stored).
//
// Halo per model: chemical potential 4 (force stencil 2, Laplacian 2), 6 in
// tiles with a solid node or a boundary node in reach (a second-layer node's
// density comes from first-layer nodes, and theirs from fluid nodes);
// pseudopotential 1; phase field 2 (its force needs mu at the node alone).
// Tiles without a solid in reach read no class at all.
//
// A lattice (or every case of a batch) is a list of tiles; one workgroup per
// tile, ids dealt so that each XCD owns a contiguous run of tiles.
//
// Bound: on small lattices the chain of a launch, one class and population
// load, the LDS passes and the stores (6 us per step at 256^2 FP32 instead of
// 22 us of dependent launches); on large ones vector instructions (560 per
// node of 3000 x 400 in FP32 with the halo's share, 0.74 per busy cycle of a
// compute unit, which issues one at most; 512 cases 713 and 0.86), then memory
// (72 bytes per node, 1.16 times that counted).  The phase field is bound by
// memory (5.4 TB/s counted over 512 cases; in FP32 its MRT collision spills 24
// registers, a part of that traffic).  Measured against the split step, per
// step: 128^2 FP64 14 instead of 30 us with the reads of a 20-step call, 3000 x
// 400 FP32 33 instead of 51 us, ten 700 x 400 cases 67 instead of 97 us, 256
// uneven cases (20 M nodes) 0.52 instead of 0.78 ms.
#pragma once

#include <vector>

#include "kernels.hpp"
#include "phasefield.hpp"

namespace lbm {

enum : int { M2_CHEM = 0, M2_PSEUDO = 1, M2_PHASE = 2 };      // the model of a launch
enum : int { T2_SOLID = 1, T2_EDGE = 2 };                     // Tile2d::flags

// 32 bytes: one scalar load gives a workgroup all it needs of its lattice
struct Tile2d {
    int c;             // case (index of the reduction slots)
    int x0, y0;        // first node
    int flags;         // T2_SOLID: a non-plain node within reach; T2_EDGE: its reach wraps around the lattice
    int nx, ny, px;    // the case's lattice
    uint32_t off;      // its first node in the packed arrays
};
static_assert(sizeof(Tile2d) == 32, "one s_load_dwordx8");

// Tile shapes: tw x th nodes per workgroup of nt threads.
struct Shape2d {
    int tw, th, nt;
};

// One launch of the step over a tile list.
struct Step2dArgs {
    int precision;             // LBM_F32 / LBM_F64 / LBM_F32_MIXED
    int model, mrt, shape;     // M2_*, 1: MRT, index of shape2d()
    const Tile2d* tiles;
    int ntiles;
    long long N;               // population stride
    const void *fin, *gin;     // pull form
    void *fout, *gout;
    void* field;               // rho (phase field: phi), stored on measure steps
    const void* wall;          // mu (psi) of the solid layers, or phi of the phase field
    const uint8_t* cls;
    WallBC bc;
    DevCtl* ctl;
    MeasureSlots* slots;       // per case
    double rho_m, inv_b;
    PhaseField pf;
    int meas;                  // 1: a measure step (field, centroid sums)
    int tick;                  // 1: count the step (launches without a finalize after them)
    int grav;                  // 1: the body force acts
};

Shape2d shape2d(int k);
// the tiles of the given lattices (flags not set)
std::vector<Tile2d> tiles2d(const Dims* dims, int n, int shape);
// the shape for this many nodes in all
int shape2d_for(long long nodes, int precision, int model);
// sets the flags of every tile from the classes (enqueues)
void tiles2d_flags(Tile2d* tiles, int ntiles, const uint8_t* cls, int model, int shape,
                   hipStream_t st);
// one step (enqueues); th and cp as the split path takes them, cp in the arithmetic type of a.precision
void step2d_launch(const Step2dArgs& a, const Thermo& th, const void* cp, hipStream_t st);

}  // namespace lbm
