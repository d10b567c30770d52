// Internal interface between the host runtime (lbm_runtime.cpp) and the HIP
// kernels (lbm_kernels.hip, lbm_adjoint.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lbm {

enum Dtype : int { kF64 = 0, kF32 = 1, kF16S = 2, kBF16S = 3 };
enum Layout : int { kDenseAB = 0, kDenseAA = 1, kTiled16 = 2, kIndirect = 3 };

constexpr int kTile = 16;
constexpr int kTileNodes = kTile * kTile;

// Per-tile scalars of the tiled step, one 128-byte row per kept tile: the
// tile-neighbour row (as tile_nbr; entry 0 = the tile itself) and, per 64-slot
// wavefront w, its fluid lanes (bit l of fluid[w] <=> slot 64 w + l is fluid).
struct alignas(128) TileMeta {
    int32_t nbr[9];
    int32_t pad[7];
    uint64_t fluid[4];
    uint64_t pad2[4];
};
static_assert(sizeof(TileMeta) == 128, "one 128-byte row per tile");

// Everything a kernel launch needs to know about a context's device state.
struct DevState {
    int dtype = 0, layout = 0;
    int nx = 0, ny = 0;
    int pitch = 0;        // dense: row pitch in elements (multiple of 64)
    size_t plane = 0;     // elements per population plane of one lattice
    void *f[2] = {nullptr, nullptr};  // lattices (DENSE_AA: f[1] = memory lent for one
                                      // call, used by launch_steps only; else null)
    const uint8_t *type = nullptr;    // node-type codes (dense / tiled)
    const uint8_t *nmask = nullptr;   // solid-neighbour bits (dense / tiled)
    const uint32_t *seg_interior = nullptr;  // dense: per 256-node row segment, 1 = all interior
    double interior_frac = 0.0;       // dense: fraction of the segments that are all interior
    const float *alpha = nullptr;     // drag coefficient, same indexing as type
                                      // (INDIRECT: per compacted node); may be null
    const int32_t *tile_xy = nullptr, *tile_nbr = nullptr;  // TILED16
    const TileMeta *tile_meta = nullptr;  // TILED16: [n_tiles], the step's per-tile scalars
    const int32_t *fluid_xy = nullptr;                      // INDIRECT: [n][2]
    const uint32_t *ind_pk = nullptr;                       // INDIRECT: packed row offsets
    const uint16_t *ind_info = nullptr;                     // INDIRECT: solid bits + edge flag
    const int32_t *ind_edge = nullptr;                      // INDIRECT: edge-node table [][8]
    double fluid_frac = 0.0;  // fluid nodes over mesh nodes
    // sparse layouts: fluid bits of the 64-column chunks [ny][pitch / 64]; INDIRECT:
    // list index of each chunk's first fluid node; TILED16: tile index of every
    // 16 x 16 square [ny / 16][nx / 16], -1 where none is kept
    const uint64_t *chunk_fluid = nullptr;
    const uint32_t *chunk_first = nullptr;
    const int32_t *tile_of = nullptr;
    const double *bc_val = nullptr;   // open-boundary values [node][2], same indexing as
                                      // alpha; read only at open-boundary nodes
    int open = 0;                     // 1 when the node types hold open-boundary codes
    int trt = 0;                      // 1: two-relaxation-time collision (omega_m below)
    int fullway = 0;                  // 1: full-way bounce-back (A-B layouts)
    double omega_m = 1.0;             // antisymmetric relaxation rate (TRT)
    int mrt = 0;                      // 1: multiple-relaxation-time collision
    double s_e = 1.0, s_eps = 1.0, s_q = 1.0;  // its energy, energy-square, flux rates
    int64_t n_tiles = 0, n_fluid = 0;
    double omega = 1.0, gx = 0.0, gy = 0.0;
    // launch_steps on squares: the lattice of every step is stored, this many elements
    // apart, the first one at f[1 - cur] (0: the last step's only)
    size_t every = 0;
    hipStream_t stream = nullptr;
    double *red_partials = nullptr;   // reduction scratch (>= red_capacity doubles)
    int64_t red_capacity = 0;
};

// Number of thread blocks the visit / reduction kernels use for this layout.
int64_t visit_blocks(const DevState &s);
// Doubles of reduction scratch (red_partials) a reduction needs: one partial per
// visit block plus the first-stage sums.
int64_t reduction_capacity(const DevState &s);

// One time step from lattice `cur` (A-B layouts write lattice 1 - cur).  For
// DENSE_AA, t is the number of steps already taken (its parity picks the
// even or odd kernel).
hipError_t launch_step(const DevState &s, int64_t t, int cur);

// Squares of n x n nodes, which lose a ring of nodes per step, that cover the lattice.
inline int64_t square_blocks(int nx, int ny, int n, int steps)
{
    const int out = n - 2 * steps;
    return (int64_t)((nx + out - 1) / out) * ((ny + out - 1) / out);
}

// Small lattices run the fused steps on squares of n x n nodes: n = 16 or 32 and the
// most steps a launch then takes (returned); n = 0 for larger lattices (strips).
// 16 x 16 nodes at four steps while that leaves at most one workgroup per CU; else
// 32 x 32 at the most steps that do; else four steps, in FP64 up to two rounds of the
// chip (one workgroup per CU: its LDS), in the narrower types up to three (two per CU).
// Measured, us per step, FP64: 256 x 64 1.29 (16, 4 steps), 1.57 (32, 8 steps), strips
// 2.56; 257^2 with a lid, TRT 2.03 (32, 6 steps), 2.53 (16, 3 steps), strips 3.8; 512^2 with a
// force 4.5 (32, 4 steps), strips 5.0; FP32 128^2 0.99 (16, 4 steps), 1.02 (32, 8 steps); 400 x
// 300 1.63 (32, 4 steps), 2.10 (16, 3 steps); 1024 x 256 with drag 2.98 (32, 4 steps), 3.4
// (32, 6 steps), strips 4.0; with a force FP64 560^2 6.3, strips 5.5; FP32 760^2 5.0,
// strips 5.7, 900^2 6.9, strips 7.5.
inline int square_steps(int nx, int ny, int dtype, int &n)
{
    n = 16;
    if (square_blocks(nx, ny, n, 4) <= 256)
        return 4;
    n = 32;
    for (int k = 8; k > 4; --k)
        if (square_blocks(nx, ny, n, k) <= 256)
            return k;
    if (square_blocks(nx, ny, n, 4) <= (dtype == kF64 ? 512 : 1500))
        return 4;
    n = 0;
    return 0;
}

// The strip kernels of the fused steps that are compiled: the most steps a launch of one may
// take (its block size and registers), 0 for a variant that there is none of.  Eight steps
// in flight where the registers allow two workgroups of 8 S wavefronts per CU; the
// variants with more live values (MRT, drag, open boundaries, TRT with a force, most on
// sparse layouts) take six.  MRT costs the 16-bit types more than strips save: sparse
// layouts, and dense ones with a force or drag or open boundaries, take it on squares only.
constexpr bool strip_heavy(bool f64, bool sparse, bool force, bool drag, bool open, bool trt,
                           bool mrt)
{
    const bool forced = force || drag;
    return mrt || open || drag || (trt && forced) || (sparse && (f64 || trt || forced));
}
constexpr int strip_steps(bool f64, bool bits16, bool sparse, bool force, bool drag, bool open,
                          bool trt, bool mrt)
{
    if (bits16 && mrt && (sparse || force || drag || open))
        return 0;
    return strip_heavy(f64, sparse, force, drag, open, trt, mrt) ? 6 : 8;
}

// Most steps one launch_steps call takes where that is faster than single steps (1: this
// lattice runs single steps only).
int max_fused_steps(const DevState &s);
// Steps of the next launch of a call with `left` steps to go: the most, or the rest where one
// launch of so few is faster than single steps, or 1.
int next_steps(const DevState &s, int64_t left);
// Fused launches that end in the lattice they start from, for `m` steps (even) of the AA
// layout: an even number of launches, sharing at most m steps in even parts (0: none).
struct ThereAndBack {
    int64_t launches = 0, steps = 0;
    int unit = 2;
    // Steps of the next launch; updates both counts.
    int next()
    {
        const int64_t even = unit * ((steps + unit * launches - 1) / (unit * launches));
        const int64_t k = even < steps - 2 * (launches - 1) ? even : steps - 2 * (launches - 1);
        steps -= k;
        --launches;
        return (int)k;
    }
};
ThereAndBack there_and_back(const DevState &s, int64_t m);
// `steps` (2 .. max_fused_steps) time steps from lattice `cur` to lattice 1 - cur in
// one launch, bitwise those of `steps` launch_step calls (fluid nodes; the slots of solid
// nodes are neither read into a result nor written).  DENSE_AA: an even number of steps
// from an odd time step, f[1] being lent memory.
hipError_t launch_steps(const DevState &s, int cur, int steps);
#define LBM_DECLARE_STEPS(place)                                              \
    hipError_t launch_steps_##place##_f64(const DevState &, int, int);        \
    hipError_t launch_steps_##place##_f32(const DevState &, int, int);        \
    hipError_t launch_steps_##place##_f16(const DevState &, int, int);        \
    hipError_t launch_steps_##place##_bf16(const DevState &, int, int);
LBM_DECLARE_STEPS(dense)
LBM_DECLARE_STEPS(aa)
LBM_DECLARE_STEPS(list)
LBM_DECLARE_STEPS(tiles)
#undef LBM_DECLARE_STEPS

// Canonical populations fc (device FP64 [9][ny][pitch]) -> stored state at step t.
// Full-way rule: fc's wall slots become the populations in flight; with
// fill_walls they are taken instead from the fluid node each slot is fed by
// (slot j of wall node w <- f_j(w - c_j)).
hipError_t launch_scatter_canonical(const DevState &s, int64_t t, int cur, const double *fc,
                                    int fill_walls);
// Rest state (rho = 1, u = 0) straight into one stored lattice (all 9 * plane
// slots), without a canonical staging buffer.
hipError_t launch_rest(const DevState &s, void *lattice);
// FP64 tiles: what a single step stores in the solid slots of a lattice (k_step_tiled).
hipError_t launch_placeholders(const DevState &s, void *lattice);
// Equilibrium (Eq. 6) from device FP64 [ny][nx] fields (null = rest) -> fc.
hipError_t launch_equilibrium(const DevState &s, const double *rho, const double *ux,
                              const double *uy, double *fc);
// Stored state -> canonical fc (solid slots untouched: clear them first).
hipError_t launch_gather_canonical(const DevState &s, int64_t t, int cur, double *fc);
// Macroscopic fields of fluid nodes (solid entries untouched).
hipError_t launch_macroscopic(const DevState &s, int64_t t, int cur, double *rho, double *ux,
                              double *uy);
// Deterministic FP64 sums over fluid nodes into *out (device): total mass, or
// the sum of u_x over the fluid nodes of column x_col.
hipError_t launch_mass(const DevState &s, int64_t t, int cur, double *out);
hipError_t launch_column_ux(const DevState &s, int64_t t, int cur, int x_col, double *out);

hipError_t launch_fill(double *p, size_t n, double v, hipStream_t stream);
hipError_t launch_copy16(const void *src, void *dst, size_t bytes, hipStream_t stream);

// ---- adjoint (DENSE_AB, F64 / F32) --------------------------------------
// Adjoint fields are dense [9][ny][pitch] in the compute type.  dJ/dg block
// partials are pairs (x, y) per block.
int64_t adjoint_blocks(const DevState &s);       // blocks of one adjoint step
int64_t adjoint_step_partials(const DevState &s);  // dJ/dg partial pairs of one adjoint step
// Pairs of adjoint scratch needed: the partials of a step or seed plus the
// first-stage sums of launch_partials_into (written right after the partials).
int64_t adjoint_scratch_pairs(const DevState &s);
int64_t adjoint_seed_blocks(const DevState &s);  // blocks of the seed kernel
// lambda_T of J = scale * sum of u_x over the fluid nodes of column x_col, read
// from the stored lattice `state`; direct dJ/dalpha terms into grad_alpha (if
// a drag field is set) and dJ/dg partials (one pair per seed block).
hipError_t launch_adjoint_seed_raw(const DevState &s, const void *state, int x_col, double scale,
                                   void *mu, double *grad_alpha, double *partials);
// One reverse step: state = stored lattice at step t, mu_in = lambda_{t+1};
// writes lambda_t, adds to grad_alpha, writes (accumulate = 0) or adds
// (accumulate = 1) the per-block dJ/dg partials.
hipError_t launch_adjoint_step_raw(const DevState &s, const void *state, const void *mu_in,
                                   void *mu_out, double *grad_alpha, double *partials,
                                   int accumulate);
// Most reverse steps a launch_adjoint_steps_raw call takes on this lattice (1: none).
int adjoint_square_steps(const DevState &s);
// `steps` reverse steps over the states number j0, j0 - 1, .. (number 0 at `first`,
// j > 0 at rest + j * every elements), with accumulate = 1; per node bitwise those of
// single steps.
hipError_t launch_adjoint_steps_raw(const DevState &s, const void *first, const void *rest,
                                    size_t every, int j0, int steps, const void *mu_in,
                                    void *mu_out, double *grad_alpha, double *partials);
// dJ/dg partial pairs of a run of reverse steps, single or several per launch.
int64_t adjoint_run_partials(const DevState &s);
// Adjoint field <-> device FP64 planes [9][ny][nx] (to_plain = 1: field -> planes).
hipError_t launch_adjoint_convert(const DevState &s, void *mu, double *plain, int to_plain);
// grad_g[0..1] += fixed-order sum of n partial pairs.
hipError_t launch_partials_into(double *partials, int64_t n, double *grad_g,
                                hipStream_t stream);
hipError_t launch_zero(double *p, int64_t n, hipStream_t stream);
// Allocation-free adjoint step: its dJ/dg partials live in a fixed per-device
// array of kNoAllocScratchDoubles doubles (1 MiB).  adjoint_step_scratch_doubles
// = the doubles one step needs there (partials plus reduction stage);
// noalloc_scratch = that array's device address on `device` (looked up once
// per device with hipGetSymbolAddress, then cached).
constexpr int64_t kNoAllocScratchDoubles = int64_t(1) << 17;
int64_t adjoint_step_scratch_doubles(const DevState &s);
hipError_t noalloc_scratch(int device, double **ptr);

}  // namespace lbm
