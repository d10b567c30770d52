// Several D2Q9 steps in one launch, on the dense lattices (A-B; AA after an odd number of
// steps), the node list and the tiles.
//
// A single step reads and writes every population once, so it cannot run
// faster than the memory moves 18 populations a node.  k_steps reads a strip of
// the lattice once, carries it through K steps on chip and writes the result of
// the K-th: the memory traffic of one step for K of them.  A workgroup owns a
// strip of 64 S columns and marches along it row by row; it holds K groups of
// S wavefronts, group j doing step j + 1 of every row.  The rows between two
// groups go through LDS (two rows of 9 populations each, one being read while
// the next is written, one barrier per row); the populations a group needs from
// the two rows before are kept in its registers.  So step j + 1 runs two rows
// behind step j, and K steps of a row are in flight at once.  The strip loses
// one column at each side per step, which neighbouring strips compute again:
// it updates 64 S - 2 halo columns, halo >= K.  The same holds for the first and
// last rows of a workgroup's part of the strip.
//
// The arithmetic is the single step's (collide, apply_open_values, the storage
// conversion between two steps), so the result is bitwise that of K single
// steps.  Boundary nodes: the node types travel with the rows; a row of interior
// nodes (one ballot) skips the bounce-back selects.
//
// Measured, 4096^2, us per step over calls of 48 steps (single launches -> fused): FP64
// 388 -> 104 (8 steps a launch), FP32 190 -> 54, FP16 99 -> 58, BF16 99 -> 61; with walls
// FP64 112, FP32 63; with a force and walls 134, 77, FP16 80; MRT 127, 81, FP16 91; TRT FP64 110;
// drag FP64 140.  The FP32 and 16-bit kernels are bound by VALU issue (0.9 to 1.0 of its cycles:
// 118 and 130 instructions a node and step, 4 cycles a wavefront each); with open boundaries
// on 512 rows 0.5: strips of 40 rows spend 17 of 57 iterations filling and draining.  FP64 moves 2.5 GB a
// launch (1.03 of one step's) in 830 us, 0.48 of the copy rate, and issues 61 % of the
// VALU cycles: what is left is the barrier per row, which keeps the two from
// overlapping fully.  A form that kept all K
// steps in one wavefront (rows in registers, lane shifts instead of LDS) ran
// FP64 125, FP32 68, FP16 75 at its best K = 4, 4, 2: K is bounded by the
// registers there, and boundary handling spilled them.
#pragma once

#include <algorithm>
#include <type_traits>

#include "lbm_dense.h"
#include "lbm_device.h"
#include "lbm_launch.h"

namespace lbm {
namespace {

// Where population i of a node lies.  kDense: the dense A-B lattice.  kDenseOpp:
// the AA lattice after an odd number of steps, which holds the post-collision
// f_i in slot opp(i) of its own node, that is the A-B state with the slots of
// opposite directions exchanged.  kList, kTiles: the sparse layouts.
enum Place : int { kDense = 0, kDenseOpp = 1, kList = 2, kTiles = 3 };

struct StripGeom {
    uint32_t nstrips;
    int steps;  // K
    int halo;   // columns at each side of a strip that only feed it
    int rows;   // rows a workgroup updates
    // sparse layouts: fluid bits of the 64-column chunks of every row, and
    // INDIRECT: the list index of each chunk's first fluid node and the nodes'
    // info words, TILED16: the tile index of every 16 x 16 square (-1: none)
    const uint64_t *chunk_fluid;
    const uint32_t *chunk_first;
    const uint16_t *info;
    const int32_t *tile_of;
    uint32_t n_fluid;
    uint64_t every;  // squares: DevState::every
};

// Slot of direction i among those of equal c_i.y (rows kept in registers).
__device__ constexpr int kLineOf[9] = {0, 1, 0, 2, 0, 1, 2, 1, 2};

// The stored value b where `m` is all ones, a where it is zero.
template <class M>
__device__ __forceinline__ M select_bits(M a, M b, uint32_t m)
{
    if constexpr (sizeof(M) == 8) {
        const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
        const uint32_t lo = ((uint32_t)y & m) | ((uint32_t)x & ~m);
        const uint32_t hi = ((uint32_t)(y >> 32) & m) | ((uint32_t)(x >> 32) & ~m);
        return __builtin_bit_cast(M, ((uint64_t)hi << 32) | lo);
    } else if constexpr (sizeof(M) == 4) {
        const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
        return __builtin_bit_cast(M, (y & m) | (x & ~m));
    } else {
        const uint32_t x = __builtin_bit_cast(uint16_t, a), y = __builtin_bit_cast(uint16_t, b);
        return __builtin_bit_cast(M, (uint16_t)((y & m) | (x & ~m)));
    }
}

// LDS layout of a strip: rows between groups, then node types and drag
// coefficients of the rows in flight (the last step lags 2 K - 1 rows behind the
// source, and one row is being written), and what the sparse layouts need to place
// the result: the list index of each wavefront's first kept column, or the tiles of
// the (at most three) tile rows in flight; with open boundaries every node's index.
template <class M, int S>
struct StripLds {
    static constexpr int kWid = 64 * S;
    static constexpr int kLp = kWid + 2;  // one column more at each end
    static __host__ __device__ constexpr int node_rows(int K) { return 2 * K + 2; }
    static __host__ __device__ constexpr uint32_t ring_bytes(int K)
    {
        return (uint32_t)(K * 2 * 9 * kLp) * (uint32_t)sizeof(M);
    }
    static __host__ __device__ constexpr uint32_t bytes(int K, bool walls, bool drag, bool open,
                                                        int place)
    {
        const uint32_t rows = (uint32_t)node_rows(K), n = rows * (uint32_t)kWid;
        return ring_bytes(K) + n * ((walls ? 2u : 0u) + (drag ? 4u : 0u)) +
               (place < kList ? 0u : open ? 4u * n : place == kList ? 4u * rows * S : 16u * kWid);
    }
};

// WALLS = false: the lattice has interior fluid nodes only.  MAXK: the most
// groups a launch may have (block size 64 S K).  LB: wavefronts per SIMD the
// registers have to allow.
template <class ST, int PH, bool WALLS, int PLACE, int S, int MAXK, int LB>
__global__ __launch_bounds__(64 * MAXK * S, LB) void k_steps(const DenseArgs<ST> k,
                                                             const StripGeom g)
{
    using R = typename ST::real;
    using M = typename ST::mem;
    using L = StripLds<M, S>;
    constexpr bool DRAG = (PH & 3) == kDragged, FORCE = (PH & 3) != kBGK, TRT = (PH & kTRT) != 0,
                   MRT = (PH & kMRT) != 0, OPEN = (PH & kOpenBC) != 0;
    constexpr bool SPARSE = PLACE >= kList;
    static_assert(WALLS || (!OPEN && !SPARSE), "the node types are needed");
    constexpr uint32_t DS = PLACE == kTiles ? kTileStride : kChunk;  // direction stride
    extern __shared__ __align__(16) unsigned char lds[];
    const int K = g.steps, NR = L::node_rows(K);
    auto ring = reinterpret_cast<M(*)[2][9][L::kLp]>(lds);
    auto node = reinterpret_cast<uint16_t(*)[L::kWid]>(lds + L::ring_bytes(K));
    auto drag = reinterpret_cast<float(*)[L::kWid]>(
        lds + L::ring_bytes(K) + (WALLS ? (uint32_t)(NR * L::kWid) * 2u : 0u));
    uint32_t *const place_lds = reinterpret_cast<uint32_t *>(
        lds + L::ring_bytes(K) + (uint32_t)(NR * L::kWid) * (DRAG ? 6u : 2u));
    auto index = reinterpret_cast<uint32_t(*)[L::kWid]>(place_lds);  // OPEN: [NR]
    auto first_kept = reinterpret_cast<uint32_t(*)[S]>(place_lds);   // kList: [NR]
    auto tile_row = reinterpret_cast<int32_t(*)[L::kWid]>(place_lds);  // kTiles: [4]

    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int j = w / S;                                         // this group's step
    const int q = (w - j * S) * 64 + (int)(threadIdx.x & 63u);  // column of the strip
    const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t seg = b / g.nstrips, strip = b - seg * g.nstrips;
    const int nx = k.nx, ny = k.ny;
    const int out = L::kWid - 2 * g.halo;
    const int x0 = (int)strip * out, y0 = (int)seg * g.rows;
    const int rows = min(g.rows, ny - y0);
    const int xu = x0 - g.halo + q;  // before the periodic wrap
    int x = xu % nx;
    if (x < 0)
        x += nx;
    const uint32_t co = col_off(x);
    const bool keep = q >= g.halo && q < g.halo + out && xu < nx;
    const uint64_t row = (uint64_t)((uint32_t)k.pitch / kChunk) * (9u * kChunk);
    auto wrap_row = [&](int a) {
        a %= ny;
        return a < 0 ? a + ny : a;
    };

    // Source rows, numbered from node row y0 - K (group 0 loads them, one row
    // ahead: two ahead measured no faster and takes the registers that let two
    // workgroups share a CU).
    struct Row {
        M v[9];
        uint32_t ty, nm;
        float al;
        uint32_t n;  // sparse: node index (a neighbour's where there is no fluid node)
    } next;
    int ly = wrap_row(y0 - K);
    // sparse: chunk and tile entries of row ly, loaded one row before its nodes
    uint64_t fl = 0;
    uint32_t c_first = 0;
    int32_t tile = -1;
    auto load_index = [&]() {
        if constexpr (SPARSE) {
            const uint32_t c = (uint32_t)ly * ((uint32_t)k.pitch / kChunk) + ((uint32_t)x >> 6);
            fl = g.chunk_fluid[c];
            if constexpr (PLACE == kList)
                c_first = g.chunk_first[c];
            else
                tile = g.tile_of[((uint32_t)ly >> 4) * ((uint32_t)nx >> 4) + ((uint32_t)x >> 4)];
        }
    };
    auto load_row = [&]() {
        if constexpr (!SPARSE) {
            const M *__restrict__ s = k.src + (uint64_t)(uint32_t)ly * row;
#pragma unroll
            for (int i = 0; i < 9; ++i)
                next.v[i] = (s + (PLACE == kDenseOpp ? kOpp[i] : i) * (int)DS)[co];
            const uint32_t n = (uint32_t)ly * (uint32_t)k.pitch + (uint32_t)x;
            if constexpr (WALLS) {
                next.ty = k.type[n];
                next.nm = k.nmask[n];
            }
            if constexpr (DRAG)
                next.al = k.alpha[n];
            ly = ly + 1 == ny ? 0 : ly + 1;
        } else {
            const uint32_t bit = (uint32_t)x & 63u;
            const bool fluid = (fl >> bit) & 1u;
            uint32_t n, o;
            if constexpr (PLACE == kList) {
                // lanes without a fluid node read the next one's populations: no
                // line more than their neighbours touch, and nothing uses them
                n = min(c_first + (uint32_t)__popcll(fl & ((uint64_t(1) << bit) - 1u)),
                        g.n_fluid - 1u);
                o = list_base(n);
                const uint32_t inf = g.info[n];
                next.nm = inf;
                next.ty = fluid ? 0u : 1u;
            } else {
                const uint32_t lx = (uint32_t)x & 15u, l = (uint32_t)ly & 15u;
                const uint32_t t = tile < 0 ? 0u : (uint32_t)tile;
                n = t * (uint32_t)kTileNodes + l * 16u + lx;
                o = tile_base(t, tile_slot(lx, l));
                next.nm = k.nmask[n];
                next.ty = OPEN ? (uint32_t)k.type[n] : 0u;
                next.ty = fluid ? next.ty : (uint32_t)kSolid;
            }
            next.n = n;
            if (fluid || PLACE == kList) {
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    next.v[i] = k.src[(uint32_t)i * DS + o];
            }
            if constexpr (DRAG)
                next.al = k.alpha[n];
            ly = ly + 1 == ny ? 0 : ly + 1;
            load_index();
        }
    };
    int nput = 0;  // slot of the next row's node data
    // lane of this wavefront's first kept column
    const int kept0 = max(0, g.halo - (w - j * S) * 64);
    const int tile_shift = wrap_row(y0 - K) & 15;  // rows above the source's first in its tile
    int tput = tile_shift;
    auto put_row = [&](M (&d)[9][L::kLp]) {
#pragma unroll
        for (int i = 0; i < 9; ++i)
            d[i][q + 1] = next.v[i];
        if constexpr (WALLS) {
            // two byte stores: were the bytes joined, the compiler would do it
            // (and wait for the row's loads) right after issuing them
            uint8_t *b = reinterpret_cast<uint8_t *>(&node[nput][q]);
            if constexpr (PLACE == kList) {
                // info word: solid neighbours in bits 0-7, boundary code in 9-12
                const uint32_t code = (next.nm >> 9) & 15u;
                b[0] = (uint8_t)(next.ty ? (uint32_t)kSolid : code ? code + kOpen - 1u : (uint32_t)kFluid);
                b[1] = (uint8_t)next.nm;
            } else {
                b[0] = (uint8_t)next.ty;
                b[1] = (uint8_t)next.nm;
            }
        }
        if constexpr (DRAG)
            drag[nput][q] = next.al;
        if constexpr (SPARSE && OPEN) {
            index[nput][q] = next.n;
        } else if constexpr (PLACE == kList) {
            if ((int)(threadIdx.x & 63u) == kept0)
                first_kept[nput][w] = next.n;
        } else if constexpr (PLACE == kTiles) {
            tile_row[(tput >> 4) & 3][q] = (int32_t)(next.n / (uint32_t)kTileNodes);
            ++tput;
        }
        nput = nput + 1 == NR ? 0 : nput + 1;
    };

    M up[2][3], mid[3], own[9];
#pragma unroll
    for (int u = 0; u < 3; ++u)
        up[0][u] = up[1][u] = mid[u] = M(0);
#pragma unroll
    for (int i = 0; i < 9; ++i)
        own[i] = M(0);
    if (j == 0) {
        load_index();
        load_row();
        put_row(ring[0][0]);
        load_row();
    }
    uint32_t node_c = kFluid;  // node data of the row being updated
    double bv0 = 0.0, bv1 = 0.0;
    lds_barrier();

    // In iteration t group j reads row t - 2 j of its input and updates the row
    // before it.  It starts with row j, the first that later steps need, and is
    // done with row rows + 2 K - 1 - j.
    const int first = 3 * j, last = rows + 2 * K - 1 + j;
    int slot = 2 * j == 0 ? 0 : NR - 2 * j;  // of the node data of the row read
    int yo = y0 - (3 * K - 1);               // node row the last step writes in iteration t
    int yn = wrap_row(y0 - K - 2 * j);       // node row read in iteration t
    auto update = [&](auto par, const bool whole) {
        constexpr int p = decltype(par)::value;
        const M(&r)[9][L::kLp] = ring[j][p];
        M n[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            n[i] = r[i][q + 1 - kCx[i]];
        const uint32_t cd = node_c;
        float al = 0.0f;
        if constexpr (DRAG)
            al = drag[slot == 0 ? NR - 1 : slot - 1][q];
        M v[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            v[i] = kCy[i] > 0 ? up[p][kLineOf[i]] : kCy[i] == 0 ? mid[kLineOf[i]] : n[i];
        if constexpr (WALLS) {
            if (__ballot(cd != 0) != 0) {
                // bit 7 + i of the node data: x - c_i is solid
#pragma unroll
                for (int i = 1; i < 9; ++i)
                    v[i] = select_bits(v[i], own[kOpp[i]],
                                       (uint32_t)((int32_t)(cd << (24 - i)) >> 31));
            }
        }
        R f[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            f[i] = ST::ld(v[i], i);
        if constexpr (WALLS) {
            if constexpr (OPEN) {
                if (__ballot(cd != 0) != 0) {
                    if (const unsigned o = open_code((uint8_t)cd)) {
                        R a0, a1;
                        open_values<R, ST::kShift>(o, bv0, bv1, a0, a1);
                        apply_open_values<R, ST::kShift>(f, o, a0, a1);
                    }
                }
            }
            node_c = node[slot][q];
            if (__ballot(node_c != 0) != 0) {
                // boundary nodes in the next row: its own values, unshifted
#pragma unroll
                for (int i = 1; i < 9; ++i)
                    own[i] = kCx[i] == 0 ? n[i] : r[i][q + 1];
                if constexpr (OPEN) {
                    if (open_code((uint8_t)node_c)) {
                        const size_t n = SPARSE ? (size_t)index[slot][q]
                                                : (size_t)(uint32_t)yn * k.pitch + (uint32_t)x;
                        const double *v = k.bc_val + 2 * n;
                        bv0 = v[0];
                        bv1 = v[1];
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (kCy[i] > 0)
                up[p][kLineOf[i]] = n[i];
            else if (kCy[i] == 0)
                mid[kLineOf[i]] = n[i];
        }
        if (!whole)
            return;
        if constexpr (SPARSE) {
            if (__ballot((cd & 0xFFu) != kSolid) == 0)
                return;  // solid nodes only: nothing uses what they would get
        }
        collide<R, DRAG, ST::kShift, FORCE, ST::kExact, TRT, MRT>(f, k.omega, k.gx, k.gy,
                                                                 DRAG ? (R)al : R(0), k.rt);
        uint64_t kept_fluid = 0;
        if constexpr (PLACE == kList && !OPEN)
            kept_fluid = __ballot(keep && (cd & 0xFFu) != kSolid);
        if (j < K - 1) {
            M(&d)[9][L::kLp] = ring[j + 1][p ^ 1];
#pragma unroll
            for (int i = 0; i < 9; ++i)
                d[i][q + 1] = ST::st(f[i], i);
        } else if (keep && (cd & 0xFFu) != kSolid) {
            if constexpr (!SPARSE) {
                M *__restrict__ d = k.dst + (uint64_t)(uint32_t)yo * row;
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    store_nt(&(d + (PLACE == kDenseOpp ? kOpp[i] : i) * (int)DS)[co],
                             ST::st(f[i], i));
            } else {
                uint32_t o;
                if constexpr (PLACE == kList) {
                    const int sc = slot == 0 ? NR - 1 : slot - 1;
                    if constexpr (OPEN)
                        o = list_base(index[sc][q]);
                    else  // kept columns never cross the seam: count the fluid ones before
                        o = list_base(first_kept[sc][w - j * S] +
                                      __builtin_amdgcn_mbcnt_hi(
                                          (uint32_t)(kept_fluid >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)kept_fluid, 0u)));
                } else {
                    uint32_t t;
                    if constexpr (OPEN)
                        t = index[slot == 0 ? NR - 1 : slot - 1][q] / (uint32_t)kTileNodes;
                    else
                        t = (uint32_t)tile_row[((yo - y0 + K + tile_shift) >> 4) & 3][q];
                    o = tile_base(t, tile_slot((uint32_t)x & 15u, (uint32_t)yo & 15u));
                }
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    if constexpr (PLACE == kTiles)
                        k.dst[(uint32_t)i * DS + o] = ST::st(f[i], i);
                    else
                        store_nt(&k.dst[(uint32_t)i * DS + o], ST::st(f[i], i));
                }
            }
        }
    };
    const int T = rows + 3 * K - 1;
    auto iter = [&](auto par, const int t) {
        constexpr int p = decltype(par)::value;
        if (t >= first && t <= last)
            update(par, t >= first + 2);
        if (j == 0 && t < rows + 2 * K - 1) {
            put_row(ring[0][p ^ 1]);
            if (t < rows + 2 * K - 2)
                load_row();
        }
        slot = slot + 1 == NR ? 0 : slot + 1;
        if constexpr (OPEN)
            yn = yn + 1 == ny ? 0 : yn + 1;
        ++yo;
        lds_barrier();
    };
    for (int t = 0; t < T; t += 2) {
        iter(std::integral_constant<int, 0>{}, t);
        iter(std::integral_constant<int, 1>{}, t + 1);
    }
}

// ------------------------------------------------------------- small lattices --
// K steps of a small lattice: a workgroup owns an N x N square of nodes, one per
// lane, loads what the square stores, and exchanges the populations through LDS
// once per step (two copies, one barrier).  The square loses one ring of nodes per
// step and writes the (N - 2 K)^2 inner ones.  Strips need a wavefront row per step
// and iterate over the rows, so a lattice of some tens of thousands of nodes leaves
// them waiting on one row after the other; here every node of a step runs at once,
// and a launch takes little more than its one read of memory and K exchanges.
// Bounce-back values are the lane's own, still in registers.
template <class M, int N>
struct SquareLds {
    static constexpr int kPad = N + 1;  // the rows and columns beyond the square
    static constexpr int kPlane = N * N + 2 * kPad;
};

template <class ST, int PH, int PLACE, int N>
__global__ __launch_bounds__(N *N) void k_steps_square(const DenseArgs<ST> k, const StripGeom g)
{
    using R = typename ST::real;
    using M = typename ST::mem;
    using L = SquareLds<M, N>;
    constexpr bool DRAG = (PH & 3) == kDragged, FORCE = (PH & 3) != kBGK, TRT = (PH & kTRT) != 0,
                   MRT = (PH & kMRT) != 0, OPEN = (PH & kOpenBC) != 0;
    constexpr uint32_t DS = PLACE == kTiles ? kTileStride : kChunk;
    __shared__ M ring[2][9][L::kPlane];
    const int K = g.steps, out = N - 2 * K;
    const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    const int by = (int)(b / g.nstrips), bx = (int)(b - (uint32_t)by * g.nstrips);
    const int tx = (int)threadIdx.x % N, ty = (int)threadIdx.x / N;
    const int xu = bx * out - K + tx, yu = by * out - K + ty;  // before the periodic wrap
    int x = xu % k.nx, y = yu % k.ny;
    x = x < 0 ? x + k.nx : x;
    y = y < 0 ? y + k.ny : y;
    const bool keep = tx >= K && tx < N - K && ty >= K && ty < N - K && xu < k.nx && yu < k.ny;
    const uint32_t cpr = (uint32_t)k.pitch / kChunk;
    // the node's place, its index in the per-node arrays, and its types
    uint64_t o;
    uint32_t n, type, nm;
    if constexpr (PLACE == kList) {
        const uint32_t c = (uint32_t)y * cpr + ((uint32_t)x >> 6), bit = (uint32_t)x & 63u;
        const uint64_t fl = g.chunk_fluid[c];
        n = min(g.chunk_first[c] + (uint32_t)__popcll(fl & ((uint64_t(1) << bit) - 1u)),
                g.n_fluid - 1u);
        const uint32_t inf = g.info[n], code = (inf >> 9) & 15u;
        type = (fl >> bit) & 1u ? (code ? code + kOpen - 1u : (uint32_t)kFluid) : (uint32_t)kSolid;
        nm = inf & 0xFFu;
        o = list_base(n);
    } else if constexpr (PLACE == kTiles) {
        const int32_t t = g.tile_of[((uint32_t)y >> 4) * ((uint32_t)k.nx >> 4) + ((uint32_t)x >> 4)];
        const uint32_t lx = (uint32_t)x & 15u, l = (uint32_t)y & 15u, kt = t < 0 ? 0u : (uint32_t)t;
        n = kt * (uint32_t)kTileNodes + l * 16u + lx;
        type = t < 0 ? (uint32_t)kSolid : (uint32_t)k.type[n];
        nm = k.nmask[n];
        o = tile_base(kt, tile_slot(lx, l));
    } else {
        n = (uint32_t)y * (uint32_t)k.pitch + (uint32_t)x;
        type = k.type[n];
        nm = k.nmask[n];
        o = dense_base(x, y, cpr);
    }
    M v[9];
#pragma unroll
    for (int i = 0; i < 9; ++i)
        v[i] = k.src[(uint64_t)((PLACE == kDenseOpp ? kOpp[i] : i) * (int)DS) + o];
    R al = R(0), b0 = R(0), b1 = R(0);
    if constexpr (DRAG)
        al = (R)k.alpha[n];
    const unsigned code = open_code((uint8_t)type);
    if constexpr (OPEN) {
        if (code)
            open_values<R, ST::kShift>(code, k.bc_val[2 * (size_t)n], k.bc_val[2 * (size_t)n + 1],
                                       b0, b1);
    }
    auto store = [&](uint64_t d) {
        if (keep && type != kSolid) {
#pragma unroll
            for (int i = 0; i < 9; ++i)
                k.dst[d + (uint64_t)((PLACE == kDenseOpp ? kOpp[i] : i) * (int)DS) + o] = v[i];
        }
    };
    const int at = (int)threadIdx.x + L::kPad;
    // wavefronts without boundary nodes skip the bounce-back selects (us per step: 800^2
    // FP32 4.65 -> 4.48, FP64 alike); in the variants that the branch made
    // slower (16 bits 512^2 2.55 -> 3.03, FP32 with drag 1024 x 256 3.08 -> 3.19) all select
    constexpr bool kSkip = sizeof(M) == 8 || (sizeof(M) == 4 && !DRAG);
    const bool walls = __ballot(nm != 0 && type != kSolid) != 0;
    auto bounce = [&](int i) { return (uint32_t)((int32_t)(nm << (32 - i)) >> 31); };
    for (int t = 0; t < K; ++t) {
        M(&r)[9][L::kPlane] = ring[t & 1];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            r[i][at] = v[i];
        lds_barrier();
        // rows of this wavefront that no later step needs any more (or yet)
        const int lo = __builtin_amdgcn_readfirstlane(ty), hi = lo + (N >= 64 ? 1 : 64 / N) - 1;
        if (hi <= t || lo >= N - 1 - t)
            continue;
        R f[9];
        M pulled[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            pulled[i] = r[i][at - kCx[i] - N * kCy[i]];
            if constexpr (!kSkip) {
                if (i > 0)
                    pulled[i] = select_bits(pulled[i], v[kOpp[i]], bounce(i));
                f[i] = ST::ld(pulled[i], i);
            }
        }
        if constexpr (kSkip) {
            if (walls) {
#pragma unroll
                for (int i = 1; i < 9; ++i)
                    pulled[i] = select_bits(pulled[i], v[kOpp[i]], bounce(i));
            }
#pragma unroll
            for (int i = 0; i < 9; ++i)
                f[i] = ST::ld(pulled[i], i);
        }
        if constexpr (OPEN) {
            if (code)
                apply_open_values<R, ST::kShift>(f, code, b0, b1);
        }
        collide<R, DRAG, ST::kShift, FORCE, ST::kExact, TRT, MRT>(f, k.omega, k.gx, k.gy, al, k.rt);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            v[i] = ST::st(f[i], i);
        if (g.every && t < K - 1)
            store((uint64_t)t * g.every);
    }
    store((uint64_t)(K - 1) * g.every);
}

// ---------------------------------------------------------------- dispatch --

// Shapes of k_steps: the steps of strip_steps, in 128 VGPRs a lane for eight FP64 steps with
// S = 1, 64 otherwise with S = 2; the heavy variants' budgets at six are 168 and 84 (at
// eight they spill: FP32 MRT 71 us per step against 65 at 4096^2, FP64 with drag 169 against
// 130).  Six FP64 steps use S = 2, since a workgroup whose wavefronts are no multiple of
// four loads the SIMDs unevenly (FP64, six steps, S = 1: 190 us per step against 118).
template <class ST, int PH, int PLACE>
struct StepsShape {
    static constexpr bool kF64 = sizeof(typename ST::mem) == 8;
    static constexpr bool k16 = sizeof(typename ST::mem) == 2;
    static constexpr bool kSparse = PLACE >= kList;
    static constexpr bool kForce = (PH & 3) == kForced, kDrag = (PH & 3) == kDragged;
    static constexpr bool kOpens = (PH & kOpenBC) != 0;
    static constexpr bool kTwo = (PH & kTRT) != 0, kMulti = (PH & kMRT) != 0;
    static constexpr bool kHeavy = strip_heavy(kF64, kSparse, kForce, kDrag, kOpens, kTwo, kMulti);
    static constexpr bool kFull = kMulti && (kForce || kDrag) && (kOpens || kSparse);
    static constexpr int S = kF64 && !kHeavy ? 1 : 2;
    static constexpr int kMax =
        strip_steps(kF64, k16, kSparse, kForce, kDrag, kOpens, kTwo, kMulti);
    static constexpr int kWaves =  // per SIMD
        kF64 ? (kHeavy ? 3 : 4) : (kFull ? 3 : (kHeavy ? 6 : 8));
};

// Rows per workgroup.  A workgroup runs rows + 3 K - 1 iterations, so long strips
// waste least, but the grid should fill whole rounds of the chip: the time goes
// with the iterations times the rounds, where a last round that leaves CUs partly
// filled costs its share less 0.3 (one of two workgroups per CU: 0.65 of a full
// round; FP64 4096^2: 1462 blocks, 3 rounds, 103 us per step; 1548 blocks, 112;
// 1978, 103; 2064, 110).  Candidates: the strip lengths that end just under 1/2, 1,
// 2 .. 8 rounds.
inline int strip_rows(int ny, uint32_t nstrips, int K, int per_cu)
{
    constexpr int kCu = 256;
    int best_rows = ny;
    double best = 1e300;
    for (int c = 0; c <= 8; ++c) {
        const int64_t target = c == 0 ? kCu : (int64_t)c * kCu * per_cu;
        const int segs = (int)std::min<int64_t>(ny, std::max<int64_t>(1, target / nstrips));
        const int rows = (ny + segs - 1) / segs;
        const int64_t blocks = (int64_t)nstrips * ((ny + rows - 1) / rows);
        const int64_t full = blocks / (kCu * per_cu), rem = blocks % (kCu * per_cu);
        const double part =
            rem == 0 ? 0.0 : 0.3 + 0.7 * (double)((rem + kCu - 1) / kCu) / (double)per_cu;
        const double cost = ((double)full + part) * (double)(rows + 3 * K - 1);
        if (cost < best) {
            best = cost;
            best_rows = rows;
        }
    }
    return best_rows;
}

// Fails, with nothing launched, on a number of steps or a variant that no kernel is made for.
template <class ST, int PH, bool WALLS, int PLACE>
hipError_t steps_launch(const DevState &s, int cur, int K)
{
    using M = typename ST::mem;
    using R = typename ST::real;
    using Sh = StepsShape<ST, PH, PLACE>;
    constexpr int S = Sh::S;
    using L = StripLds<M, S>;
    const uint32_t bpr = (uint32_t)((s.nx + 255) / 256);
    const DenseArgs<ST> k{(const M *)s.f[cur],
                          (M *)s.f[1 - cur],
                          s.type,
                          s.nmask,
                          s.seg_interior,
                          s.alpha,
                          s.bc_val,
                          s.nx,
                          s.ny,
                          s.pitch,
                          bpr,
                          0u,
                          (R)s.omega,
                          (R)s.gx,
                          (R)s.gy,
                          Rates<R>{(R)s.omega_m, (R)s.s_e, (R)s.s_eps, (R)s.s_q},
                          0};
    StripGeom g;
    g.chunk_fluid = s.chunk_fluid;
    g.chunk_first = s.chunk_first;
    g.info = s.ind_info;
    g.tile_of = s.tile_of;
    g.n_fluid = (uint32_t)s.n_fluid;
    g.steps = K;
    g.every = s.every;
    int square = 0;
    const int most = square_steps(s.nx, s.ny, s.dtype, square);
    if (K < 2 || K > (square ? most : Sh::kMax) || (s.every && !square))
        return hipErrorInvalidValue;
    if (square) {
        const int in = square - 2 * K;
        g.nstrips = (uint32_t)((s.nx + in - 1) / in);
        const uint32_t blocks = g.nstrips * (uint32_t)((s.ny + in - 1) / in);
        if (square == 16)
            k_steps_square<ST, PH, PLACE, 16><<<blocks, 256, 0, s.stream>>>(k, g);
        else
            k_steps_square<ST, PH, PLACE, 32><<<blocks, 1024, 0, s.stream>>>(k, g);
        return hipGetLastError();
    }
    if constexpr (Sh::kMax > 0) {
        g.halo = K <= 4 ? 4 : 8;  // strips start at a multiple of 32 or 64 bytes (FP64)
        const int out = L::kWid - 2 * g.halo;
        g.nstrips = (uint32_t)((s.nx + out - 1) / out);
        const uint32_t lds = L::bytes(K, WALLS, (PH & 3) == kDragged, (PH & kOpenBC) != 0,
                                      PLACE);
        const int per_cu = std::max(1, std::min((int)(163840u / lds), Sh::kWaves * 4 / (S * K)));
        g.rows = strip_rows(s.ny, g.nstrips, K, per_cu);
        const uint32_t blocks = g.nstrips * (uint32_t)((s.ny + g.rows - 1) / g.rows);
        k_steps<ST, PH, WALLS, PLACE, S, Sh::kMax, Sh::kWaves>
            <<<blocks, (uint32_t)(64 * S * K), lds, s.stream>>>(k, g);
    }
    return hipGetLastError();
}

template <class ST, int COLL, int PLACE>
hipError_t steps_phys(const DevState &s, int cur, int K)
{
    const bool force = s.gx != 0.0 || s.gy != 0.0;
    if (s.open) {
        if (s.alpha)
            return steps_launch<ST, kDragged | kOpenBC | COLL, true, PLACE>(s, cur, K);
        if (force)
            return steps_launch<ST, kForced | kOpenBC | COLL, true, PLACE>(s, cur, K);
        return steps_launch<ST, kBGK | kOpenBC | COLL, true, PLACE>(s, cur, K);
    }
    if (s.alpha)
        return steps_launch<ST, kDragged | COLL, true, PLACE>(s, cur, K);
    if (force)
        return steps_launch<ST, kForced | COLL, true, PLACE>(s, cur, K);
    if constexpr (PLACE < kList) {
        if (s.interior_frac == 1.0)
            return steps_launch<ST, kBGK | COLL, false, PLACE>(s, cur, K);
    }
    return steps_launch<ST, kBGK | COLL, true, PLACE>(s, cur, K);
}

template <class ST, int PLACE>
hipError_t steps_placed(const DevState &s, int cur, int K)
{
    if (s.mrt)
        return steps_phys<ST, kMRT, PLACE>(s, cur, K);
    if (s.trt)
        return steps_phys<ST, kTRT, PLACE>(s, cur, K);
    return steps_phys<ST, 0, PLACE>(s, cur, K);
}

}  // namespace
}  // namespace lbm
