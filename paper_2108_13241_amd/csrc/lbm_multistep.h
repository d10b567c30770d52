// Several D2Q9 steps in one launch (dense A-B layout).
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
// Measured, Taylor-Green 4096^2, us per step (single steps before): FP64 400 -> 117
// (8 steps a launch), FP32 192 -> 61, FP16 103 -> 65.  The FP32 and 16-bit kernels are
// then bound by VALU issue (95 % of it at FP32), FP64 by VALU (0.6) and memory
// together.  A form that kept all K steps in one wavefront (rows in registers, lane
// shifts instead of LDS) ran FP64 125, FP32 68, FP16 75 at its best K = 4, 4, 2: K is
// bounded by the registers there, and boundary handling spilled them.
#pragma once

#include <algorithm>
#include <type_traits>

#include "lbm_dense.h"
#include "lbm_device.h"
#include "lbm_launch.h"

namespace lbm {
namespace {

struct StripGeom {
    uint32_t nstrips;
    int steps;  // K
    int halo;   // columns at each side of a strip that only feed it
    int rows;   // rows a workgroup updates
};

// Slot of direction i among those of equal c_i.y (rows kept in registers).
__device__ constexpr int kLineOf[9] = {0, 1, 0, 2, 0, 1, 2, 1, 2};

// Barrier that orders LDS only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS layout of a strip: rows between groups, then node types and drag
// coefficients of the rows in flight (the last step lags 2 K - 1 rows behind the
// source, and one row is being written).
template <class M, int S>
struct StripLds {
    static constexpr int kWid = 64 * S;
    static constexpr int kLp = kWid + 2;  // one column more at each end
    static __host__ __device__ constexpr int node_rows(int K) { return 2 * K + 2; }
    static __host__ __device__ constexpr uint32_t ring_bytes(int K)
    {
        return (uint32_t)(K * 2 * 9 * kLp) * (uint32_t)sizeof(M);
    }
    static __host__ __device__ constexpr uint32_t bytes(int K, bool walls, bool drag)
    {
        return ring_bytes(K) + (uint32_t)(node_rows(K) * kWid) * ((walls ? 2u : 0u) + (drag ? 4u : 0u));
    }
};

// WALLS = false: the lattice has interior fluid nodes only.  MAXK: the most
// groups a launch may have (block size 64 S K).  LB: wavefronts per SIMD the
// registers have to allow.
template <class ST, int PH, bool WALLS, int S, int MAXK, int LB>
__global__ __launch_bounds__(64 * MAXK * S, LB) void k_steps(const DenseArgs<ST> k,
                                                             const StripGeom g)
{
    using R = typename ST::real;
    using M = typename ST::mem;
    using L = StripLds<M, S>;
    constexpr bool DRAG = (PH & 3) == kDragged, FORCE = (PH & 3) != kBGK, TRT = (PH & kTRT) != 0,
                   MRT = (PH & kMRT) != 0, OPEN = (PH & kOpenBC) != 0;
    static_assert(WALLS || !OPEN, "open boundaries need the node types");
    extern __shared__ __align__(16) unsigned char lds[];
    const int K = g.steps, NR = L::node_rows(K);
    auto ring = reinterpret_cast<M(*)[2][9][L::kLp]>(lds);
    auto node = reinterpret_cast<uint16_t(*)[L::kWid]>(lds + L::ring_bytes(K));
    auto drag = reinterpret_cast<float(*)[L::kWid]>(
        lds + L::ring_bytes(K) + (WALLS ? (uint32_t)(NR * L::kWid) * 2u : 0u));

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
    } next;
    int ly = wrap_row(y0 - K);
    auto load_row = [&]() {
        const M *__restrict__ s = k.src + (uint64_t)(uint32_t)ly * row;
#pragma unroll
        for (int i = 0; i < 9; ++i)
            next.v[i] = (s + i * (int)kChunk)[co];
        const uint32_t n = (uint32_t)ly * (uint32_t)k.pitch + (uint32_t)x;
        if constexpr (WALLS) {
            next.ty = k.type[n];
            next.nm = k.nmask[n];
        }
        if constexpr (DRAG)
            next.al = k.alpha[n];
        ly = ly + 1 == ny ? 0 : ly + 1;
    };
    int nput = 0;  // slot of the next row's node data
    auto put_row = [&](M (&d)[9][L::kLp]) {
#pragma unroll
        for (int i = 0; i < 9; ++i)
            d[i][q + 1] = next.v[i];
        if constexpr (WALLS) {
            // two byte stores: were the bytes joined, the compiler would do it
            // (and wait for the row's loads) right after issuing them
            uint8_t *b = reinterpret_cast<uint8_t *>(&node[nput][q]);
            b[0] = (uint8_t)next.ty;
            b[1] = (uint8_t)next.nm;
        }
        if constexpr (DRAG)
            drag[nput][q] = next.al;
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
        R f[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            f[i] = ST::ld(kCy[i] > 0 ? up[p][kLineOf[i]] : kCy[i] == 0 ? mid[kLineOf[i]] : n[i], i);
        if constexpr (WALLS) {
            if (__ballot(cd != 0) != 0) {
                const uint32_t sm = cd >> 8;
#pragma unroll
                for (int i = 1; i < 9; ++i)
                    f[i] = (sm >> (i - 1)) & 1u ? ST::ld(own[kOpp[i]], i) : f[i];
                if constexpr (OPEN) {
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
                        const double *v = k.bc_val +
                                          2 * ((size_t)(uint32_t)yn * k.pitch + (uint32_t)x);
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
        collide<R, DRAG, ST::kShift, FORCE, ST::kExact, TRT, MRT>(f, k.omega, k.gx, k.gy,
                                                                 DRAG ? (R)al : R(0), k.rt);
        if (j < K - 1) {
            M(&d)[9][L::kLp] = ring[j + 1][p ^ 1];
#pragma unroll
            for (int i = 0; i < 9; ++i)
                d[i][q + 1] = ST::st(f[i], i);
        } else if (keep && (cd & 0xFFu) != kSolid) {
            M *__restrict__ d = k.dst + (uint64_t)(uint32_t)yo * row;
#pragma unroll
            for (int i = 0; i < 9; ++i)
                store_nt(&(d + i * (int)kChunk)[co], ST::st(f[i], i));
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

// ---------------------------------------------------------------- dispatch --

// Shapes of k_steps.  Eight steps in flight where the registers allow two
// workgroups of 8 S wavefronts per CU (128 VGPRs in FP64 with S = 1, 64 otherwise
// with S = 2); the variants with more live values (MRT, drag, open boundaries)
// take six, whose budgets are 168 and 84 (at eight they spill: FP32 MRT 71 us per
// step against 65 at 4096^2, FP64 with drag 169 against 130).  Six FP64 steps use
// S = 2, since a workgroup whose wavefronts are no multiple of four loads the
// SIMDs unevenly (FP64, six steps, S = 1: 190 us per step against 118).
template <class ST, int PH>
struct StepsShape {
    static constexpr bool kHeavy = (PH & (kMRT | kOpenBC)) != 0 || (PH & 3) == kDragged ||
                                   ((PH & kTRT) != 0 && (PH & 3) != kBGK);
    static constexpr bool kFull = (PH & kMRT) != 0 && (PH & kOpenBC) != 0 && (PH & 3) != kBGK;
    static constexpr bool kF64 = sizeof(typename ST::mem) == 8;
    static constexpr int S = kF64 && !kHeavy ? 1 : 2;
    static constexpr int kMax = kHeavy ? 6 : 8;
    static constexpr int kWaves =  // per SIMD
        kF64 ? (kHeavy ? 3 : 4) : (kFull ? 3 : (kHeavy ? 6 : 8));
};

// Rows per workgroup.  A workgroup runs rows + 3 K - 1 iterations, so long strips
// waste least, but the grid should fill whole rounds of the chip: the time goes
// with the iterations times the rounds, where a last round that leaves CUs partly
// filled costs its share less 0.3 (one of two workgroups per CU: 0.65 of a full
// round; FP64 4096^2: 1462 blocks, 3 rounds, 106 us per step; 1548 blocks, 114;
// 1978, 107; 2064, 112).  Candidates: the strip lengths that end just under 1/2, 1,
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

template <class ST, int PH, bool WALLS>
void steps_launch(const DevState &s, int cur, int K)
{
    using M = typename ST::mem;
    using R = typename ST::real;
    using Sh = StepsShape<ST, PH>;
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
    g.steps = K;
    g.halo = K <= 4 ? 4 : 8;  // strips start at a multiple of 32 or 64 bytes (FP64)
    const int out = L::kWid - 2 * g.halo;
    g.nstrips = (uint32_t)((s.nx + out - 1) / out);
    const uint32_t lds = L::bytes(K, WALLS, (PH & 3) == kDragged);
    const int per_cu = std::max(1, std::min((int)(163840u / lds), Sh::kWaves * 4 / (S * K)));
    g.rows = strip_rows(s.ny, g.nstrips, K, per_cu);
    const uint32_t blocks = g.nstrips * (uint32_t)((s.ny + g.rows - 1) / g.rows);
    k_steps<ST, PH, WALLS, S, Sh::kMax, Sh::kWaves>
        <<<blocks, (uint32_t)(64 * S * K), lds, s.stream>>>(k, g);
}

template <class ST, int COLL>
void steps_phys(const DevState &s, int cur, int K)
{
    const bool force = s.gx != 0.0 || s.gy != 0.0;
    if (s.open) {
        if (s.alpha)
            steps_launch<ST, kDragged | kOpenBC | COLL, true>(s, cur, K);
        else if (force)
            steps_launch<ST, kForced | kOpenBC | COLL, true>(s, cur, K);
        else
            steps_launch<ST, kBGK | kOpenBC | COLL, true>(s, cur, K);
    } else if (s.alpha) {
        steps_launch<ST, kDragged | COLL, true>(s, cur, K);
    } else if (force) {
        steps_launch<ST, kForced | COLL, true>(s, cur, K);
    } else if (s.interior_frac == 1.0) {
        steps_launch<ST, kBGK | COLL, false>(s, cur, K);
    } else {
        steps_launch<ST, kBGK | COLL, true>(s, cur, K);
    }
}

template <class ST>
hipError_t steps_typed(const DevState &s, int cur, int K)
{
    if (s.mrt)
        steps_phys<ST, kMRT>(s, cur, K);
    else if (s.trt)
        steps_phys<ST, kTRT>(s, cur, K);
    else
        steps_phys<ST, 0>(s, cur, K);
    return hipGetLastError();
}

}  // namespace
}  // namespace lbm
