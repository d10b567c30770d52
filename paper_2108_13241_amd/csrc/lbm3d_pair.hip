// Two D3Q19 steps in one launch (dense A-B layout, and the AA layout after an odd
// number of steps, whose lattice is an A-B lattice with opposite slots exchanged).
//
// A step reads and writes 19 populations a node, so its time is that of the
// memory; k_pair3 reads and writes them once for two steps.  A workgroup owns some
// columns and marches along z.  In each plane it pulls the populations from the
// source lattice, collides and leaves the result in LDS; after one barrier every
// lane pulls its node of the plane before from LDS (populations of older planes
// are in its registers), collides again and stores.  The second step loses the
// outer ring of columns, which the neighbouring workgroups compute again.  The
// arithmetic is the single step's (collide3 and the storage conversion in between),
// so the result is bitwise that of two.
//
// Shape: one workgroup per CU with all the LDS that two planes need (the node's own
// values of the plane before, for bounce-back, are only read by their own lane, so
// two planes do for lattices with walls as well): 64 x 13 written columns of the
// 66 x 15 computed (FP64: 32 x 13 of 34 x 15).  The written columns are aligned, so
// that stores are whole lines; with 14 x 14 columns, whose stores are parts of
// lines, the memory rewrites each line twice and FP32 took 725 us per step at 256^3.
// Two groups of wavefronts, one per step, took 304 at 32 x 13, and two workgroups
// per CU 306; this shape 275.  It moves 2.7 GB per pair, 1.06 of the least, at 4.9
// TB/s: the vector units are busy 40 % of the time and the barrier keeps that from
// overlapping all of the memory's.
//
// us per step, single -> pairs: 256^3 FP32 421 -> 270, FP64 837 -> 534; 128^3 FP32
// 56 -> 40, FP64 120 -> 76; 192^3 with 40 % of its nodes in spheres and a force,
// FP32 265 -> 175, FP64 435 -> 299.
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "lbm3d_device.h"

namespace lbm3 {
namespace {

// A workgroup's columns: W written ones along x, aligned to W, and a ring of one
// around them.  Lanes 0 .. W * kHigh - 1 take rows of W, the last W lanes the
// ring's two columns, so that a wavefront's loads and stores are whole lines.
template <int N, int W>
struct Cols {
    static constexpr int kHigh = N / W - 1, kWide = W + 2;
    static constexpr int kNodes = kWide * kHigh;
    static constexpr int kRows = kHigh - 2;  // rows written
    static_assert(2 * kHigh <= W);
};

struct PairArgs {
    const void *src;
    void *dst;
    const uint8_t *type;
    const uint32_t *nmask;
    int nx, ny, nz, pitch;
    uint32_t tiles_x, tiles;
    int planes;  // planes a workgroup writes
};

// Slot of direction i among those of equal c_i.z (five up, nine level, five down).
__device__ constexpr int line_of(int i)
{
    int n = 0;
    for (int k = 0; k < i; ++k)
        n += kCz[k] == kCz[i];
    return n;
}

__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr uint32_t kSolidBit = 1u << 31;

template <class C, class M>
constexpr uint32_t pair_lds_bytes()
{
    return 2u * (uint32_t)(Q * C::kNodes) * (uint32_t)sizeof(M);
}

// OPP: the AA layout (population i in slot opp(i)).  LB: wavefronts per SIMD.
template <class ST, bool FORCE, bool TRT, bool MRT, bool WALLS, bool OPP, int N, int W, int LB>
__global__ __launch_bounds__(N, LB) void k_pair3(
    const PairArgs k, typename ST::real omega, typename ST::real gx, typename ST::real gy,
    typename ST::real gz, Rates3<typename ST::real> rt)
{
    using R = typename ST::real;
    using M = typename ST::mem;
    using C = Cols<N, W>;
    constexpr int kPlane = Q * C::kNodes;
    extern __shared__ __align__(16) unsigned char lds[];
    M *const plane = reinterpret_cast<M *>(lds);  // [2][Q][kNodes]

    const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t seg = b / k.tiles, tile = b - seg * k.tiles;
    const uint32_t by = tile / k.tiles_x, bx = tile - by * k.tiles_x;
    const int z0 = (int)seg * k.planes, P = min(k.planes, k.nz - z0);
    const uint32_t row = (uint32_t)k.pitch / kChunk * (uint32_t)(Q * kChunk);
    const uint64_t slab = (uint64_t)row * (uint32_t)k.ny;  // elements of a z plane
    auto slot = [](int i) { return (OPP ? kOpp[i] : i) * (int)kChunk; };

    int tx = (int)threadIdx.x % W + 1, ty = (int)threadIdx.x / W;
    if (ty == C::kHigh) {
        const int h = tx <= 2 * C::kHigh ? tx - 1 : 0;  // lanes past the end repeat the first
        tx = (h & 1) * (W + 1);
        ty = h / 2;
    }
    const int q = ty * C::kWide + tx;
    const int xu = (int)bx * W - 1 + tx, yu = (int)by * C::kRows - 1 + ty;  // before the wrap
    int x = xu % k.nx, y = yu % k.ny;
    x = x < 0 ? x + k.nx : x;
    y = y < 0 ? y + k.ny : y;
    const bool keep = tx > 0 && tx <= W && ty > 0 && ty <= C::kRows && xu < k.nx && yu < k.ny;
    const int q1 = keep ? q : C::kWide + 1;  // its neighbours are in the square
    uint32_t o[3][3];  // [dy + 1][dx + 1]: column offset inside a plane
    {
        const uint32_t c[3] = {col_off(wrap_dec(x, k.nx)), col_off(x), col_off(wrap_inc(x, k.nx))};
        const uint32_t r[3] = {(uint32_t)wrap_dec(y, k.ny) * row, (uint32_t)y * row,
                               (uint32_t)wrap_inc(y, k.ny) * row};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                o[a][d] = r[a] + c[d];
    }
    const M *__restrict__ src = (const M *)k.src;
    M *__restrict__ dst = (M *)k.dst;

    // plane number n is z0 - 1 + n; the first step computes 0 .. P + 1, the second
    // 1 .. P, one iteration later
    int z = z0 > 0 ? z0 - 1 : k.nz - 1;  // plane of the next populations
    int zn = z;                          // and of the next node data
    uint32_t ty_n = kFluid, nm_n = 0;
    auto load_node = [&]() {
        if constexpr (WALLS) {
            const uint32_t n = ((uint32_t)zn * (uint32_t)k.ny + (uint32_t)y) * (uint32_t)k.pitch + (uint32_t)x;
            ty_n = k.type[n];
            nm_n = k.nmask[n];
            zn = wrap_inc(zn, k.nz);
        }
    };
    M v[Q];
    uint32_t nm = 0, nm1 = 0;
    auto load_plane = [&]() {
        const M *p[3] = {src + slab * (uint32_t)wrap_dec(z, k.nz), src + slab * (uint32_t)z,
                         src + slab * (uint32_t)wrap_inc(z, k.nz)};
        nm = ty_n == kSolid ? kSolidBit : nm_n;
        load_node();
#pragma unroll
        for (int i = 0; i < Q; ++i)
            v[i] = (p[1 - kCz[i]] + slot(i))[o[1 - kCy[i]][1 - kCx[i]]];
        if constexpr (WALLS) {
            if (__ballot((nm & ~kSolidBit) != 0) != 0) {
                // bounce-back: the node's own opposite slot
#pragma unroll
                for (int i = 1; i < Q; ++i)
                    if ((nm >> (i - 1)) & 1u)
                        v[i] = (p[1] + slot(kOpp[i]))[o[1][1]];
            }
        }
        z = wrap_inc(z, k.nz);
    };
    M up[2][5], mid[9];
#pragma unroll
    for (int u = 0; u < 5; ++u)
        up[0][u] = up[1][u] = M(0);
#pragma unroll
    for (int u = 0; u < 9; ++u)
        mid[u] = M(0);
    auto iter = [&](auto par, const int t) {
        constexpr int p = decltype(par)::value;
        R f[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i)
            f[i] = ST::ld(v[i], i);
        const uint32_t nm2 = nm1;  // plane t - 1
        nm1 = nm;
        if (t <= P)
            load_plane();
        collide3<R, ST::kShift, FORCE, TRT, MRT>(f, omega, gx, gy, gz, rt);
#pragma unroll
        for (int i = 0; i < Q; ++i)
            plane[p * kPlane + i * C::kNodes + q] = ST::st(f[i], i);
        lds_barrier();
        M n[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i)
            n[i] = plane[p * kPlane + i * C::kNodes + q1 - kCx[i] - C::kWide * kCy[i]];
        if (t >= 2 && keep) {
            M w[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i)
                w[i] = kCz[i] > 0 ? up[p][line_of(i)] : kCz[i] == 0 ? mid[line_of(i)] : n[i];
            if constexpr (WALLS) {
                if (__ballot(nm2 != 0) != 0) {
                    // the node's own values of the plane before, which no other lane
                    // overwrites
#pragma unroll
                    for (int i = 1; i < Q; ++i)
                        if ((nm2 >> (i - 1)) & 1u)
                            w[i] = plane[(1 - p) * kPlane + kOpp[i] * C::kNodes + q1];
                }
            }
            R g[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i)
                g[i] = ST::ld(w[i], i);
            collide3<R, ST::kShift, FORCE, TRT, MRT>(g, omega, gx, gy, gz, rt);
            if (!(nm2 & kSolidBit)) {
                M *d = dst + slab * (uint32_t)(z0 + t - 2);
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    __builtin_nontemporal_store(ST::st(g[i], i), &(d + slot(i))[o[1][1]]);
            }
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (kCz[i] > 0)
                up[p][line_of(i)] = n[i];
            else if (kCz[i] == 0)
                mid[line_of(i)] = n[i];
        }
    };
    load_node();
    load_plane();
    int t = 0;
    for (; t < P + 1; t += 2) {
        iter(std::integral_constant<int, 0>{}, t);
        iter(std::integral_constant<int, 1>{}, t + 1);
    }
    if (t == P + 1)
        iter(std::integral_constant<int, 0>{}, t);
}

// Planes per workgroup: as few rounds of the chip as possible times the iterations
// (planes + 2).
inline int pair_planes(int nz, uint32_t tiles)
{
    constexpr int64_t kCu = 256;
    int best = nz;
    int64_t cost = INT64_MAX;
    for (int64_t rounds = 1; rounds <= 8; ++rounds) {
        const int64_t segs = std::min<int64_t>(nz, std::max<int64_t>(1, rounds * kCu / tiles));
        const int planes = (int)((nz + segs - 1) / segs);
        const int64_t blocks = (int64_t)tiles * ((nz + planes - 1) / planes);
        const int64_t c = (blocks + kCu - 1) / kCu * (planes + 2);
        if (c < cost) {
            cost = c;
            best = planes;
        }
    }
    return best;
}

inline bool forced(const State3 &s) { return s.gx != 0.0 || s.gy != 0.0 || s.gz != 0.0; }

template <class ST, bool FORCE, bool TRT, bool MRT, bool WALLS, bool OPP>
void pair_launch(const State3 &s, const void *src, void *dst)
{
    using M = typename ST::mem;
    using R = typename ST::real;
    constexpr int N = sizeof(M) == 8 ? 512 : 1024, W = sizeof(M) == 8 ? 32 : 64;
    using C = Cols<N, W>;
    constexpr int LB = N / 256;  // one workgroup per CU
    constexpr uint32_t lds = pair_lds_bytes<C, M>();
    PairArgs k;
    k.src = src;
    k.dst = dst;
    k.type = s.type;
    k.nmask = s.nmask;
    k.nx = s.nx;
    k.ny = s.ny;
    k.nz = s.nz;
    k.pitch = s.pitch;
    k.tiles_x = (uint32_t)((s.nx + W - 1) / W);
    k.tiles = k.tiles_x * (uint32_t)((s.ny + C::kRows - 1) / C::kRows);
    k.planes = pair_planes(s.nz, k.tiles);
    const uint32_t blocks = k.tiles * (uint32_t)((s.nz + k.planes - 1) / k.planes);
    k_pair3<ST, FORCE, TRT, MRT, WALLS, OPP, N, W, LB><<<blocks, N, lds, s.stream>>>(
        k, (R)s.omega, (R)s.gx, (R)s.gy, (R)s.gz,
        Rates3<R>{(R)s.omega_m, (R)s.s_e, (R)s.s_eps, (R)s.s_q, (R)s.s_pi, (R)s.s_m});
}

// pair_compiled3 has excluded what is not compiled here.
template <class ST, bool TRT, bool MRT, bool OPP>
void pair_phys(const State3 &s, const void *src, void *dst)
{
    if constexpr (sizeof(typename ST::mem) == 2) {
        pair_launch<ST, false, TRT, MRT, false, OPP>(s, src, dst);
    } else {
        // (MRT with a force: FP64 only)
        constexpr bool kForce = !MRT || sizeof(typename ST::mem) == 8;
        if (kForce && forced(s))
            pair_launch<ST, kForce, TRT, MRT, true, OPP>(s, src, dst);
        else if (s.interior_frac == 1.0)
            pair_launch<ST, false, TRT, MRT, false, OPP>(s, src, dst);
        else
            pair_launch<ST, false, TRT, MRT, true, OPP>(s, src, dst);
    }
}

template <class ST>
hipError_t pair_typed(const State3 &s, const void *src, void *dst)
{
    auto coll = [&](auto opp) {
        constexpr bool OPP = decltype(opp)::value;
        if (s.mrt)
            pair_phys<ST, false, true, OPP>(s, src, dst);
        else if (s.trt)
            pair_phys<ST, true, false, OPP>(s, src, dst);
        else
            pair_phys<ST, false, false, OPP>(s, src, dst);
    };
    if (s.aa)
        coll(std::true_type{});
    else
        coll(std::false_type{});
    return hipGetLastError();
}

}  // namespace

// The lattices that k_pair3 is compiled for: dense ones under the halfway rule, with the node
// offsets inside a z plane in 32 bits; 16-bit types without solid nodes and force, FP32
// MRT without a force (both slower than single steps otherwise, see below).
bool pair_compiled3(const State3 &s)
{
    if (s.list || s.blocks || s.fullway || !s.f[1] ||
        (uint64_t)s.ny * (uint32_t)s.pitch * Q >= (uint64_t(1) << 31))
        return false;
    if (s.dtype == LBM_F16_SHIFTED || s.dtype == LBM_BF16_SHIFTED)
        return s.interior_frac == 1.0 && !forced(s);
    return !(s.dtype == LBM_F32 && s.mrt && forced(s));
}

// The 32-bit and 64-bit types take pairs from the size on at which a pair beats two
// launches.  Measured, us per step, single against pairs: 32^3 FP32 4.9 / 4.8, with
// a force 4.1 / 6.4; 48^3 6.6 / 5.0 and 7.1 / 6.7.  Where most rows hold solid nodes
// 64^3 is even in FP32 (12.1 / 12.0) and better in FP64 (20 / 16), and on the AA layout,
// whose single step reads half as much there, still worse (9.5 / 11.4).  The 16-bit
// types pay the same arithmetic for half the bytes: pairs pay off only without solid
// nodes and force and once a lattice exceeds the 256 MB memory-side cache (200^3 141 /
// 119, 320^3 485 / 363; 160^3 61 / 66; walls and a force at 256^3 216 / 254).  MRT with
// a force in FP32 needs more registers than 16 wavefronts have (192^3 281 / 310).
// A single step skips rows without fluid nodes, in the cache or on the AA layout at little
// cost, so mostly solid lattices stay with it (spheres, fluid fraction 0.1 / 0.3 / 0.6): A-B
// FP32 96 x 80 x 64 11.6 / 16.4, 16.2 / 16.8, 18.2 / 16.9, but 128^3 67 / 42 and 84 / 49; AA FP64
// 128^3 42 / 67, 69 / 77, 90 / 82; AA FP32 96 x 80 x 64 11.9 / 16.2, 13.9 / 16.5, 14.7 / 16.8, 128^3
// 28 / 37, 44 / 44, 55 / 48, 256 x 256 x 128 97 / 131, 184 / 162, 240 / 177.
bool pair_supported3(const State3 &s)
{
    if (!pair_compiled3(s))
        return false;
    const uint64_t nodes = (uint64_t)s.ny * (uint32_t)s.pitch * (uint32_t)s.nz;
    if (s.dtype == LBM_F16_SHIFTED || s.dtype == LBM_BF16_SHIFTED)
        return nodes * Q * 2 > (uint64_t(256) << 20);
    if (s.interior_frac >= 0.9)
        return nodes >= (1u << 17);
    const bool f64 = s.dtype == LBM_F64;
    if (s.aa)
        return f64 ? nodes >= (1u << 19) && s.fluid_frac >= 0.45
                   : nodes >= (1u << 20) && s.fluid_frac >= 0.35;
    const bool cached = 2 * nodes * Q * (f64 ? 8 : 4) <= (uint64_t(256) << 20);
    return nodes >= (1u << 18) && (f64 || !cached || s.fluid_frac >= 0.45);
}

hipError_t launch_pair3(const State3 &s, int from)
{
    if (!pair_compiled3(s))
        return hipErrorInvalidValue;
    const void *src = s.f[from];
    void *dst = s.f[1 - from];
    switch (s.dtype) {
    case LBM_F64: return pair_typed<F64>(s, src, dst);
    case LBM_F32: return pair_typed<Shifted<float>>(s, src, dst);
    case LBM_F16_SHIFTED: return pair_typed<Shifted<_Float16>>(s, src, dst);
    case LBM_BF16_SHIFTED: return pair_typed<Shifted<__bf16>>(s, src, dst);
    }
    return hipErrorInvalidValue;
}

}  // namespace lbm3
