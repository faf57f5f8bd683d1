// PLIC curvature of a VoF fill-level lattice on gfx950 (Sec. 4.1-4.2 and
// Appendix B of Lehmann & Gekle, arXiv 2006.12838), forward and backward.
//
// Layout: phi, kappa, grad_kappa, grad_phi are X*Y*Z floats, x fastest.  The
// lattice is cut into 64x4x4 tiles, the tiles into groups of 4 or 16 consecutive
// ones (more where that would make over 8192 groups).  A forward is two launches:
//  1. a streaming scan over the whole lattice, one workgroup per group, that
//     writes the zero result everywhere and records each tile's interface
//     bitmask (0 < phi < 1, away from the outer layer) with its prefix counts,
//     and, per group, a list of work items (8 interface cells of a tile each);
//  2. the work items, each interface cell on a group of 4 lanes (16 where items
//     are few): the wavefront finds its items through the groups' counts, a
//     group finds its cell from
//     the bitmask, stages its neighbourhood in LDS, and its lanes share out the
//     interface neighbours (their PLIC offsets and rows of the normal
//     equations).  One workgroup turns the groups' cell counts into first rows
//     for a later backward.
// Sums over the neighbours are formed in a fixed order, so results are bitwise
// reproducible.  No launch needs a cleared counter: nothing is reset first.
// The backward (after the same scan, or reusing its forward's records) stores
// each interface cell's 27 contributions in its row, rows in tile order; a
// direct gather, one workgroup per tile, sums for every cell next to the
// interface its sources' rows in a fixed order (tiles away from the interface
// get their zeros beside the work items); a fallback gather handles the tiles
// with a source whose row did not fit the workspace, recomputing those rows.
// The interface is one cell thick (about 0.2 % of a 256^3 sphere lattice), so
// the scan carries the HBM traffic and the list kernels the arithmetic.
//
// Floating-point contraction is limited to single expressions in this file,
// so the per-cell arithmetic gives the same bits in every kernel that inlines
// it (a contribution stored by the work items and one recomputed by the
// fallback gather are identical).
#pragma clang fp contract(on)

#include <hip/hip_runtime.h>

#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <unordered_map>

#include "plic_host.hpp"
#include "plic_math.hpp"

namespace plic {
namespace {

constexpr int TX = 64, TY = 4, TZ = 4;       // tile
constexpr int kTile = TX * TY * TZ;           // 1024 cells
constexpr int kThreads = 256;                 // 4 wave64
constexpr int kCellsPerThread = kTile / kThreads;
constexpr int kPersistentBlocks = 2048;
constexpr int kCellBlocks = 4096;             // wavefronts of the cell kernels: 4 per SIMD
constexpr int kGatherBlocks = 1792;           // workgroups of the direct gather: 7 per CU, all it holds
// wavefronts of a scanning workgroup, one tile each: 16, or 4 on lattices whose
// scan is no more than its latency (48 x 44 x 37: 5 us, against 8.5 with 16 on 7 CUs)
constexpr int kScanWaves = 16, kFewScanWaves = 4, kFewTiles = 4096;
constexpr int scan_waves(int ntiles) { return ntiles > kFewTiles ? kScanWaves : kFewScanWaves; }
constexpr int kMaxGroups = 8192;              // groups of tiles: 128 per lane of a wavefront that looks for items
constexpr int kFallbackBlocks = 256;            // one per CU of an MI355X

// fixed auxiliary vector r of Sec. 4.2 (non-collinear with the normal)
constexpr double kR0 = 0.56270900, kR1 = 0.32704452, kR2 = 0.75921047;

// neighbour q = (dz+1)*9 + (dy+1)*3 + (dx+1); centre q = 13
enum Normal : int { kNormalPY = PLIC_NORMAL_PY, kNormalCM = PLIC_NORMAL_CM };

__host__ __device__ constexpr int q_dx(int q) { return q % 3 - 1; }
__host__ __device__ constexpr int q_dy(int q) { return (q / 3) % 3 - 1; }
__host__ __device__ constexpr int q_dz(int q) { return q / 9 - 1; }

__device__ __forceinline__ bool is_iface(float p) { return p > 0.0f && p < 1.0f; }

// ---------------------------------------------------------------------------
// LDL^T factorisation and solve of the symmetric 5x5 normal equations
// (App. B.3).  The lower triangle of m holds M on entry and L on exit; dinv
// holds the reciprocals of D (0 for a dropped parameter), so that the solves
// (the fit and, in the backward, its adjoint) multiply instead of divide.
// Only the leading N = min(5, #points) parameters are fitted (reduced
// dimension, the rest stay 0); a pivot below pivot_rel times the largest
// diagonal entry of the leading block drops its parameter.  True when every
// pivot is at least kSteady of that entry: rounding of M is then not enlarged
// by more than about 1 / kSteady (to 1e-11 in FP64, 1e-5 in FP32).
// ---------------------------------------------------------------------------
template <class F> constexpr F kSteady = sizeof(F) == 8 ? F(1e-5) : F(0.0078125);

template <class F>
__device__ __forceinline__ bool ldlt_factor(F (&m)[5][5], int N, bool (&act)[5], F (&dinv)[5]) {
    F maxd = F(0);
#pragma unroll
    for (int j = 0; j < 5; ++j)
        if (j < N) maxd = M<F>::fmax(maxd, m[j][j]);
    const F tol = M<F>::pivot_rel * maxd;
    bool steady = true;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        F dj = m[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) dj -= m[j][k] * m[j][k] * m[k][k];
        act[j] = (j < N) && (dj > tol) && (maxd > F(0));
        steady = steady && (j >= N || dj >= kSteady<F> * maxd);
        const F inv = act[j] ? F(1) / dj : F(0);
        m[j][j] = act[j] ? dj : F(0);
        dinv[j] = inv;
#pragma unroll
        for (int i = j + 1; i < 5; ++i) {
            F sij = m[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) sij -= m[i][k] * m[j][k] * m[k][k];
            m[i][j] = sij * inv;
        }
    }
    return steady;
}

template <class F>
__device__ __forceinline__ void ldlt_solve(const F (&m)[5][5], const bool (&act)[5], const F (&dinv)[5],
                                           const F (&rhs)[5], F (&x)[5]) {
    F y[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        F t = rhs[j];
#pragma unroll
        for (int k = 0; k < j; ++k) t -= m[j][k] * y[k];
        y[j] = act[j] ? t : F(0);
    }
#pragma unroll
    for (int j = 4; j >= 0; --j) {
        F t = y[j] * dinv[j];
#pragma unroll
        for (int i = j + 1; i < 5; ++i) t -= m[i][j] * x[i];
        x[j] = act[j] ? t : F(0);
    }
}

// mean curvature of the paraboloid at the origin (App. B.2), negated so that a
// fluid drop (normal pointing out of the fluid) is positive
template <class F>
__device__ __forceinline__ F kappa_of(const F (&a)[5]) {
    const F A = a[0], B = a[1], C = a[2], H = a[3], I = a[4];
    const F w = H * H + I * I + F(1);
    return -(A * (I * I + F(1)) + B * (H * H + F(1)) - C * H * I) / (w * M<F>::sqrt(w));
}

// a value through an opaque move: what a loop derives from it is then
// recomputed in every iteration (a few ALU instructions) instead of being kept
// in registers across the loop, where it would spill
__device__ __forceinline__ int opaque(int v) {
    int t;
    asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"(v));
    return t;
}
__device__ __forceinline__ int thread_index_per_iteration() { return opaque(static_cast<int>(threadIdx.x)); }

// lower-triangle index of the 5x5 normal matrix
__host__ __device__ constexpr int tri(int i, int k) { return i * (i + 1) / 2 + k; }

// weight of neighbour offset e in the fill-level gradient (App. B.1):
// Parker-Youngs 4 / 2 / 1 for |e|^2 = 1 / 2 / 3, centre of mass 1
template <int NRM>
__host__ __device__ constexpr int nrm_weight(int e2) {
    return NRM == kNormalCM ? 1 : (e2 == 1 ? 4 : (e2 == 2 ? 2 : 1));
}

// fill-level gradient of the 3^3 neighbourhood centred at LDS index c
template <int NRM, class T>
__device__ __forceinline__ void gradient27(const float* __restrict__ s, int c, int sy, int sz, T& gx, T& gy, T& gz) {
    gx = T(0); gy = T(0); gz = T(0);
#pragma unroll
    for (int q = 0; q < 27; ++q) {
        if (q == 13) continue;
        const int e2 = q_dx(q) * q_dx(q) + q_dy(q) * q_dy(q) + q_dz(q) * q_dz(q);
        const T w = T(nrm_weight<NRM>(e2)) * T(s[c + q_dz(q) * sz + q_dy(q) * sy + q_dx(q)]);
        gx += T(q_dx(q)) * w;
        gy += T(q_dy(q)) * w;
        gz += T(q_dz(q)) * w;
    }
}

// ---------------------------------------------------------------------------
// One interface cell on a group of kLanes = 4 lanes.  About ten of a cell's
// 26 neighbours are interface cells, and only those have a point: the group
// lists them (the centre among them) by a bitmask, and lane j takes the list's
// entries j, j + kLanes, ...  So the lanes that solve a PLIC problem are nearly
// always full, where one lane per slot of the 3x3x3 leaves six of ten idle; and
// what is computed once per cell (normal, frame, LDL^T, kappa) is repeated on
// few lanes.  The fit's sums run over the entries of each lane in list order
// and then over the group by lane permutations, always in the same order, so
// every call gives the same bits.  Bound by instruction issue and the latency
// of its chains: with 16 lanes per cell, two slots each, a spray of 24 drops
// (512 x 384 x 384, mixed precision) took 183 us forward and 308 us adjoint,
// the 256^3 sphere 16.4 us forward; with 4 lanes 88, 188 (the gradient's zeros,
// 14 us, included) and 14 us.
// An ill-conditioned fit shows the rounding of its sums in its result, many
// times enlarged.  Where a pivot falls below kSteady of the largest diagonal
// entry, the sums are formed again over the 16 pairs of neighbours (l, l + 16)
// of the 26 in order, so that they do not depend on how the lanes shared out
// the list (one such cell moved by 5e-5 of the spray's whole gradient).  Cells on
// 4 lanes are then done again four at a time on 16 lanes each: on their own 4 lanes,
// whose wavefront waits for them, a 100 x 98 x 99 lattice's forward and backward
// took 47.2 us instead of 44.0, a 120 x 118 x 119 one's 44.7 instead of 42.6.  Cells on 16
// lanes form them at once, from the points that are there: done again from the
// start, the forward of a 64^3 lattice with specks in 2 % of its cells took 17.8 us
// instead of 15.2, of a 32^3 one with specks in 20 % 18.6 instead of 15.6.
// ---------------------------------------------------------------------------
constexpr int kRowFloatsH = 26 * 3;             // a cell's adjoints of its neighbours' own gradients
constexpr unsigned kCentre = 1u << 13;
constexpr int kLanes = 4;                       // lanes per interface cell
constexpr int kWideLanes = 16;                  // where cells are few
constexpr int kWaveCells = 64 / kLanes;         // cells of a wavefront
constexpr int kRounds = (27 + kLanes - 1) / kLanes;

// scratch of one wavefront: the offsets of each lane's entries by round; the
// neighbour offsets (x, y, z) with their weights in the gradient (taken apart
// from q each time, they were a twelfth of the instructions); with ADJ, the
// gradients of the points' fill levels by neighbour, and the centre's
// own derivatives
template <class T, class F> union OffsetLds {
    T D[kRounds][64];
    struct {                                    // a call with 16 lanes per cell has two rounds of offsets,
        T D[2][64];                             // and room for two entries' terms of each cell's sums
        F terms[64 / kWideLanes][2 * 20];
    } wide;
};
template <bool OWN> struct OwnLds {};
template <> struct OwnLds<true> {
    float4 own[kRounds][64];                    // each entry's own normal and its factor 1 / |h| (0: the centre's)
};
template <class T, class F, bool ADJ, bool OWN = false> struct CellLds : OwnLds<OWN> {
    OffsetLds<T, F> o;
    float4 e[27];
};
template <class T, class F, bool OWN> struct CellLds<T, F, true, OWN> : OwnLds<OWN> {
    OffsetLds<T, F> o;
    float4 e[27];
    T pb[kWaveCells][27];
    T cen[kWaveCells][4];
    int4 at[kWaveCells];                        // place and row (kept here, not in registers, for a second call)
};

// Neighbour normals: an adjoint in FP32 points keeps each entry's own normal from
// its PLIC problem for its point and its adjoint (they were formed three times,
// from 26 levels each): 36.2 -> 30.4 us for 5 drops in 150 x 131 x 118, forward
// and backward of the spray 966 -> 906 us.  Its 7 KiB leave the two wavefronts
// per SIMD that its registers allow; a forward would drop from four to two (the
// 5 drops 29.0 -> 25.7 us, but the spray 258 -> 297), an FP64 adjoint from two to
// one.
template <class T, bool ADJ, bool NBR> constexpr bool kKeepOwn = NBR && ADJ && sizeof(T) == 4;

template <int NRM, class Lds> __device__ __forceinline__ void init_cells(Lds& L, int lane) {
    if (lane < 27) {
        const int dx = q_dx(lane), dy = q_dy(lane), dz = q_dz(lane);
        L.e[lane] = make_float4(dx, dy, dz, nrm_weight<NRM>(dx * dx + dy * dy + dz * dz));
    }
    __syncwarp();
}

template <int CTRL> __device__ __forceinline__ float quad_move(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ double quad_move(double x) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ unsigned quad_move(unsigned x) {
    return static_cast<unsigned>(__builtin_amdgcn_mov_dpp(static_cast<int>(x), CTRL, 0xF, 0xF, true));
}
// quad_perm [1,0,3,2] and [2,3,0,1]; each row of 16 turned up by 4 and by 8
// lanes; the row's last lane to all of it; lane i of 8 to lane 7 - i
constexpr int kSwap1 = 0xB1, kSwap2 = 0x4E, kTurn4 = 0x124, kTurn8 = 0x128, kLast = 0x15F, kHalfMirror = 0x141;

// Sums over a group's entries, the same bits for 4 lanes and for 16: partial
// sum j runs over the entries j, j + 4, j + 8, ... in that order.  With 4 lanes
// it is lane j's own.  With 16, lane j + 4 r has entry j + 4 r of each run of 16,
// and the partial sums go around the row: added to by the entry of the lane
// they are on, then turned to the next four lanes.  add() adds this lane's entry
// (zeros where it has none) to acc; more: there is another run of 16.
template <int LANES, int N, class F, class Add>
__device__ __forceinline__ void add_entries(F (&acc)[N], bool more, Add add) {
    add();
    if constexpr (LANES == kWideLanes) {
        auto turn = [&] {
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = quad_move<kTurn4>(acc[i]);
        };
#pragma unroll
        for (int r = 1; r < 4; ++r) { turn(); add(); }
        if (more) turn();                       // uniform per group
    }
}
// the four partial sums together, on every lane of the group (of 16: those of
// the last four lanes, which the last entries were added to)
template <int LANES, class F> __device__ __forceinline__ F group_sum(F x) {
    x += quad_move<kSwap1>(x);
    x += quad_move<kSwap2>(x);
    if constexpr (LANES == kWideLanes) x = quad_move<kLast>(x);
    return x;
}

// inclusive sums over the lanes below, in each half of the wavefront or all of
// it, by row shifts and row broadcasts (every lane active); through LDS
// (__shfl_up) a step of these costs about a hundred cycles of latency
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned scan_step(unsigned x) {
    return x + static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ unsigned half_scan(unsigned x) {
    x = scan_step<0x111, 0xF>(x);                 // row_shr 1, 2, 4, 8
    x = scan_step<0x112, 0xF>(x);
    x = scan_step<0x114, 0xF>(x);
    x = scan_step<0x118, 0xF>(x);
    return scan_step<0x142, 0xA>(x);              // row_bcast 15 into rows 1 and 3
}
__device__ __forceinline__ unsigned wave_scan(unsigned x) {
    return scan_step<0x143, 0xC>(half_scan(x));   // row_bcast 31 into rows 2 and 3
}
__device__ __forceinline__ unsigned from_lane(unsigned x, int lane) {   // lane: the same on every lane
    return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), lane));
}

// the k-th set bit of word (k below its count)
__device__ __forceinline__ int nth_bit(unsigned word, int k) {
    int bit = 0;
#pragma unroll
    for (int st = 16; st; st >>= 1) {
        const int low = __popc(word & ((1u << st) - 1u));
        const bool up = k >= low;
        k -= up ? low : 0;
        bit += up ? st : 0;
        word >>= up ? st : 0;
    }
    return bit;
}

// lane j's entries of the list, one after the other: j, j + LANES, ...
template <int LANES> struct Entries;
template <> struct Entries<kLanes> {
    unsigned rest;
    __device__ __forceinline__ Entries(unsigned list, int j) : rest(list) {
#pragma unroll
        for (int i = 0; i < kLanes - 1; ++i) rest = i < j ? rest & (rest - 1u) : rest;
    }
    __device__ __forceinline__ bool any() const { return rest != 0u; }      // this lane has one
    __device__ __forceinline__ bool has() const { return true; }
    __device__ __forceinline__ bool more() const { return false; }
    __device__ __forceinline__ int q() const { return __ffs(static_cast<int>(rest)) - 1; }
    __device__ __forceinline__ void next() {
#pragma unroll
        for (int i = 0; i < kLanes; ++i) rest &= rest - 1u;
    }
};
template <> struct Entries<kWideLanes> {
    unsigned list;
    int e, j;
    __device__ __forceinline__ Entries(unsigned l, int lane) : list(l), e(lane), j(lane) {}
    __device__ __forceinline__ bool any() const { return e - j < __popc(list); }            // a lane of the group has one
    __device__ __forceinline__ bool has() const { return e < __popc(list); }
    __device__ __forceinline__ bool more() const { return e - j + kWideLanes < __popc(list); }
    __device__ __forceinline__ int q() const { return has() ? nth_bit(list, e) : 13; }
    __device__ __forceinline__ void next() { e += kWideLanes; }
};

// neighbour q's point (x, y in the frame, z along n), centre normal
template <class T, class F>
__device__ __forceinline__ void cell_point(const float4& e, T D, T D0, T bx0, T bx1, T bx2, T by0, T by1, T by2,
                                           T n0, T n1, T n2, F& x, F& y, F& z) {
    const T ex = T(e.x), ey = T(e.y), ez = T(e.z);
    x = F(ex * bx0 + ey * bx1 + ez * bx2);
    y = F(ex * by0 + ey * by1 + ez * by2);
    z = F(ex * n0 + ey * n1 + ez * n2 + (D - D0));
}

// where a cell lies in the lattice (the neighbour-normal variant asks whether
// its neighbours' 3^3 does too)
struct Place {
    int x, y, z, X, Y, Z;
};

// neighbour-normal variant: the normal of interface neighbour q's plane, its
// own -h / |h| (h its 3^3 fill-level gradient) when its 3^3 lies in the lattice
// and h does not vanish, else the centre normal that m holds on entry (the rule
// of the oracle's variant)
template <int NRM, class T>
__device__ __forceinline__ void own_normal(const float* __restrict__ s, int c, int sy, int sz, int q,
                                           const Place& at, T (&m)[3], bool& own, T& ih_out) {
    const int dx = q_dx(q), dy = q_dy(q), dz = q_dz(q);
    const int ax = at.x + dx, ay = at.y + dy, az = at.z + dz;
    const bool inside = ax >= 1 && ay >= 1 && az >= 1 && ax <= at.X - 2 && ay <= at.Y - 2 && az <= at.Z - 2;
    if (inside) {
        T hx, hy, hz;
        gradient27<NRM, T>(s, c + dz * sz + dy * sy + dx, sy, sz, hx, hy, hz);
        const T h2 = hx * hx + hy * hy + hz * hz;
        if (h2 >= T(1e-24)) {
            const T ih = M<T>::rcp(M<T>::sqrt(h2));
            m[0] = -hx * ih; m[1] = -hy * ih; m[2] = -hz * ih;
            own = true;
            ih_out = ih;
        }
    }
}

// neighbour-normal variant: neighbour q's point, the foot of its own plane
// e + D m - D0 n, in the frame
template <class T, class F>
__device__ __forceinline__ void cell_point_own(const float4& e, T D, T D0, const T (&m)[3], T bx0, T bx1, T bx2,
                                               T by0, T by1, T by2, T n0, T n1, T n2, F& x, F& y, F& z) {
    const T P0 = T(e.x) + D * m[0] - D0 * n0, P1 = T(e.y) + D * m[1] - D0 * n1, P2 = T(e.z) + D * m[2] - D0 * n2;
    x = F(P0 * bx0 + P1 * bx1 + P2 * bx2);
    y = F(P0 * by0 + P1 * by1 + P2 * by2);
    z = F(P0 * n0 + P1 * n1 + P2 * n2);
}

// The fit's 20 sums over the pairs of neighbours (l, l + 16) of the 26 in
// order, for the few cells that need them so, on 16 lanes: lane l has the
// terms of pair l.  They go through LDS, two pairs at a time, and each lane adds up one
// or two of the 20 sums.
template <class F, class Point>
__device__ __forceinline__ void ordered_sums(int l, unsigned mask, unsigned list, Point point, F (&terms)[2 * 20],
                                             F (&sum)[20]) {
    const int qa = l < 13 ? l : l + 1, qb = min(l + 17, 26);
    F xa = F(0), ya = F(0), za = F(0), xb = F(0), yb = F(0), zb = F(0);
    if ((mask >> qa) & 1u) point(qa, __popc(list & ((1u << qa) - 1u)), xa, ya, za);
    if (l < 10 && ((mask >> qb) & 1u)) point(qb, __popc(list & ((1u << qb) - 1u)), xb, yb, zb);
    const int i0 = l, i1 = min(16 + l, 19);
    F acc0 = F(0), acc1 = F(0);
    __syncwarp();
#pragma unroll 1
    for (int b = 0; b < 8; ++b) {
        if (l / 2 == b) {
            F* t = terms + (l % 2) * 20;
            const F Qa[5] = {xa * xa, ya * ya, xa * ya, xa, ya}, Qb[5] = {xb * xb, yb * yb, xb * yb, xb, yb};
#pragma unroll
            for (int i = 0; i < 5; ++i) {
#pragma unroll
                for (int k = 0; k <= i; ++k) t[tri(i, k)] = Qa[i] * Qa[k] + Qb[i] * Qb[k];
                t[15 + i] = za * Qa[i] + zb * Qb[i];
            }
        }
        __syncwarp();
        acc0 += terms[i0]; acc0 += terms[20 + i0];
        acc1 += terms[i1]; acc1 += terms[20 + i1];
        __syncwarp();
    }
    terms[i0] = acc0;
    terms[i1] = acc1;
    __syncwarp();
#pragma unroll
    for (int k = 0; k < 20; ++k) sum[k] = terms[k];
    __syncwarp();
}

// The groups of 4 lanes that were not done, four of the wavefront at a time on
// 16 lanes each: again(src) with the first lane of such a group, or -1 where none is
// left.  Every lane of the wavefront must call it.
template <class Again>
__device__ __forceinline__ void redo_groups(bool done, int lane, Again again) {
    static_assert(kLanes == 4, "every fourth lane is the first of its group");
    for (unsigned long long left = __ballot(!done) & 0x1111111111111111ull; left;) {
        int src = -1;
#pragma unroll
        for (int k = 0; k < 64 / kWideLanes; ++k, left &= left - 1ull)
            if (lane / kWideLanes == k) src = __ffsll(left) - 1;
        __syncwarp();
        again(src);
        __syncwarp();
    }
}

// s: LDS fill levels, c: centre index, sy/sz: LDS strides, lane: lane in the
// wavefront, LANES per cell.  Every lane of the group must call it.  False, with
// nothing written, when the fit is ill-conditioned on 4 lanes:
// the caller then calls it again on 16 with ORDERED (from the fill levels:
// with both kinds of sums in one call, what had to be kept in registers for the
// second made the first slower, 38.4 -> 42.0 us for a 220 x 218 x 219 forward).
// kappa: the same bits on every lane.  With ADJ,
// also writes out[q * ostride] = gk * d kappa / d phi_q (q = 0..26), with the
// interface mask, the PLIC cases and the active fit parameters held fixed.
// With NBR (neighbour normals: each interface neighbour's point from its own
// normal m = -h / |h|), out holds the derivative with every m held fixed, and
// outh[3t .. 3t+2] = gk * d kappa / d h of neighbour slot t (the 26 offsets
// other than the centre; zero where the neighbour keeps the centre normal);
// spreading that over the neighbour's 3^3 is left to the gathers.
template <int LANES, bool ORDERED, int SOLVER, class T, class U, class F, bool ADJ, int NRM, bool NBR = false>
__device__ __forceinline__ bool curv_cell(const float* __restrict__ s, int c, int sy, int sz, int lane,
                                          float gk, float* __restrict__ out, unsigned ostride,
                                          float* __restrict__ outh, CellLds<T, F, ADJ, kKeepOwn<T, ADJ, NBR>>& L,
                                          float& kappa,
                                          const Place& where = {}) {
    using mt = M<T>;
    constexpr int kPasses = (27 + LANES - 1) / LANES;
    const int j = lane % LANES, cell = lane / LANES;
    T gx, gy, gz;
    gradient27<NRM, T>(s, c, sy, sz, gx, gy, gz);
    // (strides 3 and 9, known at compile time: the 27 levels are in a row)
    auto at = [&](int q) { return sy == 3 && sz == 9 ? c - 13 + q : c + q_dz(q) * sz + q_dy(q) * sy + q_dx(q); };
    // interface mask of the 27 cells, 7 tests per lane (2 with 16 lanes)
    unsigned mask = 0u;
#pragma unroll
    for (int k = 0; k < kPasses; ++k) {
        const int q = j + k * LANES;
        if (is_iface(s[at(min(q, 26))]) && q < 27) mask |= 1u << (k * LANES);
    }
    mask <<= j;
    mask |= quad_move<kSwap1>(mask);
    mask |= quad_move<kSwap2>(mask);
    if constexpr (LANES == kWideLanes) {
        mask |= quad_move<kTurn4>(mask);
        mask |= quad_move<kTurn8>(mask);
    }
    mask &= ~kCentre;
    const unsigned list = mask | kCentre;
    const T gn2 = gx * gx + gy * gy + gz * gz;
    if (!(gn2 >= T(1e-24))) {                   // no usable normal: kappa = 0 (uniform per group)
        if constexpr (ADJ) {
            for (int q = j; q < 27; q += LANES) out[static_cast<unsigned>(q) * ostride] = 0.0f;
            if constexpr (NBR)
                for (int t = j; t < 78; t += LANES) outh[t] = 0.0f;
        }
        kappa = 0.0f;
        return true;
    }
    const T ign = mt::rcp(mt::sqrt(gn2));
    const T n0 = -gx * ign, n1 = -gy * ign, n2 = -gz * ign;
    // local frame (Sec. 4.2): b_z = n, b_y = n x r / |n x r|, b_x = b_y x b_z
    T r0 = T(kR0), r1 = T(kR1), r2 = T(kR2);
    T u0 = n1 * r2 - n2 * r1, u1 = n2 * r0 - n0 * r2, u2 = n0 * r1 - n1 * r0;
    T un2 = u0 * u0 + u1 * u1 + u2 * u2;
    if (un2 < T(1e-12)) {
        r0 = T(kR1); r1 = T(kR2); r2 = T(kR0);
        u0 = n1 * r2 - n2 * r1; u1 = n2 * r0 - n0 * r2; u2 = n0 * r1 - n1 * r0;
        un2 = u0 * u0 + u1 * u1 + u2 * u2;
    }
    const T iun = mt::rcp(mt::sqrt(un2));
    const T by0 = u0 * iun, by1 = u1 * iun, by2 = u2 * iun;
    const T bx0 = by1 * n2 - by2 * n1, bx1 = by2 * n0 - by0 * n2, bx2 = by0 * n1 - by1 * n0;
    // PLIC offsets of the entries with the centre normal (neighbour normals:
    // each interface neighbour with its own)
    int k = 0;
#pragma unroll 1
    for (Entries<LANES> en(list, j); en.any() && en.has(); en.next(), ++k) {
        const int q = en.q();
        const T p = T(s[at(q)]);
        if constexpr (NBR) {
            T mq[3] = {n0, n1, n2}, ih;
            bool own = false;
            if (q != 13) own_normal<NRM, T>(s, c, sy, sz, q, where, mq, own, ih);
            if constexpr (kKeepOwn<T, ADJ, NBR>)
                L.own[k][lane] = make_float4(mq[0], mq[1], mq[2], own ? ih : 0.0f);
            L.o.D[k][lane] = offset<SOLVER, T, U>(mq[0], mq[1], mq[2], p);
        } else {
            L.o.D[k][lane] = offset<SOLVER, T, U>(n0, n1, n2, p);
        }
    }
    __syncwarp();
    const int c13 = __popc(mask & (kCentre - 1u));          // the centre's place in the list
    const T D0 = L.o.D[c13 / LANES][(lane & ~(LANES - 1)) + c13 % LANES];
    F sum[20];
#pragma unroll
    for (int i = 0; i < 20; ++i) sum[i] = F(0);
    // the point of neighbour q, whose offset is entry e of the list
    auto point = [&](int q, int e, F& x, F& y, F& z) {
        const T D = L.o.D[e / LANES][(lane & ~(LANES - 1)) + e % LANES];
        if constexpr (NBR) {
            T mq[3] = {n0, n1, n2};
            if constexpr (kKeepOwn<T, ADJ, NBR>) {
                const float4 m = L.own[e / LANES][(lane & ~(LANES - 1)) + e % LANES];
                mq[0] = m.x; mq[1] = m.y; mq[2] = m.z;
            } else {
                bool own = false;
                T ih;
                own_normal<NRM, T>(s, c, sy, sz, q, where, mq, own, ih);
            }
            cell_point_own<T, F>(L.e[q], D, D0, mq, bx0, bx1, bx2, by0, by1, by2, n0, n1, n2, x, y, z);
        } else {
            cell_point<T, F>(L.e[q], D, D0, bx0, bx1, bx2, by0, by1, by2, n0, n1, n2, x, y, z);
        }
    };
    if constexpr (!ORDERED) {
        int e = j;
#pragma unroll 1
        for (Entries<LANES> en(list, j); en.any(); en.next(), e += LANES) {
            const int q = en.q();
            if (LANES == kLanes && q == 13) continue;
            F x = F(0), y = F(0), z = F(0);
            if (LANES == kLanes || q != 13) point(q, e, x, y, z);
            const F Q[5] = {x * x, y * y, x * y, x, y};
            add_entries<LANES>(sum, en.more(), [&] {
#pragma unroll
                for (int i = 0; i < 5; ++i) {
#pragma unroll
                    for (int l = 0; l <= i; ++l) sum[tri(i, l)] += Q[i] * Q[l];
                    sum[15 + i] += z * Q[i];
                }
            });
        }
#pragma unroll
        for (int i = 0; i < 20; ++i) sum[i] = group_sum<LANES>(sum[i]);
    } else {
        static_assert(LANES == kWideLanes, "lane l has pair l");
        ordered_sums<F>(j, mask, list, point, L.o.wide.terms[cell], sum);
    }
    const int npts = __popc(mask);
    F m[5][5], b[5];
    bool act[5];
    F a[5], dinv[5];
    auto factor = [&] {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            b[i] = sum[15 + i];
#pragma unroll
            for (int l = 0; l <= i; ++l) m[i][l] = sum[tri(i, l)];
        }
        return ldlt_factor<F>(m, npts < 5 ? npts : 5, act, dinv);
    };
    const bool steady = factor();
    if constexpr (!ORDERED) {
        if (!steady) {
            if constexpr (LANES == kLanes) return false;
            ordered_sums<F>(j, mask, list, point, L.o.wide.terms[cell], sum);
            factor();
        }
    }
    ldlt_solve<F>(m, act, dinv, b, a);
    kappa = float(kappa_of<F>(a));
    if constexpr (ADJ) {
        // d kappa / d(A,B,C,H,I), kappa = -(A(I^2+1) + B(H^2+1) - CHI) / W^(3/2)
        const F A = a[0], B = a[1], C = a[2], H = a[3], I = a[4];
        const F W = H * H + I * I + F(1);
        const F iW32 = F(1) / (W * M<F>::sqrt(W));
        const F num = A * (I * I + F(1)) + B * (H * H + F(1)) - C * H * I;
        const F g = -F(gk);
        F abar[5];
        abar[0] = g * (I * I + F(1)) * iW32;
        abar[1] = g * (H * H + F(1)) * iW32;
        abar[2] = g * (-H * I) * iW32;
        abar[3] = g * ((F(2) * B * H - C * I) * iW32 - F(3) * num * H * iW32 / W);
        abar[4] = g * ((F(2) * A * I - C * H) * iW32 - F(3) * num * I * iW32 / W);
#pragma unroll
        for (int i = 0; i < 5; ++i) abar[i] = act[i] ? abar[i] : F(0);
        F lam[5];
        ldlt_solve<F>(m, act, dinv, abar, lam);              // M symmetric: lambda = M^-1 abar
        // each point: zbar = lam.Q, Qbar = lam (z - a.Q) - a (lam.Q); the frame's
        // adjoint rows of a lane's points add up
        F arow[10];
#pragma unroll
        for (int i = 0; i < 10; ++i) arow[i] = F(0);
        k = 0;
#pragma unroll 1
        for (Entries<LANES> en(list, j); en.any(); en.next(), ++k) {
            const int q = en.q();
            T xbar = T(0), ybar = T(0), zt = T(0);              // the point's adjoint and what it multiplies
            T v0 = T(0), v1 = T(0), v2 = T(0), w0 = T(0), w1 = T(0), w2 = T(0);
            if (LANES == kLanes || en.has()) {
                const T p = T(s[at(q)]), D = L.o.D[k][lane];
                T mq[3] = {n0, n1, n2}, ih = T(0);
                bool own = false;
                if constexpr (kKeepOwn<T, ADJ, NBR>) {
                    const float4 m = L.own[k][lane];
                    mq[0] = m.x; mq[1] = m.y; mq[2] = m.z;
                    ih = m.w;
                    own = ih != 0.0f;
                } else if constexpr (NBR) {
                    if (q != 13) own_normal<NRM, T>(s, c, sy, sz, q, where, mq, own, ih);
                }
                T cq[3];
                const T dv = offset_grad_from_d0<T>(mq[0], mq[1], mq[2], p, D, cq);   // 1/A, centroid
                if (q == 13) {
                    L.cen[cell][0] = cq[0]; L.cen[cell][1] = cq[1]; L.cen[cell][2] = cq[2]; L.cen[cell][3] = dv;
                    if constexpr (LANES == kLanes) continue;
                } else {
                    F x, y, z;
                    if constexpr (NBR) cell_point_own<T, F>(L.e[q], D, D0, mq, bx0, bx1, bx2, by0, by1, by2, n0, n1, n2, x, y, z);
                    else cell_point<T, F>(L.e[q], D, D0, bx0, bx1, bx2, by0, by1, by2, n0, n1, n2, x, y, z);
                    const F Q[5] = {x * x, y * y, x * y, x, y};
                    F zq = F(0), aQ = F(0);
#pragma unroll
                    for (int i = 0; i < 5; ++i) { zq += lam[i] * Q[i]; aQ += a[i] * Q[i]; }
                    F Qbar[5];
#pragma unroll
                    for (int i = 0; i < 5; ++i) Qbar[i] = lam[i] * (z - aQ) - a[i] * zq;
                    xbar = T(F(2) * x * Qbar[0] + y * Qbar[2] + Qbar[3]);
                    ybar = T(F(2) * y * Qbar[1] + x * Qbar[2] + Qbar[4]);
                    zt = T(zq);
                    const T ex = T(L.e[q].x), ey = T(L.e[q].y), ez = T(L.e[q].z);
                    if constexpr (NBR) {
                        // x = P.b_x, y = P.b_y, z = P.n with P = e + D m - D0 n, D = d0(phi_q, m)
                        v0 = ex + D * mq[0] - D0 * n0; v1 = ey + D * mq[1] - D0 * n1; v2 = ez + D * mq[2] - D0 * n2;
                        const T Pb0 = xbar * bx0 + ybar * by0 + zt * n0;
                        const T Pb1 = xbar * bx1 + ybar * by1 + zt * n1;
                        const T Pb2 = xbar * bx2 + ybar * by2 + zt * n2;
                        const T Dbar = Pb0 * mq[0] + Pb1 * mq[1] + Pb2 * mq[2];
                        const T mb0 = D * Pb0 + Dbar * cq[0], mb1 = D * Pb1 + Dbar * cq[1], mb2 = D * Pb2 + Dbar * cq[2];
                        L.pb[cell][q] = Dbar * dv;
                        // n enters through z = P.n, through -D0 n in P, and as m where the neighbour keeps it
                        w0 = zt * v0 - D0 * Pb0 + (own ? T(0) : mb0);
                        w1 = zt * v1 - D0 * Pb1 + (own ? T(0) : mb1);
                        w2 = zt * v2 - D0 * Pb2 + (own ? T(0) : mb2);
                        // m = -h / |h|: the adjoint of h, gathered later at that neighbour
                        // and spread over its 3^3 by the gradient's weights
                        const T md = mq[0] * mb0 + mq[1] * mb1 + mq[2] * mb2;
                        float* o = outh + 3 * (q < 13 ? q : q - 1);
                        o[0] = own ? float(-(mb0 - mq[0] * md) * ih) : 0.0f;
                        o[1] = own ? float(-(mb1 - mq[1] * md) * ih) : 0.0f;
                        o[2] = own ? float(-(mb2 - mq[2] * md) * ih) : 0.0f;
                    } else {
                        L.pb[cell][q] = zt * dv;
                        v0 = ex; v1 = ey; v2 = ez;
                        w0 = ex + cq[0]; w1 = ey + cq[1]; w2 = ez + cq[2];
                    }
                }
            }
            add_entries<LANES>(arow, en.more(), [&] {
                arow[0] += F(xbar * v0); arow[1] += F(xbar * v1); arow[2] += F(xbar * v2);
                arow[3] += F(ybar * v0); arow[4] += F(ybar * v1); arow[5] += F(ybar * v2);
                if constexpr (NBR) {
                    arow[6] += F(w0); arow[7] += F(w1); arow[8] += F(w2);
                } else {
                    arow[6] += F(zt * w0); arow[7] += F(zt * w1); arow[8] += F(zt * w2);
                }
                arow[9] += F(zt);
            });
        }
        __syncwarp();
        T asum[10];
#pragma unroll
        for (int i = 0; i < 10; ++i) asum[i] = T(group_sum<LANES>(arow[i]));
        const T c00 = L.cen[cell][0], c01 = L.cen[cell][1], c02 = L.cen[cell][2], dvc = L.cen[cell][3];
        const T sbx0 = asum[0], sbx1 = asum[1], sbx2 = asum[2], sz_ = asum[9];
        // the centre offset D0 enters every z with a minus sign
        T nb0 = asum[6] - sz_ * c00, nb1 = asum[7] - sz_ * c01, nb2 = asum[8] - sz_ * c02;
        // b_x = b_y x n
        const T yb0 = asum[3] + (n1 * sbx2 - n2 * sbx1);
        const T yb1 = asum[4] + (n2 * sbx0 - n0 * sbx2);
        const T yb2 = asum[5] + (n0 * sbx1 - n1 * sbx0);
        nb0 += sbx1 * by2 - sbx2 * by1;
        nb1 += sbx2 * by0 - sbx0 * by2;
        nb2 += sbx0 * by1 - sbx1 * by0;
        // b_y = u / |u|, u = n x r
        const T bd = by0 * yb0 + by1 * yb1 + by2 * yb2;
        const T ub0 = (yb0 - by0 * bd) * iun, ub1 = (yb1 - by1 * bd) * iun, ub2 = (yb2 - by2 * bd) * iun;
        nb0 += r1 * ub2 - r2 * ub1;
        nb1 += r2 * ub0 - r0 * ub2;
        nb2 += r0 * ub1 - r1 * ub0;
        // n = -g / |g|
        const T nd = n0 * nb0 + n1 * nb1 + n2 * nb2;
        const T gb0 = -(nb0 - n0 * nd) * ign, gb1 = -(nb1 - n1 * nd) * ign, gb2 = -(nb2 - n2 * nd) * ign;
#pragma unroll
        for (int kk = 0; kk < kPasses; ++kk) {
            const int q = j + kk * LANES;
            if (q < 27) {
                const float4 e = L.e[q];
                const bool on = (mask >> q) & 1u;
                const T ph = on ? L.pb[cell][q] : T(0);
                const float v = float(ph + T(e.w) * (T(e.x) * gb0 + T(e.y) * gb1 + T(e.z) * gb2));
                out[static_cast<unsigned>(q) * ostride] = q == 13 ? float(-sz_ * dvc) : v;
                if constexpr (NBR) {
                    if (!on && q != 13) {
                        float* o = outh + 3 * (q < 13 ? q : q - 1);
                        o[0] = 0.0f; o[1] = 0.0f; o[2] = 0.0f;
                    }
                }
            }
        }
    }
    return true;
}

// ---------------------------------------------------------------------------
// Fill levels of a box [x0-H, x0+TX+H) x ... into LDS, every load issued
// before the first store (out-of-lattice cells read as 0).
// ---------------------------------------------------------------------------
template <int RX, int RY, int RZ>
__device__ __forceinline__ void load_region(float* __restrict__ s, const float* __restrict__ phi, int gx0,
                                            int gy0, int gz0, int X, int Y, int Z) {
    constexpr int R = RX * RY * RZ, IT = (R + kThreads - 1) / kThreads;
    float v[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int i = threadIdx.x + it * kThreads;
        const int lx = i % RX, ly = (i / RX) % RY, lz = i / (RX * RY);
        const int gx = gx0 + lx, gy = gy0 + ly, gz = gz0 + lz;
        v[it] = 0.0f;
        if (i < R && gx >= 0 && gx < X && gy >= 0 && gy < Y && gz >= 0 && gz < Z)
            v[it] = phi[(static_cast<int64_t>(gz) * Y + gy) * X + gx];
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int i = threadIdx.x + it * kThreads;
        if (i < R) s[i] = v[it];
    }
}

// Ordered compaction: appends every i in [0, n) with pred(i) to out, in
// increasing i; returns the count (same on every thread).  Block-wide.
template <class Pred>
__device__ __forceinline__ int ordered_compact(int n, Pred pred, unsigned short* out, int* wcount) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int cnt = 0;
    for (int base = 0; base < n; base += kThreads) {
        const int i = base + tid;
        const bool is = i < n && pred(i);
        const unsigned long long bal = __ballot(is);
        if (lane == 0) wcount[wave] = __popcll(bal);
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            before += w < wave ? wcount[w] : 0;
            total += wcount[w];
        }
        if (is) {
            const unsigned long long below = lane ? (bal & ((~0ull) >> (64 - lane))) : 0ull;
            out[cnt + before + __popcll(below)] = static_cast<unsigned short>(i);
        }
        cnt += total;
        __syncthreads();
    }
    return cnt;
}

// ---------------------------------------------------------------------------
// Workspace (caller device memory, 4-byte aligned):
//   [0, 256)  header: [2] overflow tiles, [16..] activity of lattices of 1 or 2 tiles
//   flags     ntiles      interface cells in the tile
//   grows     ntiles      first contribution row of each group (the prefix of
//                         the groups' cell counts in order; before that pass
//                         the counts themselves)
//   mask      32 ntiles   interface bit of each of the tile's 1024 cells
//   prefix    32 ntiles   set bits of mask before word w; word 0, where that
//                         is 0, holds the interface cells of the group before
//                         the tile
//   items     128 ntiles  work items (tile << 7 | part), 8 interface cells
//                         each, every group's from its first tile's place on
//   gitems    ntiles      work items of each group; then, 64 bits per 64 tiles,
//                         the tiles with an interface cell in their 3x3x3
//                         tiles (backward)
//   over      ntiles      the gather's tiles with a source cell without a row
//   contrib   the rest:   27 floats per row (backward contributions), entry q
//             of every row together (index q * rows + row): the gather's lanes
//             read entry q of neighbouring cells' rows at once
// mask and prefix are written, and read, only for tiles with interface cells.
// The fixed part (everything but contrib) is 784 bytes per tile.
// The backward stores the 27 contributions of an interface cell in its row
// when that fits; cells beyond the capacity are recomputed by the fallback
// gather, so every workspace size >= the fixed part is correct and a larger
// one is faster.
// ---------------------------------------------------------------------------
constexpr int kPartCells = 8;                 // interface cells per work item
constexpr int kMaxParts = kTile / kPartCells; // 128
constexpr int kWords = kTile / 32;            // mask words per tile
constexpr size_t kFixedPerTile = sizeof(unsigned) * (1 + 1 + kWords + kWords + kMaxParts + 1 + 1);
constexpr size_t kRowBytes = 27 * sizeof(float);
constexpr size_t kDefaultRowsPerTile = 16;    // contribution rows budgeted per tile by default
// rows are 32-bit indices: the groups' first rows saturate at kRowCap, so that
// such a row plus a cell's rank in its group (below 2^21: at most 2048 tiles)
// never wraps and is past the store, so the cell is recomputed; the
// capacity is at most kRowLimit rows, so an entry's index q * rows + row stays
// below 2^30 (a 32-bit byte offset from the store's base)
constexpr unsigned kRowCap = 0xF0000000u;
constexpr int64_t kMaxTiles = int64_t(1) << 24;      // see check_lattice
constexpr int64_t kMaxGroupTiles = kScanWaves * ((kMaxTiles + kScanWaves * kMaxGroups - 1) / (kScanWaves * kMaxGroups));
static_assert(kRowCap + kMaxGroupTiles * kTile < int64_t(1) << 32);
constexpr unsigned kRowLimit = (1u << 30) / 27u;
// The neighbour-normal variant's backward: a row holds the 27 contributions
// and, per neighbour, the adjoint of that neighbour's own fill-level gradient
// (26 x 3, together, after the contributions of all rows), followed in the
// workspace by one 3-vector per row, the sum of those adjoints at the row's cell
constexpr int kRowFloatsNbr = 27 + kRowFloatsH;
constexpr size_t kRowBytesNbr = (kRowFloatsNbr + 3) * sizeof(float);
constexpr unsigned kRowLimitNbr = (1u << 30) / kRowFloatsNbr;
// budgeted per tile by default: without a fallback a missing row is NaN, so
// the default leaves room for interfaces that cross a tile several times
constexpr size_t kDefaultRowsPerTileNbr = 64;

constexpr int kOverflow = 2;                    // header word: overflow tiles

struct Workspace {
    unsigned* counter;  // header
    unsigned* flags;
    unsigned* grows;
    unsigned* mask;
    unsigned* prefix;
    unsigned* items;
    unsigned* gitems;
    unsigned* over;
    float* contrib;
    float* hbar;        // neighbour-normal backward: 3 floats per row
    unsigned* act;      // activity, 2 words per 64 tiles
    unsigned rows;      // contribution capacity
    int per;            // tiles per group
    int groups;
    int segs;           // runs of 64 tiles
};

// 16 bytes at any 4-byte boundary (one access on gfx950)
struct Four {
    float v[4];
};

typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// 4 consecutive cells along x, those inside the lattice
__device__ __forceinline__ void store_four(float* __restrict__ out, int x, int y, int z, int X, int Y, int Z,
                                           const Four& r) {
    if (x < X && y < Y && z < Z) {
        float* p = out + (static_cast<int64_t>(z) * Y + y) * X + x;
        if (x + 4 <= X) {
            __builtin_memcpy(p, &r, sizeof(r));
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (x + k < X) p[k] = r.v[k];
        }
    }
}

// ---------------------------------------------------------------------------
// 1. streaming scan, one workgroup per group of tiles: zero output everywhere
// (ZERO: the forward; the backward's gather writes the zeros), each tile's
// interface count; of the tiles with interface cells the bitmask, the set bits
// before each of its words and the work items; the group's counts.  A wavefront
// takes a tile (one more per round where a group has over 16): lane l handles,
// in layer u = 0..3, the 4 consecutive cells 4l .. 4l+3.  Bound by HBM: many
// short workgroups stream faster than wavefronts that walk over several tiles
// with the next one's loads in flight (97 against 111 us for 512 x 384 x 384).
// The zeros are non-temporal stores: they are not read again, and 256 MB of
// last-level cache then keep phi, which is (256^3, repeated: 17 against 24 us).
// ---------------------------------------------------------------------------
template <bool ZERO, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_curv_scan(const float* __restrict__ phi, float* __restrict__ out,
                                                          Workspace ws, int X, int Y, int Z, int ntx, int nty,
                                                          int ntiles) {
    __shared__ unsigned count[WAVES];
    const int g = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gfirst = g * ws.per, glast = min(gfirst + ws.per, ntiles);
    unsigned* items = ws.items + static_cast<size_t>(gfirst) * kMaxParts;
    unsigned nitems = 0u, ncells = 0u;                        // of the rounds before
    for (int r0 = gfirst; r0 < glast; r0 += WAVES) {
        const int tile = r0 + wave;
        unsigned total = 0u;
        if (tile < glast) {                                   // uniform per wavefront
            const int x0 = (tile % ntx) * TX, y0 = ((tile / ntx) % nty) * TY, z0 = (tile / (ntx * nty)) * TZ;
            const int x = x0 + (lane % 16) * 4, y = y0 + lane / 16;
            float v[4][4];
            if (x0 + TX <= X && y0 + TY <= Y && z0 + TZ <= Z) {
                const int64_t at = (static_cast<int64_t>(z0) * Y + y) * X + x, plane = static_cast<int64_t>(Y) * X;
#pragma unroll
                for (int u = 0; u < 4; ++u) __builtin_memcpy(v[u], phi + at + u * plane, 16);
                if constexpr (ZERO) {
                    const float4u zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        __builtin_nontemporal_store(zero, reinterpret_cast<float4u*>(out + at + u * plane));
                }
            } else {
                // cells outside the lattice read one inside (no branch, whose
                // join would wait for each load; the mask leaves them out)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float* p = phi + (static_cast<int64_t>(min(z0 + u, Z - 1)) * Y + min(y, Y - 1)) * X;
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[u][k] = p[min(x + k, X - 1)];
                }
                if constexpr (ZERO) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) store_four(out, x, y, z0 + u, X, Y, Z, Four{{0.0f, 0.0f, 0.0f, 0.0f}});
                }
            }
            unsigned nib[4], some = 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                nib[u] = 0u;
                const bool yz_in = y >= 1 && y <= Y - 2 && z0 + u >= 1 && z0 + u <= Z - 2;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    nib[u] |= (yz_in && x + k >= 1 && x + k <= X - 2 && is_iface(v[u][k])) ? (1u << k) : 0u;
                some |= nib[u];
            }
            if (__any(some != 0u)) {                          // uniform
                // mask word 8u + l / 8 from the nibbles of 8 lanes, then word l
                // to lane l and the set bits before it
                unsigned mw = 0u;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    unsigned w = nib[u] << (4 * (lane % 8));
                    w |= quad_move<kSwap1>(w);
                    w |= quad_move<kSwap2>(w);
                    w |= quad_move<kHalfMirror>(w);
                    const unsigned o = __shfl(w, (lane % 8) * 8, 64);
                    mw = lane / 8 == u ? o : mw;
                }
                const unsigned c = __popc(mw), incl = half_scan(c);
                total = from_lane(incl, kWords - 1);
                if (lane < kWords) {
                    ws.mask[static_cast<size_t>(tile) * kWords + lane] = mw;
                    if (lane) ws.prefix[static_cast<size_t>(tile) * kWords + lane] = incl - c;
                }
            }
        }
        if (lane == 0) count[wave] = total;
        __syncthreads();
        // the round's tiles, one per lane: the cells and items before each
        const unsigned mine = lane < WAVES ? count[lane] : 0u, parts = (mine + kPartCells - 1) / kPartCells;
        const unsigned cells = wave_scan(mine), its = wave_scan(parts);
        if (wave == 0 && lane < WAVES && r0 + lane < glast) {
            ws.flags[r0 + lane] = mine;
            if (mine) ws.prefix[static_cast<size_t>(r0 + lane) * kWords] = ncells + cells - mine;
        }
        const unsigned n = from_lane(parts, wave), before = nitems + from_lane(its, wave) - n;
        for (unsigned p = static_cast<unsigned>(lane); p < n; p += 64u)
            items[before + p] = (static_cast<unsigned>(tile) << 7) | p;
        ncells += from_lane(cells, 63);
        nitems += from_lane(its, 63);
        if (r0 + WAVES < glast) __syncthreads();         // count reused by the next round
    }
    if (threadIdx.x == 0) {
        ws.gitems[g] = nitems;
        ws.grows[g] = ncells;
        if (g == 0) ws.counter[kOverflow] = 0u;
    }
}

// First rows of the groups, by one wavefront: lane l takes a run of consecutive
// groups.  Rows go to the interface cells in tile order, saturated at kRowCap,
// so the cells that get a row for a given workspace size are always the same.
__device__ __forceinline__ void group_rows(const Workspace& ws) {
    const int lane = threadIdx.x, run = (ws.groups + 63) / 64, g0 = lane * run;
    const unsigned* cells = ws.grows;
    unsigned long long sum = 0ull;
#pragma unroll 8
    for (int k = 0; k < run; ++k) sum += g0 + k < ws.groups ? cells[g0 + k] : 0u;
    unsigned long long before = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long o = __shfl_up(before, d, 64);
        if (lane >= d) before += o;
    }
    before -= sum;
    for (int k = 0; k < run; ++k) {
        if (g0 + k >= ws.groups) break;
        const unsigned c = cells[g0 + k];
        ws.grows[g0 + k] = static_cast<unsigned>(before < kRowCap ? before : kRowCap);
        before += c;
    }
}

__global__ __launch_bounds__(64) void k_curv_rows(Workspace ws) { group_rows(ws); }

// The work items in one sequence: lane l owns the groups l, l + 64, ... and the
// items go by lane, then by group.  A wavefront sums its lanes' groups once
// (256^3: 16 coalesced loads) and finds any item from that: there is no list
// over the whole lattice, so no counter to clear first and none that every tile
// would have to wait for (one word's atomics are served one at a time, about 12
// ns each: over 9000 tiles with interface cells, half of the scan's time).
struct ItemFinder {
    unsigned mine, before, total;       // items of this lane's groups, of lower lanes, of all

    __device__ __forceinline__ static unsigned of_group(const Workspace& ws, int g) {
        return g < ws.groups ? ws.gitems[g] : 0u;
    }

    __device__ __forceinline__ explicit ItemFinder(const Workspace& ws) {
        const int lane = threadIdx.x & 63, n = (ws.groups + 63) / 64;
        mine = 0u;
        for (int k0 = 0; k0 < n; k0 += 8) {
            unsigned c[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = of_group(ws, (k0 + k) * 64 + lane);
#pragma unroll
            for (int k = 0; k < 8; ++k) mine += c[k];
        }
        const unsigned incl = wave_scan(mine);
        before = incl - mine;
        total = from_lane(incl, 63);
    }

    // item lo for the wavefront's lower half, hi for its upper half (both below
    // total); every lane must call it
    __device__ __forceinline__ unsigned item(const Workspace& ws, int lane, unsigned lo, unsigned hi) const {
        const int l0 = __ffsll(__ballot(before <= lo && lo - before < mine)) - 1;
        const int l1 = __ffsll(__ballot(before <= hi && hi - before < mine)) - 1;
        const int owner = lane & 32 ? l1 : l0, k = lane & 31;
        unsigned rest = lane & 32 ? hi - from_lane(before, l1) : lo - from_lane(before, l0);
        // up to 64 groups, one a lane: that is the group, without a second look at the
        // counts (forwards of 48 x 46 x 47 12.2 -> 11.9 us, FP64 13.1 -> 12.8)
        if (ws.groups <= 64) return ws.items[static_cast<size_t>(owner) * ws.per * kMaxParts + rest];
        // the owner's groups, a run of up to 4 per lane of the half
        const int run = (ws.groups + 64 * 32 - 1) / (64 * 32);
        unsigned c[kMaxGroups / (64 * 32)], sum = 0u;
#pragma unroll
        for (int i = 0; i < kMaxGroups / (64 * 32); ++i) {
            c[i] = i < run ? of_group(ws, (k * run + i) * 64 + owner) : 0u;
            sum += c[i];
        }
        const unsigned excl = half_scan(sum) - sum;
        const unsigned hit = static_cast<unsigned>(__ballot(excl <= rest && rest - excl < sum) >> (lane & 32));
        const int at = __ffs(static_cast<int>(hit)) - 1;
        rest -= __shfl(excl, at, 32);
        int g = at * run;
        if (run > 1) {
#pragma unroll
            for (int i = 0; i < kMaxGroups / (64 * 32) - 1; ++i) {
                const unsigned n = __shfl(c[i], at, 32);
                if (i + 1 < run && rest >= n && g == at * run + i) { rest -= n; ++g; }
            }
        }
        return ws.items[(static_cast<size_t>(g) * 64 + owner) * ws.per * kMaxParts + rest];
    }
};

// ---------------------------------------------------------------------------
// 2. work items: up to kPartCells interface cells of a tile, each cell on a
// group of 4 lanes, or of 16 (k_curv_quads; the neighbour-normal variant stages each
// cell's 5x5x5 neighbourhood, for each neighbour's own 3x3x3).  Forward:
// kappa.  Backward: the cell's contributions gk * d kappa / d phi_q into its
// contribution row (when it fits).
// ---------------------------------------------------------------------------

// this half wavefront's view of a tile: lane j (0..31) holds mask word j and
// the set bits before it; row: the tile's first contribution row
__device__ __forceinline__ void tile_words(const Workspace& ws, int tile, int j, unsigned& mw, unsigned& pw,
                                           unsigned& row) {
    mw = ws.mask[static_cast<size_t>(tile) * kWords + j];
    const unsigned p = ws.prefix[static_cast<size_t>(tile) * kWords + j];
    row = ws.grows[tile / ws.per] + __shfl(p, 0, 32);
    pw = j ? p : 0u;
}

// the cell of rank first + r (in cell order) of the half's tile, below its
// count; r: 0 .. RANKS-1.  The word that holds each rank by one ballot.
template <int RANKS>
__device__ __forceinline__ int tile_cell(unsigned mw, unsigned pw, unsigned first, int r, int lane) {
    unsigned words = 0u;
    const unsigned end = pw + __popc(mw);
#pragma unroll
    for (int k = 0; k < RANKS; ++k) {
        const unsigned long long in = __ballot(pw <= first + k && first + k < end);
        const unsigned half = lane & 32 ? static_cast<unsigned>(in >> 32) : static_cast<unsigned>(in);
        words = r == k ? half : words;
    }
    const int w = __ffs(static_cast<int>(words)) - 1;
    const unsigned word = __shfl(mw, w, 32);
    return w * 32 + nth_bit(word, static_cast<int>(first + r - __shfl(pw, w, 32)));
}

// zero on the whole tile, by one wavefront
__device__ __forceinline__ void zero_tile(float* __restrict__ out, int tile, int lane, int X, int Y, int Z, int ntx,
                                          int nty) {
    const int x0 = (tile % ntx) * TX, y0 = ((tile / ntx) % nty) * TY, z0 = (tile / (ntx * nty)) * TZ;
    const int x = x0 + (lane % 16) * 4, y = y0 + lane / 16;
    if (x0 + TX <= X && y0 + TY <= Y && z0 + TZ <= Z) {
        const int64_t at = (static_cast<int64_t>(z0) * Y + y) * X + x, plane = static_cast<int64_t>(Y) * X;
        const float4u zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(zero, reinterpret_cast<float4u*>(out + at + u * plane));
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) store_four(out, x, y, z0 + u, X, Y, Z, Four{{0.0f, 0.0f, 0.0f, 0.0f}});
    }
}

// Backward, one wavefront per 64 tiles: which of them have an interface cell in
// their 3x3x3 tiles (their cells can receive a contribution: the gather's
// tiles), and a zero gradient for the others.  Beside the work items in one
// launch: those are bound by instruction issue and leave HBM idle.
__device__ __forceinline__ void zero_away(float* __restrict__ gphi, const Workspace& ws, int seg, int part, int parts,
                                          int X, int Y, int Z, int ntx, int nty, int ntiles) {
    const int lane = threadIdx.x, tile = seg * 64 + lane, ntz = ntiles / (ntx * nty);
    bool act = false;
    if (tile < ntiles) {
        const int tx = tile % ntx, ty = (tile / ntx) % nty, tz = tile / (ntx * nty);
        unsigned any = 0u;
#pragma unroll
        for (int q = 0; q < 27; ++q) {
            // (a neighbour outside the lattice is taken for the nearest inside: one of the 27 as well)
            const int ax = min(max(tx + q_dx(q), 0), ntx - 1), ay = min(max(ty + q_dy(q), 0), nty - 1),
                      az = min(max(tz + q_dz(q), 0), ntz - 1);
            any |= ws.flags[(az * nty + ay) * ntx + ax];
        }
        act = any != 0u;
    }
    const unsigned long long bits = __ballot(act);
    if (lane < 2) ws.act[2 * seg + lane] = static_cast<unsigned>(bits >> (32 * lane));
    const int end = min(ntiles - seg * 64, 64);
    for (int t = part; t < end; t += parts)
        if (!((bits >> t) & 1ull)) zero_tile(gphi, seg * 64 + t, lane, X, Y, Z, ntx, nty);
}

// The backward's first workgroups are zero_away's: one per CU at most (one per
// run of 64 tiles, 1152 of them, kept the work items from the SIMDs: 209 against
// 183 us for the spray), and up to 16 to a run where runs are few: with one
// each, a 64 x 62 x 63 lattice's forward and backward took 42.1 us instead of 33.3.
__host__ __device__ inline unsigned zero_parts(const Workspace& ws) {
    return ws.segs >= 256 ? 1u : (ws.segs <= 16 ? 16u : 256u / static_cast<unsigned>(ws.segs));
}
__host__ __device__ inline unsigned zero_blocks(const Workspace& ws) {
    return ws.segs >= 256 ? 256u : static_cast<unsigned>(ws.segs) * zero_parts(ws);
}

// Up to this many work items the cells take 16 lanes each instead of 4: the chip
// then holds few more wavefronts than there are, or none, and the time is that of
// one cell's chain, which 16 lanes shorten (one round of PLIC problems and points
// instead of three or four).  Both give the same bits.  The line lies where the
// two meet: later for Newton, whose chain is the longest and varies, and with
// neighbour normals, later forward than adjoint there (fewer wavefronts fit), and
// earlier where FP64 points halve the wavefronts that fit.  Graph-timed us with 4 and
// with 16 lanes, one drop in a box, at items
//   SZ forward, mixed     837 13.9 13.5, 1078 14.1 14.7   FP32 1359 15.1 14.7, 1650 15.6 16.4
//                 FP64    837 15.5 15.2, 947 14.8 16.2
//      adjoint, mixed     947 23.5 23.1, 1078 24.9 25.0   FP32 1359 24.9 24.5, 1514 24.1 25.5
//   Newton forward, mixed 1514 21.0 19.1, 1650 19.5 20.9  FP32 1972 19.7 17.8, 2659 21.7 22.4
//                 FP64    2324 33.1 30.7, 2659 35.1 34.9
//      adjoint, mixed     1514 30.2 30.0, 1650 29.7 33.1  FP64 1972 46.5 39.3, 2324 42.9 45.3
//   with neighbour normals, SZ forward, mixed 1972 23.2 22.0, 2659 26.6 29.1  FP64 1205 23.8 22.5, 1359 23.9 26.1
//      adjoint, mixed     1078 42.0 39.6, 1359 43.7 44.7  FP64 1514 52.9 52.5, 1650 52.1 56.0
//   Newton adjoint, mixed 1514 48.7 46.6, 1650 47.5 48.6  FP64 2324 67.8 64.0, 2659 72.2 75.3
// (analytic as SZ; nested as SZ or a little later: FP64 forward with neighbour
// normals 1650 32.7 30.1, 1808 31.6 32.4).
template <int SOLVER, class T, class F, bool ADJ, bool NBR> constexpr unsigned wide_items() {
    if (sizeof(T) == 8 && SOLVER == kNewton) return ADJ ? 2048 : 2560;
    if (sizeof(T) == 8) return NBR ? (ADJ ? 1536 : (SOLVER == kNested ? 1700 : 1300)) : 900;
    if (NBR) return ADJ ? (SOLVER == kNewton ? 1536 : 1300) : 2048;
    if (SOLVER == kNewton) return sizeof(F) == 4 && !ADJ ? 2048 : 1536;
    return sizeof(F) == 4 ? 1400 : 1024;
}

// wavefronts per SIMD: what the registers allow without scratch memory
template <class T, bool ADJ, bool NBR>
constexpr int cell_waves() {
    return sizeof(T) == 4 ? (ADJ ? (NBR ? 2 : 3) : 4) : 2;
}

// This wavefront's share of the work items, LANES lanes per cell: each 32-lane
// half takes an item, or a quarter of one (2 of its 8 cells) with 16 lanes.  A
// group finds its cell, the i-th interface cell of the tile in cell order, from the
// tile's bitmask and prefix counts, stages the cell's fill levels and runs
// curv_cell.  The forward writes kappa, the backward (ADJ) the cell's
// contribution row when it fits the workspace.
template <int LANES, int SOLVER, class T, class U, class F, bool ADJ, int NRM, bool NBR, int NB>
__device__ __forceinline__ void cell_items(const ItemFinder& finder, unsigned block, unsigned blocks,
                                           float (&nbh)[kWaveCells][NB],
                                           CellLds<T, F, ADJ, kKeepOwn<T, ADJ, NBR>>& lds,
                                           const float* __restrict__ phi, const float* __restrict__ gkap,
                                           float* __restrict__ out_field, const Workspace& ws, int X, int Y, int Z, int ntx,
                                           int nty) {
    constexpr int H = NBR ? 2 : 1, W = 2 * H + 1, C = (H * W + H) * W + H;
    constexpr unsigned kHalfCells = 32 / LANES, kShares = kPartCells / kHalfCells;   // shares of an item
    const unsigned total = finder.total * kShares;
    auto contributions = [&](unsigned row) { return ADJ ? ws.contrib + row : nullptr; };
    auto adjoints = [&](unsigned row) {
        return ADJ && NBR ? ws.contrib + 27u * ws.rows + static_cast<size_t>(row) * kRowFloatsH : nullptr;
    };
    for (unsigned it = 2u * block; it < total; it += 2u * blocks) {
        const int lane = thread_index_per_iteration(), l32 = lane & 31, cell = lane / LANES, j = lane % LANES;
        const bool second = it + 1u < total;
        const unsigned mine = it + (second && lane >= 32 ? 1u : 0u);
        const unsigned e = finder.item(ws, lane, it / kShares, (it + (second ? 1u : 0u)) / kShares);
        const int tile = static_cast<int>(e >> 7), part = static_cast<int>(e & 127u);
        unsigned mw, pw, row;
        tile_words(ws, tile, l32, mw, pw, row);
        const unsigned n = __shfl(pw + __popc(mw), kWords - 1, 32);
        const unsigned i0 = static_cast<unsigned>(part) * kPartCells + mine % kShares * kHalfCells, ic = i0 + cell % kHalfCells;
        // (n > i0 but for the last item's shares beyond the tile's cells)
        const unsigned i1 = min(i0, n - 1u);
        const int cl = tile_cell<kHalfCells>(mw, pw, i1, static_cast<int>(min(ic, n - 1u) - i1), lane);
        row += ic;
        // uniform per group; a row that does not fit is recomputed by the gather
        const bool on = ic < n && (second || lane < 32) && (!ADJ || row < ws.rows);
        const int gx = (tile % ntx) * TX + cl % TX, gy = ((tile / ntx) % nty) * TY + (cl / TX) % TY,
                  gz = (tile / (ntx * nty)) * TZ + cl / (TX * TY);
        const int64_t gi = (static_cast<int64_t>(gz) * Y + gy) * X + gx;
        float gk = 0.0f, kv = 0.0f;
        bool done = true;
        if (on) {
            if constexpr (ADJ) {
                gk = gkap[gi];
                if (LANES == kLanes && j == 0) lds.at[cell] = make_int4(gx, gy, gz, static_cast<int>(row));
            }
            if constexpr (NBR) {
                // 25 rows of 5 levels, those outside the lattice read as 0
                for (int r = j; r < W * W; r += LANES) {
                    const int ay = gy + r % W - H, az = gz + r / W - H;
                    const bool in = ay >= 0 && ay < Y && az >= 0 && az < Z;
                    const float* p = phi + (static_cast<int64_t>(az) * Y + ay) * X + (gx - H);
                    float v[W];
#pragma unroll
                    for (int t = 0; t < W; ++t) v[t] = in && gx + t - H >= 0 && gx + t - H < X ? p[t] : 0.0f;
#pragma unroll
                    for (int t = 0; t < W; ++t) nbh[cell][r * W + t] = v[t];
                }
            } else {
                // 9 rows of 3 consecutive levels, all in the lattice (an interface
                // cell lies off the outer layer)
                constexpr int kLoads = (9 + LANES - 1) / LANES;
                float v[kLoads][3];
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    const int r = min(j + u * LANES, 8);
                    const float* p = phi + (static_cast<int64_t>(gz + r / 3 - 1) * Y + (gy + r % 3 - 1)) * X + (gx - 1);
                    v[u][0] = p[0]; v[u][1] = p[1]; v[u][2] = p[2];
                }
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    const int r = j + u * LANES;
                    if (r < 9) { nbh[cell][3 * r] = v[u][0]; nbh[cell][3 * r + 1] = v[u][1]; nbh[cell][3 * r + 2] = v[u][2]; }
                }
            }
            __syncwarp();
            done = curv_cell<LANES, false, SOLVER, T, U, F, ADJ, NRM, NBR>(nbh[cell], C, W, W * W, lane, gk, contributions(row), ws.rows,
                                                                           adjoints(row), lds, kv, Place{gx, gy, gz, X, Y, Z});
        }
        if constexpr (!ADJ)
            if (on && done && j == 0) out_field[gi] = kv;
        if constexpr (LANES == kLanes) redo_groups(done, lane, [&](int src) {
            const int from = max(src, 0);
            Place at{0, 0, 0, X, Y, Z};
            unsigned r = 0u;
            float g = 0.0f;
            if constexpr (ADJ) {
                const int4 p = lds.at[from / LANES];
                at.x = p.x; at.y = p.y; at.z = p.z;
                r = static_cast<unsigned>(p.w);
                if (src >= 0) g = gkap[(static_cast<int64_t>(at.z) * Y + at.y) * X + at.x];
            } else {
                at.x = __shfl(gx, from, 64); at.y = __shfl(gy, from, 64); at.z = __shfl(gz, from, 64);
            }
            float k = 0.0f;
            if (src >= 0)
                curv_cell<kWideLanes, true, SOLVER, T, U, F, ADJ, NRM, NBR>(nbh[src / LANES], C, W, W * W, lane, g, contributions(r),
                                                                            ws.rows, adjoints(r), lds, k, at);
            if constexpr (!ADJ)
                if (src >= 0 && lane % kWideLanes == 0) out_field[(static_cast<int64_t>(at.z) * Y + at.y) * X + at.x] = k;
        });
        __syncwarp();                                        // nbh and lds reused by the next pair
    }
}

template <int SOLVER, class T, class U, class F, bool ADJ, int NRM, bool NBR>
__global__ __launch_bounds__(64, (cell_waves<T, ADJ, NBR>())) void k_curv_quads(
    const float* __restrict__ phi, const float* __restrict__ gkap, float* __restrict__ out_field, Workspace ws, int X,
    int Y, int Z, int ntx, int nty, int ntiles) {
    // the cell's 3x3x3 fill levels (5x5x5 with neighbour normals)
    constexpr int NB = NBR ? 125 : 27;
    __shared__ float nbh[kWaveCells][NB];
    __shared__ CellLds<T, F, ADJ, kKeepOwn<T, ADJ, NBR>> lds;
    unsigned block = blockIdx.x, blocks = gridDim.x;
    if constexpr (ADJ) {
        if (block == 0 && threadIdx.x == 0) ws.counter[kOverflow] = 0u;   // the gather, a later launch, counts there
        const unsigned nzero = zero_blocks(ws), parts = zero_parts(ws);
        if (block < nzero) {
            for (unsigned b = block; b < static_cast<unsigned>(ws.segs) * parts; b += nzero)
                zero_away(out_field, ws, static_cast<int>(b / parts), static_cast<int>(b % parts), static_cast<int>(parts), X, Y,
                          Z, ntx, nty, ntiles);
            return;
        }
        block -= nzero;
        blocks -= nzero;
    } else {
        --blocks;                                            // the last one: the groups' first rows
        if (__builtin_expect(block == blocks, 0)) {
            group_rows(ws);
            return;
        }
    }
    init_cells<NRM>(lds, static_cast<int>(threadIdx.x));
    const ItemFinder finder(ws);
    if (finder.total <= wide_items<SOLVER, T, F, ADJ, NBR>())
        cell_items<kWideLanes, SOLVER, T, U, F, ADJ, NRM, NBR>(finder, block, blocks, nbh, lds, phi, gkap, out_field, ws, X, Y,
                                                               Z, ntx, nty);
    else
        cell_items<kLanes, SOLVER, T, U, F, ADJ, NRM, NBR>(finder, block, blocks, nbh, lds, phi, gkap, out_field, ws, X, Y, Z,
                                                           ntx, nty);
}

// ---------------------------------------------------------------------------
// 3. backward gathers: every cell next to the interface adds the
// contributions of its interface neighbours in a fixed order (deterministic,
// no atomics).  The direct gather reads them from the stored rows; a tile with
// a source whose row did not fit goes to the overflow list, where the fallback
// gather copies the stored rows and recomputes the missing ones.
// ---------------------------------------------------------------------------
constexpr int B_RX = TX + 4, B_RY = TY + 4, B_RZ = TZ + 4;
constexpr int C_RX = TX + 2, C_RY = TY + 2, C_RZ = TZ + 2, C_REGION = C_RX * C_RY * C_RZ;
constexpr int kChunk = 128;
constexpr int kCopyBatch = 8;                 // contribution loads in flight per thread
constexpr unsigned short kNoSlot = 0xFFFFu;

// contribution row of an interior interface cell: its group's first row, the
// group's cells before its tile, and its rank in the tile in cell order
__device__ __forceinline__ unsigned contrib_row(const Workspace& ws, int gx, int gy, int gz, int ntx, int nty) {
    const int ctile = ((gz / TZ) * nty + gy / TY) * ntx + gx / TX;
    const int l = ((gz % TZ) * TY + gy % TY) * TX + gx % TX;
    const unsigned* pre = ws.prefix + static_cast<size_t>(ctile) * kWords;
    const unsigned w = ws.mask[static_cast<size_t>(ctile) * kWords + l / 32];
    return ws.grows[ctile / ws.per] + pre[0] + (l >= 32 ? pre[l / 32] : 0u) + __popc(w & ((1u << (l % 32)) - 1u));
}

// Fallback gather over the overflow list: the tiles with a source cell whose
// row did not fit in the workspace.  Candidates (interface cells of the tile
// grown by one) are processed in chunks of kChunk in region order: stored rows
// are copied, missing ones recomputed (halo 2 in LDS); each target then adds
// its 27 neighbours' entries in q order.  With at most kChunk candidates this
// is the direct gather's order, so the result is the same bits.
template <int SOLVER, class T, class U, class F, int NRM>
__global__ __launch_bounds__(kThreads) void k_curv_gather_fallback(const float* __restrict__ phi,
                                                                    const float* __restrict__ gkap,
                                                                    float* __restrict__ gphi, Workspace ws, int X,
                                                                    int Y, int Z, int ntx, int nty) {
    constexpr int RX = B_RX, RY = B_RY, RZ = B_RZ, H = 2;
    __shared__ float s[RX * RY * RZ];
    __shared__ unsigned short cand[C_REGION];
    __shared__ unsigned short slot[C_REGION];
    __shared__ float contrib[kChunk][27];
    __shared__ unsigned crow[kChunk];
    __shared__ int wcount[kThreads / 64];
    __shared__ CellLds<T, F, true> cells[kThreads / 64];
    const int tid = threadIdx.x;
    const unsigned ntl = *static_cast<volatile unsigned*>(ws.counter + kOverflow);
    if (ntl == 0u) return;
    CellLds<T, F, true>& lds = cells[tid >> 6];
    init_cells<NRM>(lds, tid & 63);
    for (int i = tid; i < C_REGION; i += kThreads) slot[i] = kNoSlot;
    for (unsigned it = blockIdx.x; it < ntl; it += gridDim.x) {
        const int tile = static_cast<int>(ws.over[it]);
        const int x0 = (tile % ntx) * TX, y0 = ((tile / ntx) % nty) * TY, z0 = (tile / (ntx * nty)) * TZ;
        load_region<RX, RY, RZ>(s, phi, x0 - H, y0 - H, z0 - H, X, Y, Z);
        __syncthreads();
        const int ncand = ordered_compact(C_REGION, [&](int ci) {
            const int lx = ci % C_RX, ly = (ci / C_RX) % C_RY, lz = ci / (C_RX * C_RY);
            const int gx = x0 - 1 + lx, gy = y0 - 1 + ly, gz = z0 - 1 + lz;
            return gx >= 1 && gy >= 1 && gz >= 1 && gx <= X - 2 && gy <= Y - 2 && gz <= Z - 2 &&
                   is_iface(s[((lz + H - 1) * RY + (ly + H - 1)) * RX + (lx + H - 1)]);
        }, cand, wcount);
        float acc[kCellsPerThread];
#pragma unroll
        for (int k = 0; k < kCellsPerThread; ++k) acc[k] = 0.0f;
        for (int c0 = 0; c0 < ncand; c0 += kChunk) {
            const int nc = min(kChunk, ncand - c0);
            // one thread per candidate: slot and contribution row
            for (int i = tid; i < nc; i += kThreads) {
                const int ci = cand[c0 + i];
                const int lx = ci % C_RX, ly = (ci / C_RX) % C_RY, lz = ci / (C_RX * C_RY);
                slot[ci] = static_cast<unsigned short>(i);
                crow[i] = contrib_row(ws, x0 - 1 + lx, y0 - 1 + ly, z0 - 1 + lz, ntx, nty);
            }
            __syncthreads();
            // stored rows: all threads, independent loads issued in batches
            const int nv = nc * 27;
            for (int b0 = 0; b0 < nv; b0 += kThreads * kCopyBatch) {
                float v[kCopyBatch];
                unsigned at[kCopyBatch];
#pragma unroll
                for (int u = 0; u < kCopyBatch; ++u) {
                    const int idx = b0 + u * kThreads + tid;
                    const int i = min(idx, nv - 1) / 27;
                    const unsigned r = idx < nv ? crow[i] : ws.rows;
                    at[u] = r < ws.rows ? static_cast<unsigned>(idx) : 0xFFFFFFFFu;
                    v[u] = r < ws.rows ? ws.contrib[static_cast<unsigned>(idx - i * 27) * ws.rows + r] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < kCopyBatch; ++u)
                    if (at[u] != 0xFFFFFFFFu) contrib[at[u] / 27][at[u] % 27] = v[u];
            }
            {
                // rows that did not fit: recomputed, one group of lanes per cell
                const int lane = tid & 63;
                for (int i0 = 0; i0 < nc; i0 += kThreads / kLanes) {
                    const int i = i0 + tid / kLanes;
                    bool done = true;
                    int centre = 0;
                    float gk = 0.0f, kv;
                    if (i < nc && crow[i] >= ws.rows) {                  // uniform per group
                        const int ci = cand[c0 + i];
                        const int lx = ci % C_RX, ly = (ci / C_RX) % C_RY, lz = ci / (C_RX * C_RY);
                        const int gx = x0 - 1 + lx, gy = y0 - 1 + ly, gz = z0 - 1 + lz;
                        gk = gkap[(static_cast<int64_t>(gz) * Y + gy) * X + gx];
                        centre = ((lz + 1) * RY + (ly + 1)) * RX + (lx + 1);
                        done = curv_cell<kLanes, false, SOLVER, T, U, F, true, NRM>(s, centre, RX, RX * RY, lane, gk, contrib[i],
                                                                                    1u, nullptr, lds, kv);
                    }
                    redo_groups(done, lane, [&](int src) {
                        const int from = max(src, 0), ai = __shfl(i, from, 64), ac = __shfl(centre, from, 64);
                        const float ag = __shfl(gk, from, 64);
                        if (src >= 0)
                            curv_cell<kWideLanes, true, SOLVER, T, U, F, true, NRM>(s, ac, RX, RX * RY, lane, ag, contrib[ai],
                                                                                    1u, nullptr, lds, kv);
                    });
                    __syncwarp();                                        // lds reused by the next cells
                }
            }
            __syncthreads();
#pragma unroll 1
            for (int k = 0; k < kCellsPerThread; ++k) {
                const int cl = tid + k * kThreads;
                const int cx = cl % TX, cy = (cl / TX) % TY, cz = cl / (TX * TY);
                // the target sits at candidate-region coordinates (cx+1, cy+1, cz+1);
                // the neighbour owning offset q is at target - e_q
                float a = acc[k];
#pragma unroll
                for (int q = 0; q < 27; ++q) {
                    const int ci = ((cz + 1 - q_dz(q)) * C_RY + (cy + 1 - q_dy(q))) * C_RX + (cx + 1 - q_dx(q));
                    const unsigned short sl = slot[ci];
                    if (sl != kNoSlot) a += contrib[sl][q];
                }
                acc[k] = a;
            }
            __syncthreads();
            for (int i = tid; i < nc; i += kThreads) slot[cand[c0 + i]] = kNoSlot;
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < kCellsPerThread; ++k) {
            const int cl = tid + k * kThreads;
            const int cx = cl % TX, cy = (cl / TX) % TY, cz = cl / (TX * TY);
            const int gx = x0 + cx, gy = y0 + cy, gz = z0 + cz;
            if (gx < X && gy < Y && gz < Z) gphi[(static_cast<int64_t>(gz) * Y + gy) * X + gx] = acc[k];
        }
        __syncthreads();                                             // LDS reused by the next tile
    }
}

// sum over the lanes of each half wavefront, by a butterfly of distances 16, 8,
// 4, 2, 1 (16 and 4 through LDS, the others by lane permutations)
__device__ __forceinline__ float half_sum(float x) {
    x += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x401F));
    x += quad_move<kTurn8>(x);
    x += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x101F));
    x += quad_move<kSwap2>(x);
    return x + quad_move<kSwap1>(x);
}

// Neighbour-normal backward, between the work items and the gather: PAIRS
// pairs of a work item's interface cells on a wavefront, one half of it per cell
// n, lane j < 26 taking the neighbour q of the adjoint's lane order.  The source
// c = n - e_q, when an interface cell, stored in slot j of its row the adjoint
// for its neighbour at +e_q, which is n: the adjoint of n's own fill-level
// gradient is the sum of these 26 slots (zero where c is no interface cell),
// formed by a fixed butterfly and written to the 3-vector beside n's row.  A
// source without a stored row makes it NaN.  Bound by the latency of its
// dependent loads (item, tile, sources, slots).
template <int PAIRS>
__device__ __forceinline__ void hgather_items(const ItemFinder& finder, const Workspace& ws, int X, int Y, int Z, int ntx,
                                              int nty) {
    constexpr unsigned kShares = kPartCells / 2 / PAIRS;     // of an item
    const int lane = threadIdx.x & 63, j = lane & 31, half = lane >> 5;
    const int q = j < 13 ? j : min(j + 1, 26);
    for (unsigned it = blockIdx.x * (kThreads / 64) + threadIdx.x / 64; it < finder.total * kShares;
         it += gridDim.x * (kThreads / 64)) {
        const unsigned e = finder.item(ws, lane, it / kShares, it / kShares), pair0 = it % kShares * PAIRS;
        const int tile = static_cast<int>(e >> 7), part = static_cast<int>(e & 127u);
        unsigned mw, pw, first;
        tile_words(ws, tile, j, mw, pw, first);
        const unsigned n = __shfl(pw + __popc(mw), kWords - 1, 32);
        unsigned row[PAIRS], r[PAIRS];
        bool on[PAIRS], src[PAIRS];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const unsigned i0 = static_cast<unsigned>(part * kPartCells + 2 * p) + 2u * pair0, i = i0 + half, at = min(i0, n - 1u);
            const int cl = tile_cell<2>(mw, pw, at, static_cast<int>(min(i, n - 1u) - at), lane);
            row[p] = first + i;
            on[p] = i < n && row[p] < ws.rows;               // (the gather sees a row that does not fit)
            // a cell off the outer layer: its 26 neighbours lie in the lattice
            const int cx = (tile % ntx) * TX + cl % TX - q_dx(q), cy = ((tile / ntx) % nty) * TY + (cl / TX) % TY - q_dy(q),
                      cz = (tile / (ntx * nty)) * TZ + cl / (TX * TY) - q_dz(q);
            const int ctile = ((cz / TZ) * nty + cy / TY) * ntx + cx / TX;
            const int l = ((cz % TZ) * TY + cy % TY) * TX + cx % TX;
            const size_t word = static_cast<size_t>(ctile) * kWords;
            const unsigned any = ws.flags[ctile], mask = ws.mask[word + l / 32], pre0 = ws.prefix[word],
                           pre = ws.prefix[word + l / 32], base = ws.grows[ctile / ws.per];
            src[p] = j < 26 && any != 0u && ((mask >> (l % 32)) & 1u);
            r[p] = base + pre0 + (l >= 32 ? pre : 0u) + __popc(mask & ((1u << (l % 32)) - 1u));
        }
        float h[PAIRS][3];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const bool stored = on[p] && src[p] && r[p] < ws.rows;
            const float* slot = ws.contrib + 27u * ws.rows + static_cast<size_t>(stored ? r[p] : 0u) * kRowFloatsH + 3 * j;
            h[p][0] = stored ? slot[0] : 0.0f;
            h[p][1] = stored ? slot[1] : 0.0f;
            h[p][2] = stored ? slot[2] : 0.0f;
        }
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const bool miss = ((__ballot(src[p] && r[p] >= ws.rows) >> (32 * half)) & 0xffffffffull) != 0ull;
#pragma unroll
            for (int c = 0; c < 3; ++c) h[p][c] = half_sum(h[p][c]);
            if (on[p] && j < 3) {
                const float v = j == 0 ? h[p][0] : (j == 1 ? h[p][1] : h[p][2]);
                ws.hbar[3u * row[p] + static_cast<unsigned>(j)] = miss ? __builtin_nanf("") : v;
            }
        }
    }
}

// With many items a wavefront takes all 8 cells of one through its loads
// together, with up to 1024 a pair of them: forward and backward of 5 drops in
// 150 x 131 x 118 (3400 items) 89.9 us with pairs and 86.8 with items, the spray
// 905 and 856; 28 x 26 x 27 34.6 and 35.7.  Between, the backward alone, pairs and
// items (mixed): 678 items 30.7 and 31.1, 837 32.6 and 32.5, 1078 38.9 and 39.3, 1514 44.3
// and 44.3, 1808 47.2 and 46.2, 2659 51.9 and 49.8.
__global__ __launch_bounds__(kThreads) void k_curv_hgather(Workspace ws, int X, int Y, int Z, int ntx, int nty) {
    const ItemFinder finder(ws);
    if (finder.total <= 1024u) hgather_items<1>(finder, ws, X, Y, Z, ntx, nty);
    else hgather_items<kPartCells / 2>(finder, ws, X, Y, Z, ntx, nty);
}

// Direct backward gather over the tiles with an interface cell in their 3x3x3
// tiles (zero_away wrote the others), one workgroup per tile, one wavefront per
// layer of it.  The mask rows of the 6 x 6 rows of cells around the tile are
// staged, each with one bit of the columns left and right of the tile and the
// contribution rows before it; a row's band (cells with an interface source
// within one cell) is the OR of its 9 neighbouring rows, each dilated by one
// cell in x.  A lane takes a band cell and adds entry q of its sources' rows
// for q = 0..26 in order, all loads issued before the first add; the tile is
// put together in LDS and written as whole lines.
// A tile with a source beyond the store goes to the overflow list, and the
// fallback gather, a later launch, rewrites all of its cells; with neighbour
// normals (NBR, which adds each source's own-gradient adjoint spread by the
// gradient weights of NRM, and has no fallback) its band becomes NaN.
// Bound by the latency of a tile's dependent loads (activity, masks, rows) and
// by instruction issue (27 sources per band cell), so compiled for 7 wavefronts
// per SIMD.  A flat interface fills a tile's layers: one wavefront per tile
// would be a chain of 12 rounds for its 768 band cells.
struct GatherLds {
    uint4 win[36][2];                             // per mask row (y, then z, from -1 to 4): see row_sources
    unsigned edge[36][2];                         // contribution rows of the sources left and right of the tile
    unsigned long long dilated[36];
    unsigned long long band[TY * TZ];
    int before[TY * TZ];                          // band cells before the row
    alignas(16) float out[kTile];
};

// x of the k-th set bit of d (k below their number)
__device__ __forceinline__ int set_bit(unsigned long long d, int k) {
    unsigned word = static_cast<unsigned>(d);
    const int low32 = __popc(word);
    int x = 0;
    if (k >= low32) { k -= low32; x = 32; word = static_cast<unsigned>(d >> 32); }
#pragma unroll
    for (int st = 16; st; st >>= 1) {
        const int low = __popc(word & ((1u << st) - 1u));
        const bool up = k >= low;
        k -= up ? low : 0;
        x += up ? st : 0;
        word >>= up ? st : 0;
    }
    return x;
}

// The sources at x + 1, x, x - 1 of mask row rr (offsets q, q + 1, q + 2 of the
// 27): bits 2, 1, 0 of the result where they are interface cells, and their
// contribution rows (at most last, where they are none).  Bit p of the extended
// row is cell p - 1, from the cell left of the tile to the one right of it; win
// holds for either half of it the contribution row of its first set bit, the
// half and the word after it.
__device__ __forceinline__ unsigned row_sources(const GatherLds& m, int rr, int x, unsigned last, unsigned (&r)[3]) {
    const uint4 w = m.win[rr][x >> 5];
    const unsigned sh = static_cast<unsigned>(x) & 31u;
    const unsigned three = __builtin_amdgcn_alignbit(w.z, w.y, sh) & 7u;
    r[2] = w.x + __popc(w.y & ((1u << sh) - 1u));
    r[1] = r[2] + (three & 1u);
    r[0] = r[1] + ((three >> 1) & 1u);
    if (x == 0) r[2] = m.edge[rr][0];
    if (x == TX - 1) r[0] = m.edge[rr][1];
#pragma unroll
    for (int k = 0; k < 3; ++k) r[k] = min(r[k], last);
    return three;
}

// The gather's tiles in one sequence over up to 4096 runs of 64 tiles, as
// ItemFinder: lane l owns runs l, l + 64, ...
struct TileFinder {
    unsigned mine, before, total;
    int seg0;

    __device__ __forceinline__ static unsigned long long of(const Workspace& ws, int seg) {
        return seg < ws.segs ? ws.act[2 * seg] | (static_cast<unsigned long long>(ws.act[2 * seg + 1]) << 32) : 0ull;
    }

    __device__ __forceinline__ TileFinder(const Workspace& ws, int first) : seg0(first) {
        const int lane = threadIdx.x & 63, n = (min(ws.segs - seg0, 4096) + 63) / 64;
        mine = 0u;
        for (int k0 = 0; k0 < n; k0 += 4) {
            unsigned long long c[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = k0 + k < n ? of(ws, seg0 + (k0 + k) * 64 + lane) : 0ull;
#pragma unroll
            for (int k = 0; k < 4; ++k) mine += static_cast<unsigned>(__popcll(c[k]));
        }
        const unsigned incl = wave_scan(mine);
        before = incl - mine;
        total = from_lane(incl, 63);
    }

    // the i-th tile, i below total, the same for the whole wavefront
    __device__ __forceinline__ int tile(const Workspace& ws, int lane, unsigned i) const {
        const int owner = __ffsll(__ballot(before <= i && i - before < mine)) - 1;
        const unsigned rest = i - from_lane(before, owner);
        const unsigned long long bits = of(ws, seg0 + lane * 64 + owner);
        const unsigned n = static_cast<unsigned>(__popcll(bits)), excl = wave_scan(n) - n;
        const int at = __ffsll(__ballot(excl <= rest && rest - excl < n)) - 1;
        const unsigned long long found = from_lane(static_cast<unsigned>(bits), at) |
                                         (static_cast<unsigned long long>(from_lane(static_cast<unsigned>(bits >> 32), at)) << 32);
        return (seg0 + at * 64 + owner) * 64 + set_bit(found, static_cast<int>(rest - from_lane(excl, at)));
    }
};

template <bool NBR, int NRM>
__global__ __launch_bounds__(kThreads, NBR ? 5 : 7) void k_curv_gather_direct(float* __restrict__ gphi, Workspace ws, int X,
                                                                       int Y, int Z, int ntx, int nty, int ntz) {
    static_assert(kThreads * 4 == kTile, "four cells of the output per thread");
    __shared__ GatherLds m;
    for (int seg0 = 0; seg0 < ws.segs; seg0 += 4096) {
        const TileFinder finder(ws, seg0);
#pragma unroll 1
        for (unsigned i = blockIdx.x; i < finder.total; i += gridDim.x) {
            const int tid = thread_index_per_iteration(), lane = tid & 63, cz = tid >> 6;
            const int tile = finder.tile(ws, lane, i);
            if (ws.rows == 0u) {                                     // nothing stored: all recomputed
                if (tid == 0) ws.over[atomicAdd(ws.counter + kOverflow, 1u)] = static_cast<unsigned>(tile);
                continue;
            }
            const int tx = tile % ntx, ty = (tile / ntx) % nty, tz = tile / (ntx * nty);
            const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
            const int ox = x0 + (lane % 16) * 4, oy = y0 + lane / 16, oz = z0 + cz;   // this lane's cells of the output
            bool miss = false;
            if (tid < 36) {
                const int yy = tid % 6 - 1, zz = tid / 6 - 1;
                const int ry = yy < 0 ? -1 : (yy >= TY ? 1 : 0), rz = zz < 0 ? -1 : (zz >= TZ ? 1 : 0);
                const int ay = ty + ry, az = tz + rz;
                const int w = ((zz - rz * TZ) * TY + (yy - ry * TY)) * 2;    // the row's first mask word
                const bool yz_in = ay >= 0 && ay < nty && az >= 0 && az < ntz;
                unsigned lo[3], hi[3], row[3], pre[3], has[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) {                        // columns left, own, right: loads
                    const int ax = tx + t - 1;
                    const bool in = yz_in && ax >= 0 && ax < ntx;
                    const int nt = in ? (az * nty + ay) * ntx + ax : tile;
                    const size_t b = static_cast<size_t>(nt) * kWords;
                    has[t] = in ? ws.flags[nt] : 0u;
                    lo[t] = ws.mask[b + w];
                    hi[t] = ws.mask[b + w + 1];
                    row[t] = ws.grows[nt / ws.per] + ws.prefix[b];
                    pre[t] = ws.prefix[b + w];
                }
#pragma unroll
                for (int t = 0; t < 3; ++t) {                        // masks are there only where has is not 0
                    lo[t] = has[t] ? lo[t] : 0u;
                    hi[t] = has[t] ? hi[t] : 0u;
                    row[t] += w ? pre[t] : 0u;
                }
                const unsigned left = hi[0] >> 31, right = lo[2] & 1u;
                const unsigned e0 = (lo[1] << 1) | left, e1 = (lo[1] >> 31) | (hi[1] << 1), e2 = (hi[1] >> 31) | (right << 1);
                const unsigned first = row[1] - left, before_left = row[0] + __popc(lo[0]) + __popc(hi[0] & 0x7FFFFFFFu);
                m.win[tid][0] = make_uint4(first, e0, e1, 0u);
                m.win[tid][1] = make_uint4(first + __popc(e0), e1, e2, 0u);
                m.edge[tid][0] = before_left;
                m.edge[tid][1] = row[2];
                const unsigned long long mid = lo[1] | (static_cast<unsigned long long>(hi[1]) << 32);
                m.dilated[tid] = mid | (mid << 1) | (mid >> 1) | left | (static_cast<unsigned long long>(right) << 63);
                // a staged source beyond the store
                miss = (mid && row[1] + static_cast<unsigned>(__popcll(mid)) > ws.rows) ||
                       (left && before_left >= ws.rows) || (right && row[2] >= ws.rows);
            }
            const bool missing = __syncthreads_or(miss);             // uniform
            if (!NBR && missing) {
                if (tid == 0) ws.over[atomicAdd(ws.counter + kOverflow, 1u)] = static_cast<unsigned>(tile);
                __syncthreads();                                     // LDS reused by the next tile
                continue;
            }
            // every wavefront forms the band of the 16 rows (the same values)
            int inc = 0;
            if (lane < TY * TZ) {
                const int by = lane % TY, bz = lane / TY;
                unsigned long long d = 0ull;
#pragma unroll
                for (int dz = 0; dz < 3; ++dz) {
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) d |= m.dilated[(bz + dz) * 6 + by + dy];
                }
                // cells past the lattice edge are not targets
                if (y0 + by >= Y || z0 + bz >= Z) d = 0ull;
                else if (X - x0 < TX) d &= (1ull << (X - x0)) - 1ull;
                const int c = __popcll(d);
                inc = static_cast<int>(half_scan(static_cast<unsigned>(c)));
                m.band[lane] = d;
                m.before[lane] = inc - c;
            }
            const int nband = static_cast<int>(from_lane(static_cast<unsigned>(inc), TY * TZ - 1));
            *reinterpret_cast<float4*>(m.out + tid * 4) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            __syncthreads();
            const unsigned last = ws.rows - 1u;
#pragma unroll 1
            for (int e = tid; e < nband; e += kThreads) {
                int row = 0;                                         // the last row with before <= e
#pragma unroll
                for (int st = TY * TZ / 2; st; st >>= 1) row += m.before[row + st] <= e ? st : 0;
                const int x = set_bit(m.band[row], e - m.before[row]), at = row / TY * 6 + row % TY;   // mask row of (y - 1, z - 1)
                float a = 0.0f;                                      // +0 + 0 stays +0: same bits as skipping
                if constexpr (NBR) {
#pragma unroll 1
                    for (int dz = -1; dz <= 1; ++dz) {
                        float v[9], hv[9][3];
                        unsigned has = 0u;                           // bit 3 row + 2 - dx
#pragma unroll
                        for (int i3 = 0; i3 < 9; i3 += 3) {
                            unsigned r[3];
                            has |= row_sources(m, at + (1 - dz) * 6 + 2 - i3 / 3, x, last, r) << i3;
#pragma unroll
                            for (int dx = 0; dx < 3; ++dx) {
                                v[i3 + dx] = (ws.contrib + static_cast<size_t>((dz + 1) * 9 + i3 + dx) * ws.rows)[r[dx]];
                                hv[i3 + dx][0] = ws.hbar[3u * r[dx]];
                                hv[i3 + dx][1] = ws.hbar[3u * r[dx] + 1u];
                                hv[i3 + dx][2] = ws.hbar[3u * r[dx] + 2u];
                            }
                        }
#pragma unroll
                        for (int k = 0; k < 9; ++k) {
                            // the source's own gradient h = sum_q w_q e_q phi_(source + e_q)
                            const int dx = k % 3 - 1, dy = k / 3 - 1, e2 = dx * dx + dy * dy + dz * dz;
                            const float wq = static_cast<float>(e2 == 0 ? 0 : nrm_weight<NRM>(e2));
                            const float t = v[k] + wq * (static_cast<float>(dx) * hv[k][0] + static_cast<float>(dy) * hv[k][1] +
                                                         static_cast<float>(dz) * hv[k][2]);
                            a += (has >> (k / 3 * 3 + 2 - k % 3)) & 1u ? t : 0.0f;
                        }
                    }
                } else {
                    float v[27];
                    unsigned has = 0u;                               // bit 3 row + 2 - dx
#pragma unroll
                    for (int i3 = 0; i3 < 27; i3 += 3) {
                        unsigned r[3];
                        has |= row_sources(m, at + (2 - i3 / 9) * 6 + 2 - (i3 / 3) % 3, x, last, r) << i3;
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx)
                            v[i3 + dx] = (ws.contrib + static_cast<size_t>(i3 + dx) * ws.rows)[r[dx]];
                    }
#pragma unroll
                    for (int q = 0; q < 27; ++q) {
                        const int on = __builtin_amdgcn_sbfe(static_cast<int>(has), q / 3 * 3 + 2 - q % 3, 1);   // 0 or all ones
                        a += __uint_as_float(__float_as_uint(v[q]) & static_cast<unsigned>(on));
                    }
                }
                m.out[row * TX + x] = a;
            }
            __syncthreads();
            if (NBR && missing) {
#pragma unroll 1
                for (int r = cz * TY; r < (cz + 1) * TY; ++r)
                    if ((m.band[r] >> lane) & 1ull) m.out[r * TX + lane] = __builtin_nanf("");
                __syncwarp();
            }
            Four o;
            const float4 t4 = *reinterpret_cast<const float4*>(m.out + tid * 4);
            o.v[0] = t4.x; o.v[1] = t4.y; o.v[2] = t4.z; o.v[3] = t4.w;
            store_four(gphi, ox, oy, oz, X, Y, Z, o);
            __syncthreads();                                         // LDS reused by the next tile
        }
    }
}

// ---- launch helpers -----------------------------------------------------------
struct Grid {
    int ntx, nty, ntz;
    int ntiles;
};

// validates the lattice; *empty when there is nothing to do
int check_lattice(int64_t X, int64_t Y, int64_t Z, bool* empty, Grid* g) {
    if (X < 0 || Y < 0 || Z < 0) return PLIC_EINVAL;
    *empty = X == 0 || Y == 0 || Z == 0;
    if (*empty) return PLIC_OK;
    const int64_t lim = 0x7fffffff;
    if (X > lim || Y > lim || Z > lim) return PLIC_EINVAL;
    if (X > (int64_t(1) << 62) / Y / Z) return PLIC_EINVAL;
    const int64_t tx = (X + TX - 1) / TX, ty = (Y + TY - 1) / TY, tz = (Z + TZ - 1) / TZ;
    if (tx > lim / ty || tx * ty > lim / tz) return PLIC_EINVAL;   // grid limit
    // a work item holds tile << 7 in 32 bits, and the work items of all tiles, up to
    // 128 each, are counted in 32 bits
    if (tx * ty * tz >= kMaxTiles) return PLIC_EINVAL;
    g->ntx = static_cast<int>(tx);
    g->nty = static_cast<int>(ty);
    g->ntz = static_cast<int>(tz);
    g->ntiles = static_cast<int>(tx * ty * tz);
    return PLIC_OK;
}

size_t fixed_bytes(const Grid& g) { return 256 + static_cast<size_t>(g.ntiles) * kFixedPerTile; }

// nbr: the neighbour-normal backward's rows (and their gradient adjoints)
Workspace carve(void* base, size_t bytes, const Grid& g, bool nbr = false) {
    char* p = static_cast<char*>(base);
    const size_t nt = static_cast<size_t>(g.ntiles);
    Workspace w;
    w.counter = reinterpret_cast<unsigned*>(p);
    w.flags = reinterpret_cast<unsigned*>(p + 256);
    w.grows = w.flags + nt;
    w.mask = w.grows + nt;
    w.prefix = w.mask + nt * kWords;
    w.items = w.prefix + nt * kWords;
    w.gitems = w.items + nt * kMaxParts;
    w.over = w.gitems + nt;
    w.contrib = reinterpret_cast<float*>(w.over + nt);
    const size_t rows = (bytes - fixed_bytes(g)) / (nbr ? kRowBytesNbr : kRowBytes);
    const unsigned limit = nbr ? kRowLimitNbr : kRowLimit;
    w.rows = static_cast<unsigned>(rows < limit ? rows : limit);
    w.hbar = nbr ? w.contrib + static_cast<size_t>(w.rows) * kRowFloatsNbr : nullptr;
    const int waves = scan_waves(g.ntiles), rounds = (g.ntiles + waves * kMaxGroups - 1) / (waves * kMaxGroups);
    w.per = waves * rounds;
    w.groups = (g.ntiles + w.per - 1) / w.per;
    w.segs = (g.ntiles + 63) / 64;
    w.act = w.groups + 2 * w.segs <= g.ntiles ? w.gitems + w.groups : w.counter + 16;   // (2 segments: 3 tiles and more)
    return w;
}

template <bool FWD>
void launch_scan(const float* phi, float* out, Workspace ws, int X, int Y, int Z, const Grid& g,
                 hipStream_t st) {
    if (scan_waves(g.ntiles) == kScanWaves)
        hipLaunchKernelGGL((k_curv_scan<FWD, kScanWaves>), dim3(ws.groups), dim3(64 * kScanWaves), 0, st, phi, out, ws,
                           X, Y, Z, g.ntx, g.nty, g.ntiles);
    else
        hipLaunchKernelGGL((k_curv_scan<FWD, kFewScanWaves>), dim3(ws.groups), dim3(64 * kFewScanWaves), 0, st, phi,
                           out, ws, X, Y, Z, g.ntx, g.nty, g.ntiles);
    // (a forward's work items finish the rows in a workgroup of their launch)
    if (!FWD) hipLaunchKernelGGL(k_curv_rows, dim3(1), dim3(64), 0, st, ws);
}

unsigned persistent_grid(int64_t items_max) {
    return static_cast<unsigned>(items_max < kPersistentBlocks ? items_max : kPersistentBlocks);
}

template <int SOLVER, class T, class U, class F, bool ADJ, int NRM, bool NBR = false>
void launch_cells(const float* phi, const float* gk, float* out, Workspace ws, int X, int Y, int Z, const Grid& g,
                  hipStream_t st) {
    // a forward's last workgroup forms the groups' first rows, a backward's first ones zero the tiles away
    const int64_t most = static_cast<int64_t>(g.ntiles) * kTile * kLanes / 64;
    const dim3 grid(static_cast<unsigned>(most < kCellBlocks ? most : kCellBlocks) + (ADJ ? zero_blocks(ws) : 1u)), block(64);
    hipLaunchKernelGGL((k_curv_quads<SOLVER, T, U, F, ADJ, NRM, NBR>), grid, block, 0, st, phi, gk, out, ws, X, Y, Z,
                       g.ntx, g.nty, g.ntiles);
}

// forward: precision picks the types, then the normal and the variant
template <int SOLVER, class T, class U, class F>
void launch_fwd_t(int normal, bool nbr, const float* phi, float* kappa, Workspace ws, int X, int Y, int Z,
                  const Grid& g, hipStream_t st) {
    if (normal == kNormalCM) {
        if (nbr) launch_cells<SOLVER, T, U, F, false, kNormalCM, true>(phi, nullptr, kappa, ws, X, Y, Z, g, st);
        else launch_cells<SOLVER, T, U, F, false, kNormalCM>(phi, nullptr, kappa, ws, X, Y, Z, g, st);
    } else {
        if (nbr) launch_cells<SOLVER, T, U, F, false, kNormalPY, true>(phi, nullptr, kappa, ws, X, Y, Z, g, st);
        else launch_cells<SOLVER, T, U, F, false, kNormalPY>(phi, nullptr, kappa, ws, X, Y, Z, g, st);
    }
}

template <int SOLVER>
void launch_fwd(int precision, int normal, bool nbr, const float* phi, float* kappa, Workspace ws, int X, int Y,
                int Z, const Grid& g, hipStream_t st) {
    if (precision == PLIC_FP32) launch_fwd_t<SOLVER, float, float, float>(normal, nbr, phi, kappa, ws, X, Y, Z, g, st);
    else if (precision == PLIC_MIXED) launch_fwd_t<SOLVER, float, double, double>(normal, nbr, phi, kappa, ws, X, Y, Z, g, st);
    else launch_fwd_t<SOLVER, double, double, double>(normal, nbr, phi, kappa, ws, X, Y, Z, g, st);
}

// backward: adjoint work items (rows that fit), direct gather of the stored
// rows (independent of solver and precision), then the fallback gather that
// recomputes the rows that did not fit
template <bool NBR, int NRM>
void launch_gather(float* gp, Workspace ws, int X, int Y, int Z, const Grid& g, hipStream_t st) {
    hipLaunchKernelGGL((k_curv_gather_direct<NBR, NRM>), dim3(g.ntiles < kGatherBlocks ? g.ntiles : kGatherBlocks),
                       dim3(kThreads), 0, st, gp, ws, X, Y, Z, g.ntx, g.nty, g.ntz);
}

template <int SOLVER, class T, class U, class F, int NRM>
void launch_bwd_t(const float* phi, const float* gk, float* gp, Workspace ws, int X, int Y, int Z,
                  const Grid& g, hipStream_t st) {
    launch_cells<SOLVER, T, U, F, true, NRM>(phi, gk, gp, ws, X, Y, Z, g, st);
    launch_gather<false, 0>(gp, ws, X, Y, Z, g, st);
    // empty where every row fits: the recommended workspace holds 16 a tile, which a
    // drop in a box of 40^3 and more does not exceed, one in 28^3 or several in 64^3 do
    // (their backwards take 53 and 96 us so, 17 and 21 with room for all).  Its registers
    // (over 256 with the accumulators) allow one workgroup per CU, so a grid of one
    // per CU (256) runs in a single round, cheap when nothing overflowed and as
    // concurrent as any larger grid when something did
    hipLaunchKernelGGL((k_curv_gather_fallback<SOLVER, T, U, F, NRM>),
                       dim3(g.ntiles < kFallbackBlocks ? g.ntiles : kFallbackBlocks), dim3(kThreads), 0, st, phi,
                       gk, gp, ws, X, Y, Z, g.ntx, g.nty);
}

// neighbour-normal backward: the rows (contributions and the neighbours'
// gradient adjoints), the gradient adjoint per interface cell, then the
// gather; there is no fallback (the entry point requires one row at least)
template <int SOLVER, class T, class U, class F, int NRM>
void launch_bwd_nbr_t(const float* phi, const float* gk, float* gp, Workspace ws, int X, int Y, int Z,
                      const Grid& g, hipStream_t st) {
    launch_cells<SOLVER, T, U, F, true, NRM, true>(phi, gk, gp, ws, X, Y, Z, g, st);
    hipLaunchKernelGGL(k_curv_hgather, dim3(persistent_grid(static_cast<int64_t>(g.ntiles) * kMaxParts)),
                       dim3(kThreads), 0, st, ws, X, Y, Z, g.ntx, g.nty);
    launch_gather<true, NRM>(gp, ws, X, Y, Z, g, st);
}

template <int SOLVER, class T, class U, class F>
void launch_bwd_n(int normal, bool nbr, const float* phi, const float* gk, float* gp, Workspace ws, int X, int Y,
                  int Z, const Grid& g, hipStream_t st) {
    if (nbr) {
        if (normal == kNormalCM) launch_bwd_nbr_t<SOLVER, T, U, F, kNormalCM>(phi, gk, gp, ws, X, Y, Z, g, st);
        else launch_bwd_nbr_t<SOLVER, T, U, F, kNormalPY>(phi, gk, gp, ws, X, Y, Z, g, st);
    } else {
        if (normal == kNormalCM) launch_bwd_t<SOLVER, T, U, F, kNormalCM>(phi, gk, gp, ws, X, Y, Z, g, st);
        else launch_bwd_t<SOLVER, T, U, F, kNormalPY>(phi, gk, gp, ws, X, Y, Z, g, st);
    }
}

template <int SOLVER>
void launch_bwd(int precision, int normal, bool nbr, const float* phi, const float* gk, float* gp, Workspace ws,
                int X, int Y, int Z, const Grid& g, hipStream_t st) {
    if (precision == PLIC_FP32)
        launch_bwd_n<SOLVER, float, float, float>(normal, nbr, phi, gk, gp, ws, X, Y, Z, g, st);
    else if (precision == PLIC_MIXED)
        launch_bwd_n<SOLVER, float, double, double>(normal, nbr, phi, gk, gp, ws, X, Y, Z, g, st);
    else
        launch_bwd_n<SOLVER, double, double, double>(normal, nbr, phi, gk, gp, ws, X, Y, Z, g, st);
}

}  // namespace

// The kernels of a forward (gk null) or a backward after its scan, for one
// solver.  Each solver compiles as an object of its own (PLIC_PART 1 to 4, the
// entry points 0; all in one where it is not set): side by side they take 49 s,
// together 180.
struct CellLaunch {
    const float *phi, *gk;
    float* out;
    void* workspace;
    size_t bytes;
    int X, Y, Z, precision, normal;
    bool nbr;
    hipStream_t st;
};
template <int SOLVER> __attribute__((visibility("hidden"))) void launch_solver(const CellLaunch& p);

#if !defined(PLIC_PART) || PLIC_PART > 0
template <int SOLVER> void launch_solver(const CellLaunch& p) {
    bool empty;
    Grid g{};
    check_lattice(p.X, p.Y, p.Z, &empty, &g);
    const Workspace ws = carve(p.workspace, p.bytes, g, p.gk && p.nbr);
    if (p.gk) launch_bwd<SOLVER>(p.precision, p.normal, p.nbr, p.phi, p.gk, p.out, ws, p.X, p.Y, p.Z, g, p.st);
    else launch_fwd<SOLVER>(p.precision, p.normal, p.nbr, p.phi, p.out, ws, p.X, p.Y, p.Z, g, p.st);
}
#endif
#if defined(PLIC_PART) && PLIC_PART > 0
template void launch_solver<PLIC_PART - 1>(const CellLaunch&);
}  // namespace plic
#else

namespace {

void launch_cells_of(int solver, const CellLaunch& p) {
    switch (solver) {
        case kSZ: launch_solver<kSZ>(p); break;
        case kNewton: launch_solver<kNewton>(p); break;
        case kNested: launch_solver<kNested>(p); break;
        default: launch_solver<kAnalytic>(p); break;
    }
}

// shared argument checks of the two entry points (the workspace's size is
// checked last, by each entry point: PLIC_EWORKSPACE only when every other
// argument is valid)
int check_common(const float* phi, int64_t X, int64_t Y, int64_t Z, int solver, int precision,
                 const void* ws, size_t ws_bytes, bool* empty, Grid* g, int64_t* n) {
    if (!valid_curvature_solver(solver) || !valid_precision(precision)) return PLIC_EINVAL;
    if (check_lattice(X, Y, Z, empty, g) != PLIC_OK) return PLIC_EINVAL;
    *n = *empty ? 0 : X * Y * Z;
    if (!valid_array(phi, *n)) return PLIC_EINVAL;
    if (!*empty) {
        if (ws == nullptr || !aligned(ws, 4)) return PLIC_EINVAL;
        if (overlap(ws, ws_bytes, phi, static_cast<size_t>(*n) * sizeof(float))) return PLIC_EINVAL;
    }
    return PLIC_OK;
}

// ---- which phi a workspace's scan records belong to -----------------------------
// The scan's records (interface masks, prefix counts, work items, tile counts)
// depend on phi and the lattice only.  The host notes, per workspace address,
// the phi and lattice of the last call that scanned into it, so that
// plic_curvature_backward_reuse_f32 skips the scan only when they match.  The
// table is bounded (cleared when full: a miss only costs a scan).
struct ScanRecord {
    const float* phi;
    int64_t X, Y, Z;
};
constexpr size_t kMaxRecords = 4096;
std::mutex g_record_mutex;
std::unordered_map<const void*, ScanRecord> g_records;

void note_scan(const void* ws, const float* phi, int64_t X, int64_t Y, int64_t Z, bool ok) {
    std::lock_guard<std::mutex> lock(g_record_mutex);
    if (!ok) {
        g_records.erase(ws);
        return;
    }
    if (g_records.size() >= kMaxRecords && g_records.find(ws) == g_records.end()) g_records.clear();
    try {
        g_records[ws] = ScanRecord{phi, X, Y, Z};
    } catch (const std::bad_alloc&) {        // no exception leaves a C entry
        g_records.clear();
    }
}

bool has_scan(const void* ws, const float* phi, int64_t X, int64_t Y, int64_t Z) {
    std::lock_guard<std::mutex> lock(g_record_mutex);
    const auto it = g_records.find(ws);
    return it != g_records.end() && it->second.phi == phi && it->second.X == X && it->second.Y == Y &&
           it->second.Z == Z;
}

// the forward launches, after validation
int curvature_forward(const float* phi, int64_t X, int64_t Y, int64_t Z, float* kappa, int solver, int precision,
                      int normal, bool nbr, void* workspace, size_t workspace_bytes, const Grid& g, hipStream_t st) {
    const Workspace ws = carve(workspace, workspace_bytes, g);
    const int x = static_cast<int>(X), y = static_cast<int>(Y), z = static_cast<int>(Z);
    launch_scan<true>(phi, kappa, ws, x, y, z, g, st);
    launch_cells_of(solver, {phi, nullptr, kappa, workspace, workspace_bytes, x, y, z, precision, normal, nbr, st});
    const int rc = launch_status();
    note_scan(workspace, phi, X, Y, Z, rc == PLIC_OK);
    return rc;
}

// the backward, after the shared checks; reuse: skip the scan when the
// workspace holds this phi's records
int curvature_backward(const float* phi, int64_t X, int64_t Y, int64_t Z, const float* grad_kappa, float* grad_phi,
                       int solver, int precision, int normal, int neighbour_normals, void* workspace,
                       size_t workspace_bytes, void* stream, bool reuse) {
    bool empty;
    Grid g{};
    int64_t n = 0;
    if (check_common(phi, X, Y, Z, solver, precision, workspace, workspace_bytes, &empty, &g, &n) != PLIC_OK)
        return PLIC_EINVAL;
    if (!valid_normal(normal) || (neighbour_normals != 0 && neighbour_normals != 1)) return PLIC_EINVAL;
    if (!valid_array(grad_kappa, n) || !valid_array(grad_phi, n)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(n) * sizeof(float);
    if (overlap(grad_phi, nb, phi, nb) || overlap(grad_phi, nb, grad_kappa, nb)) return PLIC_EINVAL;
    if (!empty && (overlap(workspace, workspace_bytes, grad_phi, nb) ||
                   overlap(workspace, workspace_bytes, grad_kappa, nb)))
        return PLIC_EINVAL;
    if (empty) return PLIC_OK;
    // the neighbour-normal backward has no fallback: it needs one row at least
    if (workspace_bytes < fixed_bytes(g) + (neighbour_normals ? kRowBytesNbr : 0)) return PLIC_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool nbr = neighbour_normals != 0;
    const Workspace ws = carve(workspace, workspace_bytes, g, nbr);
    const int x = static_cast<int>(X), y = static_cast<int>(Y), z = static_cast<int>(Z);
    const bool scan = !(reuse && has_scan(workspace, phi, X, Y, Z));
    if (scan) launch_scan<false>(phi, grad_phi, ws, x, y, z, g, st);
    launch_cells_of(solver, {phi, grad_kappa, grad_phi, workspace, workspace_bytes, x, y, z, precision, normal, nbr, st});
    const int rc = launch_status();
    if (scan || rc != PLIC_OK) note_scan(workspace, phi, X, Y, Z, rc == PLIC_OK);
    return rc;
}

// ---- the forward without a caller workspace ------------------------------------
// A file-scope device array serves as the workspace of plic_curvature_noalloc_f32
// (every GPU the library runs on holds its own copy, for the life of the
// process).  Host code reaches it only through the address that
// hipGetSymbolAddress returns on each device; the array's name in host code
// is not a device address.
constexpr size_t kScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// the current device's scratch address, looked up once per device
int scratch_for_current_device(void** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_last_hip_error(static_cast<int>(e));
        return PLIC_EHIP;
    }
    if (dev < 0 || dev >= kMaxDevices) return PLIC_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            set_last_hip_error(static_cast<int>(e != hipSuccess ? e : hipErrorInvalidSymbol));
            return PLIC_EHIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return PLIC_OK;
}

}  // namespace
}  // namespace plic

using namespace plic;

extern "C" {

size_t plic_curvature_workspace_bytes(int64_t X, int64_t Y, int64_t Z) {
    bool empty;
    Grid g;
    if (check_lattice(X, Y, Z, &empty, &g) != PLIC_OK || empty) return 0;
    return fixed_bytes(g) + static_cast<size_t>(g.ntiles) * kDefaultRowsPerTile * kRowBytes;
}

size_t plic_curvature_workspace_bytes_ex(int64_t X, int64_t Y, int64_t Z, int neighbour_normals) {
    bool empty;
    Grid g;
    if (neighbour_normals != 0 && neighbour_normals != 1) return 0;
    if (check_lattice(X, Y, Z, &empty, &g) != PLIC_OK || empty) return 0;
    if (!neighbour_normals) return fixed_bytes(g) + static_cast<size_t>(g.ntiles) * kDefaultRowsPerTile * kRowBytes;
    return fixed_bytes(g) + static_cast<size_t>(g.ntiles) * kDefaultRowsPerTileNbr * kRowBytesNbr;
}

int plic_curvature_ex_f32(const float* phi, int64_t X, int64_t Y, int64_t Z, float* kappa, int solver,
                          int precision, int normal, int neighbour_normals, void* workspace, size_t workspace_bytes,
                          void* stream) {
    bool empty;
    Grid g{};
    int64_t n = 0;
    if (check_common(phi, X, Y, Z, solver, precision, workspace, workspace_bytes, &empty, &g, &n) != PLIC_OK)
        return PLIC_EINVAL;
    if (!valid_normal(normal) || (neighbour_normals != 0 && neighbour_normals != 1)) return PLIC_EINVAL;
    if (!valid_array(kappa, n)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(n) * sizeof(float);
    if (overlap(phi, nb, kappa, nb)) return PLIC_EINVAL;
    if (!empty && overlap(workspace, workspace_bytes, kappa, nb)) return PLIC_EINVAL;
    if (empty) return PLIC_OK;
    if (workspace_bytes < fixed_bytes(g)) return PLIC_EWORKSPACE;
    return curvature_forward(phi, X, Y, Z, kappa, solver, precision, normal, neighbour_normals != 0, workspace,
                             workspace_bytes, g, static_cast<hipStream_t>(stream));
}

int plic_curvature_f32(const float* phi, int64_t X, int64_t Y, int64_t Z, float* kappa, int solver,
                       int precision, void* workspace, size_t workspace_bytes, void* stream) {
    return plic_curvature_ex_f32(phi, X, Y, Z, kappa, solver, precision, PLIC_NORMAL_PY, 0, workspace,
                                 workspace_bytes, stream);
}

int plic_curvature_noalloc_f32(const float* phi, int64_t X, int64_t Y, int64_t Z, float* kappa, int solver,
                               int precision, void* stream) {
    bool empty;
    Grid g{};
    if (!valid_curvature_solver(solver) || !valid_precision(precision)) return PLIC_EINVAL;
    if (check_lattice(X, Y, Z, &empty, &g) != PLIC_OK) return PLIC_EINVAL;
    const int64_t n = empty ? 0 : X * Y * Z;
    if (!valid_array(phi, n) || !valid_array(kappa, n)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(n) * sizeof(float);
    if (overlap(phi, nb, kappa, nb)) return PLIC_EINVAL;
    if (empty) return PLIC_OK;
    if (fixed_bytes(g) > kScratchBytes) return PLIC_EWORKSPACE;          // beyond the static scratch
    void* ws = nullptr;
    const int rc = scratch_for_current_device(&ws);
    if (rc != PLIC_OK) return rc;
    return curvature_forward(phi, X, Y, Z, kappa, solver, precision, PLIC_NORMAL_PY, false, ws, kScratchBytes, g,
                             static_cast<hipStream_t>(stream));
}


int plic_curvature_backward_ex_f32(const float* phi, int64_t X, int64_t Y, int64_t Z, const float* grad_kappa,
                                   float* grad_phi, int solver, int precision, int normal, int neighbour_normals,
                                   void* workspace, size_t workspace_bytes, void* stream) {
    return curvature_backward(phi, X, Y, Z, grad_kappa, grad_phi, solver, precision, normal, neighbour_normals,
                              workspace, workspace_bytes, stream, false);
}

int plic_curvature_backward_reuse_f32(const float* phi, int64_t X, int64_t Y, int64_t Z, const float* grad_kappa,
                                      float* grad_phi, int solver, int precision, int normal, int neighbour_normals,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    return curvature_backward(phi, X, Y, Z, grad_kappa, grad_phi, solver, precision, normal, neighbour_normals,
                              workspace, workspace_bytes, stream, true);
}

int plic_curvature_backward_f32(const float* phi, int64_t X, int64_t Y, int64_t Z, const float* grad_kappa,
                                float* grad_phi, int solver, int precision, void* workspace,
                                size_t workspace_bytes, void* stream) {
    return plic_curvature_backward_ex_f32(phi, X, Y, Z, grad_kappa, grad_phi, solver, precision, PLIC_NORMAL_PY, 0,
                                          workspace, workspace_bytes, stream);
}

int plic_curvature_status(const void* workspace, size_t workspace_bytes, int64_t X, int64_t Y, int64_t Z,
                          int neighbour_normals, int64_t* interface_cells, size_t* bytes_for_all_rows, void* stream) {
    bool empty;
    Grid g{};
    if (check_lattice(X, Y, Z, &empty, &g) != PLIC_OK || empty) return PLIC_EINVAL;
    if (neighbour_normals != 0 && neighbour_normals != 1) return PLIC_EINVAL;
    if (workspace == nullptr || !aligned(workspace, 4)) return PLIC_EINVAL;
    const bool nbr = neighbour_normals != 0;
    if (workspace_bytes < fixed_bytes(g) + (nbr ? kRowBytesNbr : 0)) return PLIC_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Workspace ws = carve(const_cast<void*>(workspace), workspace_bytes, g, nbr);
    // the call's interface count is the sum of the tiles' counts the scan wrote
    const size_t ntiles = static_cast<size_t>(g.ntiles);
    const std::unique_ptr<unsigned[]> flags(new (std::nothrow) unsigned[ntiles]);
    hipError_t e = flags ? hipStreamSynchronize(st) : hipErrorOutOfMemory;
    if (e == hipSuccess) e = hipMemcpy(flags.get(), ws.flags, ntiles * sizeof(unsigned), hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
        set_last_hip_error(static_cast<int>(e));
        return PLIC_EHIP;
    }
    uint64_t cells = 0;
    for (size_t k = 0; k < ntiles; ++k) cells += flags[k];
    const size_t row_bytes = nbr ? kRowBytesNbr : kRowBytes;
    if (interface_cells) *interface_cells = static_cast<int64_t>(cells);
    if (bytes_for_all_rows) *bytes_for_all_rows = fixed_bytes(g) + static_cast<size_t>(cells) * row_bytes;
    return nbr && cells > ws.rows ? PLIC_EWORKSPACE : PLIC_OK;
}

}  // extern "C"
#endif  // PLIC_PART
