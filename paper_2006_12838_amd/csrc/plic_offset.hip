// Batched PLIC kernels on gfx950: inversion (four solvers), forward volume and
// the backward (vector-Jacobian) pass of the inversion.
//
// Layout: V0 and d0 hold one element per problem; the normals are either three
// such arrays (nx, ny, nz) or, ROWS, one array of rows (x, y, z).  Each thread
// handles VEC consecutive problems with loads and stores of 16 bytes per array (4
// floats or 2 doubles; 2 floats where batches are not large); VEC = 1 covers
// unaligned pointers, and the last block, when it is not whole, goes element by
// element.  One pass over HBM, no reuse.
// The inversion kernels settle the closed-form cases in registers and pack the
// rest (the cubic cases, about 40 % of uniformly random problems) densely in
// LDS before the iterative / trigonometric stage, so that stage runs on full
// wavefronts.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "plic_host.hpp"
#include "plic_math.hpp"

namespace plic {
namespace {

constexpr int kBlock = 256;
// Large float batches: the backward streams 5 input and 4 output arrays;
// workgroups of 512 keep twice the consecutive bytes of each array in flight per
// workgroup, which the memory system serves faster for this many streams
// (measured: a plain 5-read / 4-write copy and this kernel both about 6 % faster
// than with 256).  Others: 256, which fill and leave the chip sooner (20,000 float
// rows 6.9 -> 5.8 us, 10,000 double rows 6.9 -> 5.0 us).
// Measured since: doubles, 16,000,001 and 32,000,011 rows, 256 and 512 threads, SZ 265.0
// and 264.2, 512.8 and 512.8; Newton 283.1 and 285.9, 546.9 and 545.4; unaligned floats,
// 16,000,001 and 64,000,001 in three arrays, SZ 111.0 and 112.4, 452.9 and 455.3.
constexpr int kBwdBlock = 512;
template <int VEC> constexpr int kBwdThreads = VEC == 4 ? kBwdBlock : kBlock;

// Input streams are read once: the loads carry the non-temporal hint (the
// "nt" bit), which keeps them from allocating in the caches as reusable data.
// Measured on a plain 4-read / 1-write stream of 2^26 floats per array:
// 0.84 of the HBM peak against 0.71 without the hint.
template <class S, int VEC> struct NVec;
template <> struct NVec<float, 2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct NVec<float, 4> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct NVec<double, 2> { typedef double type __attribute__((ext_vector_type(2))); };

template <class S, int VEC>
__device__ __forceinline__ void load(const S* __restrict__ p, int64_t i, S (&v)[VEC]) {
    if constexpr (VEC == 1) {
        v[0] = __builtin_nontemporal_load(p + i);
    } else {
        using V = typename NVec<S, VEC>::type;
        const V t = __builtin_nontemporal_load(reinterpret_cast<const V*>(p + i));
#pragma unroll
        for (int k = 0; k < VEC; ++k) v[k] = t[k];
    }
}

// Outputs are written once and not read back by the kernel: non-temporal
// stores, so they do not sit in the last-level cache as dirty lines that the
// next kernel in the stream has to write back.
template <class S, int VEC>
__device__ __forceinline__ void store(S* __restrict__ p, int64_t i, const S (&v)[VEC]) {
    if constexpr (VEC == 1) {
        __builtin_nontemporal_store(v[0], p + i);
    } else {
        using V = typename NVec<S, VEC>::type;
        V t;
#pragma unroll
        for (int k = 0; k < VEC; ++k) t[k] = v[k];
        __builtin_nontemporal_store(t, reinterpret_cast<V*>(p + i));
    }
}

// Loads VEC consecutive elements at i, or those below count (others 0).
// full: the block's problems all lie below count (uniform per block).  VEC = 1
// goes without the hint: its lines are shared by more lanes, and by blocks, than
// one access covers (64,000,001 unaligned problems, rows, SZ: 395 us, with it 402; 4,000,037
// 25.2 and 28.4; volume 224 and 248).
template <class S, int VEC>
__device__ __forceinline__ void load_part(const S* p, int64_t i, int64_t count, bool full, S (&v)[VEC]) {
    if (VEC == 1 && full) {
        v[0] = p[i];
    } else if (full) {
        load<S, VEC>(p, i, v);
    } else {
#pragma unroll
        for (int k = 0; k < VEC; ++k) v[k] = i + k < count ? p[i + k] : S(0);
    }
}

template <class S, int VEC>
__device__ __forceinline__ void store_part(S* p, int64_t i, int64_t count, bool full, const S (&v)[VEC]) {
    if (VEC == 1 && full) {
        p[i] = v[0];
    } else if (full) {
        store<S, VEC>(p, i, v);
    } else {
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            if (i + k < count) p[i + k] = v[k];
    }
}

// ---------------------------------------------------------------------------
// Normals as rows (x, y, z): the 64 VEC rows of a wavefront are 3 KiB of
// consecutive memory (1.5 with 2 floats).  They move as three 16-byte (8-byte)
// accesses per lane over whole cache lines, and change places through LDS to
// and from the VEC rows of each lane; the 48-byte stride of a lane's rows there
// meets every bank once per 8 lanes.  Rows loaded lane by lane instead would touch each line three times,
// and split into component arrays beforehand they cost three strided copies:
// the volume of 10,000,019 rows took 104.6 us so (75 of them the copies) and
// takes 32.5 us here (6.2 TB/s).
// ---------------------------------------------------------------------------
template <class S, int VEC> struct RowStage {
    typename NVec<S, VEC>::type v[3 * 64];
};
template <class S> struct RowStage<S, 1> {};

// keep, when not null, receives a copy of the rows
template <class S, int VEC>
__device__ __forceinline__ void load_rows(const S* n, S* keep, int64_t i, int64_t count, bool full,
                                          RowStage<S, VEC>& st, S (&a)[VEC], S (&b)[VEC], S (&c)[VEC]) {
    if constexpr (VEC > 1) {
        if (full) {
            using V = typename NVec<S, VEC>::type;
            const int lane = threadIdx.x & 63;
            const int64_t first = (i - static_cast<int64_t>(lane) * VEC) * 3;
            V t[3];
#pragma unroll
            for (int j = 0; j < 3; ++j)
                t[j] = __builtin_nontemporal_load(reinterpret_cast<const V*>(n + first) + j * 64 + lane);
#pragma unroll
            for (int j = 0; j < 3; ++j) st.v[j * 64 + lane] = t[j];
            if (keep) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    __builtin_nontemporal_store(t[j], reinterpret_cast<V*>(keep + first) + j * 64 + lane);
            }
            __syncwarp();
            S f[3 * VEC];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const V r = st.v[lane * 3 + j];
#pragma unroll
                for (int k = 0; k < VEC; ++k) f[j * VEC + k] = r[k];
            }
#pragma unroll
            for (int k = 0; k < VEC; ++k) { a[k] = f[3 * k]; b[k] = f[3 * k + 1]; c[k] = f[3 * k + 2]; }
            __syncwarp();
            return;
        }
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        const bool in = full || i + k < count;
        const S* r = n + (i + k) * 3;
        a[k] = in ? r[0] : S(0); b[k] = in ? r[1] : S(0); c[k] = in ? r[2] : S(0);
        if (keep && in) {
            S* o = keep + (i + k) * 3;
            o[0] = a[k]; o[1] = b[k]; o[2] = c[k];
        }
    }
}

template <class S, int VEC>
__device__ __forceinline__ void store_rows(S* n, int64_t i, int64_t count, bool full, RowStage<S, VEC>& st,
                                           const S (&a)[VEC], const S (&b)[VEC], const S (&c)[VEC]) {
    if constexpr (VEC > 1) {
        if (full) {
            using V = typename NVec<S, VEC>::type;
            const int lane = threadIdx.x & 63;
            const int64_t first = (i - static_cast<int64_t>(lane) * VEC) * 3;
            S f[3 * VEC];
#pragma unroll
            for (int k = 0; k < VEC; ++k) { f[3 * k] = a[k]; f[3 * k + 1] = b[k]; f[3 * k + 2] = c[k]; }
            __syncwarp();
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                V r;
#pragma unroll
                for (int k = 0; k < VEC; ++k) r[k] = f[j * VEC + k];
                st.v[lane * 3 + j] = r;
            }
            __syncwarp();
#pragma unroll
            for (int j = 0; j < 3; ++j)
                __builtin_nontemporal_store(st.v[j * 64 + lane], reinterpret_cast<V*>(n + first) + j * 64 + lane);
            return;
        }
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        if (i + k < count) {
            S* o = n + (i + k) * 3;
            o[0] = a[k]; o[1] = b[k]; o[2] = c[k];
        }
    }
}

// LDS of one workgroup: its open problems packed densely.  The cubic stage
// replaces each problem's n1 with its root (the thread that reads an entry
// writes it), which keeps the FP32 kernels within 20 KiB of LDS: 8
// workgroups, 8 waves per SIMD.
template <class T, int VEC> struct PackLds {
    Open<T> q[kBlock * VEC];
    int count[VEC][kBlock / 64];
};

// Reduced offsets d (solver units) of the VEC problems of every thread of the
// workgroup; every thread must call it.  The closed-form cases finish in
// registers; the open ones are packed into LDS in (k, wave, lane) order and
// solved one per lane, so the iterative or trigonometric stage runs on full
// wavefronts instead of on the fraction of lanes that need it.  The result of
// each problem does not depend on the packing (the same stages run on the
// same values), so it equals the one-thread-per-problem offset().
template <int SOLVER, class T, class U, int VEC>
__device__ __forceinline__ void solve_packed(const Reduced<T> (&r)[VEC], const bool (&valid)[VEC], T (&d)[VEC],
                                             PackLds<T, VEC>& sm) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Open<T> o[VEC];
    bool open[VEC];
    unsigned long long bal[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        open[k] = valid[k] && !closed_stage<SOLVER>(r[k], d[k], o[k]);
        bal[k] = __ballot(open[k]);
        if (lane == 0) sm.count[k][wave] = __popcll(bal[k]);
    }
    __syncthreads();
    const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
    int slot[VEC];
    int total = 0;
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            const int c = sm.count[k][w];
            before += w < wave ? c : 0;
            all += c;
        }
        slot[k] = total + before + __popcll(bal[k] & below);
        total += all;
        if (open[k]) sm.q[slot[k]] = o[k];
    }
    __syncthreads();
#pragma unroll 1
    for (int e = tid; e < total; e += kBlock) sm.q[e].n1 = cubic_stage<SOLVER, T, U>(sm.q[e]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < VEC; ++k)
        if (open[k]) d[k] = sm.q[slot[k]].n1;
}

// S: storage type, T: bulk arithmetic, U: cubic-case arithmetic.  d0 may be
// V0 (each element is read and written by the same thread).  ROWS: the normals
// are the rows of nx (ny, nz unused), and keep may ask for a copy of them.
// The last block may reach past count: it takes the checked loads and stores,
// in the same launch (a launch of its own for it cost 5 us at any size).
template <class S, class T, int VEC, bool ROWS> union OffsetLds {
    PackLds<T, VEC> pack;
    RowStage<S, VEC> rows[ROWS ? kBlock / 64 : 1];
};

template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
__device__ __forceinline__ void offset_block(const S* __restrict__ nx, const S* __restrict__ ny,
                                             const S* __restrict__ nz, const S* V0, S* d0, S* keep, int64_t i,
                                             int64_t count, bool full, OffsetLds<S, T, VEC, ROWS>& sm) {
    S a[VEC], b[VEC], c[VEC], v[VEC];
    if constexpr (ROWS) {
        load_rows<S, VEC>(nx, keep, i, count, full, sm.rows[threadIdx.x >> 6], a, b, c);
    } else {
        load_part<S, VEC>(nx, i, count, full, a); load_part<S, VEC>(ny, i, count, full, b);
        load_part<S, VEC>(nz, i, count, full, c);
    }
    load_part<S, VEC>(V0, i, count, full, v);
    if constexpr (ROWS && VEC > 1) __syncthreads();        // the packing reuses the LDS
    Reduced<T> r[VEC];
    bool valid[VEC];
    T d[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        r[k] = reduce(T(a[k]), T(b[k]), T(c[k]), T(v[k]));
        valid[k] = full || i + k < count;
        d[k] = T(0);
    }
    solve_packed<SOLVER, T, U, VEC>(r, valid, d, sm.pack);
    S out[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k)
        out[k] = S(finish<SOLVER>(r[k], d[k], T(a[k]), T(b[k]), T(c[k]), T(v[k])));
    store_part<S, VEC>(d0, i, count, full, out);
}

// FP64 arithmetic on float arrays, four problems a thread, closed forms: the second
// copy of the block, which checks, took these kernels from 126 registers to 130 and
// more, from 4 wavefronts per SIMD to 3 (64,000,001 problems in three arrays, SZ: 484 us,
// and 456 where the last block has a launch of its own).  Their last block goes one
// problem a thread instead, in fewer registers: 450 us, 4 wavefronts; rows
// 525 -> 511, analytic 494 -> 468.
template <int SOLVER, class S, class T, int VEC, bool ROWS>
constexpr bool kOneByOne = sizeof(S) == 4 && sizeof(T) == 8 && VEC == 4 && (SOLVER == kSZ || (SOLVER == kAnalytic && ROWS));

// FP64 arithmetic on unaligned float arrays: the last block's threads past count
// solve its last problem again (the same bits to the same place; V0, which d0 may
// be, is read before the packing's barriers and d0 written after them), so there is
// no second copy of the block: 64,000,001 problems, analytic 657 -> 626 us (at most 88
// registers, not 92), Kawano's variant 813 -> 713 (5 wavefronts per SIMD, not 4),
// Newton 563 -> 555, nested 725 -> 716; SZ is no faster (652 and 664).
template <int SOLVER, class S, class T, int VEC>
constexpr bool kLastAgain = sizeof(S) == 4 && sizeof(T) == 8 && VEC == 1 && SOLVER != kSZ;

template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
__global__ __launch_bounds__(kBlock, (kOneByOne<SOLVER, S, T, VEC, ROWS> ? 4 : 1)) void k_offset(
    const S* __restrict__ nx, const S* __restrict__ ny, const S* __restrict__ nz, const S* V0, S* d0, S* keep, int64_t count) {
    __shared__ OffsetLds<S, T, VEC, ROWS> sm;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * (kBlock * VEC), i = first + threadIdx.x * VEC;
    if constexpr (kLastAgain<SOLVER, S, T, VEC>) {
        offset_block<SOLVER, S, T, U, VEC, ROWS>(nx, ny, nz, V0, d0, keep, min(i, count - 1), count, true, sm);
    } else if (first + kBlock * VEC <= count) {
        offset_block<SOLVER, S, T, U, VEC, ROWS>(nx, ny, nz, V0, d0, keep, i, count, true, sm);
    } else if constexpr (kOneByOne<SOLVER, S, T, VEC, ROWS>) {
        auto& one = reinterpret_cast<OffsetLds<S, T, 1, ROWS>&>(sm);   // (8 KiB more would cost a wavefront per SIMD too)
        static_assert(sizeof(one) <= sizeof(sm));
#pragma unroll 1
        for (int64_t base = first; base < count; base += kBlock)
            offset_block<SOLVER, S, T, U, 1, ROWS>(nx, ny, nz, V0, d0, keep, base + threadIdx.x, count, false, one);
    } else {
        offset_block<SOLVER, S, T, U, VEC, ROWS>(nx, ny, nz, V0, d0, keep, i, count, false, sm);
    }
}

template <class S, class T, int VEC, bool ROWS>
__device__ __forceinline__ void volume_block(const S* __restrict__ nx, const S* __restrict__ ny,
                                             const S* __restrict__ nz, const S* d0, S* V0, int64_t i, int64_t count,
                                             bool full, RowStage<S, VEC>* rows) {
    S a[VEC], b[VEC], c[VEC], v[VEC], r[VEC];
    // FP64 arithmetic on three float arrays: a thread of the last block whose problems
    // all lie below count takes the vector accesses too (1,003 problems 4.2 -> 3.7 us)
    if constexpr (sizeof(S) == 4 && sizeof(T) == 8 && VEC > 1 && !ROWS) full = full || i + VEC <= count;
    if constexpr (ROWS) {
        load_rows<S, VEC>(nx, nullptr, i, count, full, rows[threadIdx.x >> 6], a, b, c);
    } else {
        load_part<S, VEC>(nx, i, count, full, a); load_part<S, VEC>(ny, i, count, full, b);
        load_part<S, VEC>(nz, i, count, full, c);
    }
    load_part<S, VEC>(d0, i, count, full, v);
#pragma unroll
    for (int k = 0; k < VEC; ++k) r[k] = S(volume<T>(T(a[k]), T(b[k]), T(c[k]), T(v[k])));
    store_part<S, VEC>(V0, i, count, full, r);
}

template <class S, class T, int VEC, bool ROWS>
__global__ __launch_bounds__(kBlock) void k_volume(const S* __restrict__ nx, const S* __restrict__ ny,
                                                   const S* __restrict__ nz, const S* d0, S* V0,
                                                   int64_t count) {
    __shared__ RowStage<S, VEC> rows[ROWS ? kBlock / 64 : 1];
    const int64_t first = static_cast<int64_t>(blockIdx.x) * (kBlock * VEC), i = first + threadIdx.x * VEC;
    if constexpr (sizeof(S) == 8 && VEC == 1 && !ROWS) {
        // unaligned doubles, 8 lanes to a line: each thread checks for itself, one copy of
        // the block, and the hint pays (64,000,001: 423 us, 444 with two copies without it)
        if (i < count) {
            S a[1], b[1], c[1], v[1];
            load<S, 1>(nx, i, a); load<S, 1>(ny, i, b); load<S, 1>(nz, i, c); load<S, 1>(d0, i, v);
            const S r[1] = {S(volume<T>(T(a[0]), T(b[0]), T(c[0]), T(v[0])))};
            store<S, 1>(V0, i, r);
        }
    } else if (first + kBlock * VEC <= count) {
        volume_block<S, T, VEC, ROWS>(nx, ny, nz, d0, V0, i, count, true, rows);
    } else {
        volume_block<S, T, VEC, ROWS>(nx, ny, nz, d0, V0, i, count, false, rows);
    }
}

// plane-sphere intersection (Sec. 3): one input and one output array;
// OP 0 inverts (V0 -> d0), OP 1 evaluates the cap volume (d0 -> V0)
template <int OP, class S, class T, int VEC>
__global__ __launch_bounds__(kBlock) void k_sphere(const S* in, S* out, int64_t count) {
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * VEC;
    if (i + VEC <= count) {
        S a[VEC], r[VEC];
        load<S, VEC>(in, i, a);
#pragma unroll
        for (int k = 0; k < VEC; ++k) r[k] = S(OP == 0 ? sphere_offset<T>(T(a[k])) : sphere_volume<T>(T(a[k])));
        store<S, VEC>(out, i, r);
    } else {
        for (int64_t j = i; j < count; ++j)
            out[j] = S(OP == 0 ? sphere_offset<T>(T(in[j])) : sphere_volume<T>(T(in[j])));
    }
}

// vector-Jacobian product of one problem given its offset d0
template <class T>
__device__ __forceinline__ void backward1(T nx, T ny, T nz, T V0, T d0, T gd, T& gx, T& gy, T& gz, T& gv) {
    T g[3];
    const T dv = offset_grad_from_d0<T>(nx, ny, nz, V0, d0, g);
    gx = gd * g[0];
    gy = gd * g[1];
    gz = gd * g[2];
    gv = gd * dv;
    if (__builtin_isnan(d0)) gx = gy = gz = gv = d0;
}

// The backward solves one problem per thread (no packing): its gradient stage
// is as long as the solve, and the packing's LDS and barriers cost more
// occupancy than they save there.  grad_d0 is loaded with the other inputs.
// ROWS: the normals and their gradients are the rows of nx and gnx.
template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
__device__ __forceinline__ void bwd_block(const S* __restrict__ nx, const S* __restrict__ ny, const S* __restrict__ nz,
                                          const S* __restrict__ V0, const S* __restrict__ gd, S* __restrict__ gnx,
                                          S* __restrict__ gny, S* __restrict__ gnz, S* __restrict__ gV0, int64_t i,
                                          int64_t count, bool full, RowStage<S, VEC>* rows) {
    S a[VEC], b[VEC], c[VEC], v[VEC], g[VEC];
    if constexpr (ROWS) {
        load_rows<S, VEC>(nx, nullptr, i, count, full, rows[threadIdx.x >> 6], a, b, c);
    } else {
        load_part<S, VEC>(nx, i, count, full, a); load_part<S, VEC>(ny, i, count, full, b);
        load_part<S, VEC>(nz, i, count, full, c);
    }
    load_part<S, VEC>(V0, i, count, full, v);
    load_part<S, VEC>(gd, i, count, full, g);
    S ox[VEC], oy[VEC], oz[VEC], ov[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        const T d0 = offset<SOLVER, T, U>(T(a[k]), T(b[k]), T(c[k]), T(v[k]));
        T x, y, z, w;
        backward1<T>(T(a[k]), T(b[k]), T(c[k]), T(v[k]), d0, T(g[k]), x, y, z, w);
        ox[k] = S(x); oy[k] = S(y); oz[k] = S(z); ov[k] = S(w);
    }
    if constexpr (ROWS) {
        store_rows<S, VEC>(gnx, i, count, full, rows[threadIdx.x >> 6], ox, oy, oz);
    } else {
        store_part<S, VEC>(gnx, i, count, full, ox); store_part<S, VEC>(gny, i, count, full, oy);
        store_part<S, VEC>(gnz, i, count, full, oz);
    }
    store_part<S, VEC>(gV0, i, count, full, ov);
}

template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
__global__ __launch_bounds__(kBwdThreads<VEC>) void k_offset_bwd(const S* __restrict__ nx, const S* __restrict__ ny,
                                                       const S* __restrict__ nz, const S* __restrict__ V0,
                                                       const S* __restrict__ gd, S* __restrict__ gnx,
                                                       S* __restrict__ gny, S* __restrict__ gnz,
                                                       S* __restrict__ gV0, int64_t count) {
    constexpr int kB = kBwdThreads<VEC>;
    __shared__ RowStage<S, VEC> rows[ROWS ? kB / 64 : 1];
    const int64_t first = static_cast<int64_t>(blockIdx.x) * (kB * VEC), i = first + threadIdx.x * VEC;
    if (first + kB * VEC <= count)
        bwd_block<SOLVER, S, T, U, VEC, ROWS>(nx, ny, nz, V0, gd, gnx, gny, gnz, gV0, i, count, true, rows);
    else
        bwd_block<SOLVER, S, T, U, VEC, ROWS>(nx, ny, nz, V0, gd, gnx, gny, gnz, gV0, i, count, false, rows);
}

inline unsigned grid_for(int64_t count, int vec, int block = kBlock) {
    const int64_t per = static_cast<int64_t>(block) * vec;
    return static_cast<unsigned>((count + per - 1) / per);
}

template <class S> constexpr int kVec = 16 / sizeof(S);

// A dispatch holds at most 2^32 - 1 work-items; batches are launched in
// chunks of 2^30 problems (a multiple of every block's problem count).
constexpr int64_t kChunkProblems = int64_t(1) << 30;

// rows of three elements advance three times as fast as single elements
template <bool ROWS, class S> S* advance(S* p, int64_t base) { return p ? p + base * (ROWS ? 3 : 1) : p; }

template <class S, class T, int VEC, bool ROWS>
void launch_volume_v(const S* nx, const S* ny, const S* nz, const S* d0, S* V0, int64_t count, hipStream_t st) {
    for (int64_t base = 0; base < count; base += kChunkProblems) {
        const int64_t n = count - base < kChunkProblems ? count - base : kChunkProblems;
        hipLaunchKernelGGL((k_volume<S, T, VEC, ROWS>), dim3(grid_for(n, VEC)), dim3(kBlock), 0, st,
                           advance<ROWS>(nx, base), advance<ROWS>(ny, base), advance<ROWS>(nz, base), d0 + base,
                           V0 + base, n);
    }
}

// ---- dispatch ------------------------------------------------------------------
template <int OP, class S>
void launch_sphere(const S* in, S* out, int64_t count, hipStream_t st) {
    const bool vec = aligned(in, 16) && aligned(out, 16);
    for (int64_t base = 0; base < count; base += kChunkProblems) {
        const int64_t n = count - base < kChunkProblems ? count - base : kChunkProblems;
        if (vec)
            hipLaunchKernelGGL((k_sphere<OP, S, S, kVec<S>>), dim3(grid_for(n, kVec<S>)), dim3(kBlock), 0, st,
                               in + base, out + base, n);
        else
            hipLaunchKernelGGL((k_sphere<OP, S, S, 1>), dim3(grid_for(n, 1)), dim3(kBlock), 0, st, in + base,
                               out + base, n);
    }
}

template <class S> struct OffsetArgs {
    const S *nx, *ny, *nz, *V0;
    S *d0, *keep;
    int64_t count;
};

template <class S> struct BwdArgs {
    const S *nx, *ny, *nz, *V0, *gd;
    S *gx, *gy, *gz, *gv;
    int64_t count;
};

template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
void launch_offset_v(const OffsetArgs<S>& p, hipStream_t st) {
    for (int64_t base = 0; base < p.count; base += kChunkProblems) {
        const int64_t n = p.count - base < kChunkProblems ? p.count - base : kChunkProblems;
        hipLaunchKernelGGL((k_offset<SOLVER, S, T, U, VEC, ROWS>), dim3(grid_for(n, VEC)), dim3(kBlock), 0, st,
                           advance<ROWS>(p.nx, base), advance<ROWS>(p.ny, base), advance<ROWS>(p.nz, base),
                           p.V0 + base, p.d0 + base, advance<ROWS>(p.keep, base), n);
    }
}

template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
void launch_bwd_v(const BwdArgs<S>& p, hipStream_t st) {
    for (int64_t base = 0; base < p.count; base += kChunkProblems) {
        const int64_t n = p.count - base < kChunkProblems ? p.count - base : kChunkProblems;
        hipLaunchKernelGGL((k_offset_bwd<SOLVER, S, T, U, VEC, ROWS>), dim3(grid_for(n, VEC, kBwdThreads<VEC>)),
                           dim3(kBwdThreads<VEC>), 0, st, advance<ROWS>(p.nx, base), advance<ROWS>(p.ny, base),
                           advance<ROWS>(p.nz, base), p.V0 + base, p.gd + base, advance<ROWS>(p.gx, base),
                           advance<ROWS>(p.gy, base), advance<ROWS>(p.gz, base), p.gv + base, n);
    }
}

// Up to this many problems of a float batch go two to a thread, more four: four
// take fewer instructions for addresses and stages, two make twice the
// wavefronts, which fill the chip sooner and leave it more evenly.  SZ, us with
// four and with two: forward of rows, 100,003 5.0 and 4.7, 300,007 6.2 and 4.9,
// 1,000,003 9.1 and 8.3, 4,000,037 24.3 and 23.0, 7,900,001 43.2 and 41.9; of three
// arrays, 1,000,003 7.8 and 6.4, 4,000,037 17.7 and 17.6, 7,900,001 29.2 and 30.4;
// backward of rows, 100,003 7.1 and 4.7, 1,000,003 11.2 and 10.0, 4,000,037 29.3 and
// 28.5, 7,900,001 53.3 and 51.0, 12,000,001 75.4 and 77.4; of three arrays, 1,000,003
// 10.6 and 9.0, 7,900,001 53.7 and 50.9.  (A volume is no faster with two at any
// size: 4,000,037 rows 14.7 and 15.3.)  The other solvers behave alike in FP32 and
// mixed arithmetic (7,900,001 rows forward: Newton 44.3 and 44.0, nested 44.5 and 43.1,
// analytic 44.7 and 41.9).  In FP64 arithmetic the closed forms fill the chip with
// fewer problems: SZ forward of rows, 1,500,001 18.1 and 18.0, 2,000,003 21.9 and 22.7,
// 2,500,001 26.1 and 27.2, 7,900,001 69.7 and 76.6; analytic 1,500,001 17.2 and 17.1, 2,000,003
// 20.6 and 21.6, 7,900,001 64.4 and 72.6, of three arrays 54.9 and 64.5; the iterative ones do not
// (Newton 7,900,001 rows 69.0 and 67.0, nested 83.0 and 82.5), nor does a backward (SZ 124.9 and
// 120.5).
constexpr int64_t kManyProblems = 8000000, kManyArrays = 4000000, kManyClosed64 = 2000000;

template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
void launch_v(const OffsetArgs<S>& p, hipStream_t st) {
    launch_offset_v<SOLVER, S, T, U, VEC, ROWS>(p, st);
}
template <int SOLVER, class S, class T, class U, int VEC, bool ROWS>
void launch_v(const BwdArgs<S>& p, hipStream_t st) {
    launch_bwd_v<SOLVER, S, T, U, VEC, ROWS>(p, st);
}

template <int SOLVER, class S, class T, class U, bool ROWS, class Args>
void launch_t(const Args& p, bool vec, hipStream_t st) {
    if (!vec) return launch_v<SOLVER, S, T, U, 1, ROWS>(p, st);
    constexpr bool kForward = std::is_same_v<Args, OffsetArgs<S>>;
    constexpr bool kClosed64 = kForward && sizeof(T) == 8 && (SOLVER == kSZ || SOLVER == kAnalytic);
    constexpr int64_t kMany = kClosed64 ? kManyClosed64 : (kForward && !ROWS ? kManyArrays : kManyProblems);
    if constexpr (sizeof(S) == 4)
        if (p.count > kMany) return launch_v<SOLVER, S, T, U, 4, ROWS>(p, st);
    launch_v<SOLVER, S, T, U, 2, ROWS>(p, st);
}

// the solver's kernel for a forward (OffsetArgs) or a backward (BwdArgs)
template <class S, class T, class U, bool ROWS, class Args>
void launch_s(int solver, const Args& p, bool vec, hipStream_t st) {
    switch (solver) {
        case kSZ: launch_t<kSZ, S, T, U, ROWS>(p, vec, st); break;
        case kNewton: launch_t<kNewton, S, T, U, ROWS>(p, vec, st); break;
        case kNested: launch_t<kNested, S, T, U, ROWS>(p, vec, st); break;
        case kKawano: launch_t<kKawano, S, T, U, ROWS>(p, vec, st); break;
        default: launch_t<kAnalytic, S, T, U, ROWS>(p, vec, st); break;
    }
}

template <bool ROWS, class Args>
void launch_f32(int solver, int precision, const Args& p, bool vec, hipStream_t st) {
    if (precision == PLIC_FP32) launch_s<float, float, float, ROWS>(solver, p, vec, st);
    else if (precision == PLIC_MIXED) launch_s<float, float, double, ROWS>(solver, p, vec, st);
    else launch_s<float, double, double, ROWS>(solver, p, vec, st);
}

template <class S>
bool all_aligned16(std::initializer_list<const void*> ps) {
    for (const void* p : ps)
        if (!aligned(p, 16)) return false;
    return true;
}

// normals as rows: 3 count elements, overlapping nothing that is written
template <class S>
int offset_rows_entry(const S* n, const S* V0, S* d0, S* keep, int64_t count, int solver, int precision, void* stream) {
    if (count < 0 || count > INT64_MAX / 64 || !valid_solver(solver) || !valid_precision(precision)) return PLIC_EINVAL;
    if (!valid_array(n, count) || !valid_array(V0, count) || !valid_array(d0, count) || !aligned(keep, sizeof(S)))
        return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(S), kb = keep ? 3 * nb : 0;
    if (overlap(d0, nb, n, 3 * nb) || (overlap(d0, nb, V0, nb) && d0 != V0)) return PLIC_EINVAL;
    if (overlap(keep, kb, n, 3 * nb) || overlap(keep, kb, V0, nb) || overlap(keep, kb, d0, nb)) return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<S>({n, V0, d0, keep});
    const OffsetArgs<S> p{n, nullptr, nullptr, V0, d0, keep, count};
    if constexpr (sizeof(S) == 4) launch_f32<true>(solver, precision, p, vec, st);
    else launch_s<double, double, double, true>(solver, p, vec, st);
    return launch_status();
}

template <class S>
int volume_rows_entry(const S* n, const S* d0, S* V0, int64_t count, int precision, void* stream) {
    if (count < 0 || count > INT64_MAX / 64 || !valid_precision(precision)) return PLIC_EINVAL;
    if (!valid_array(n, count) || !valid_array(d0, count) || !valid_array(V0, count)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(S);
    if (overlap(V0, nb, n, 3 * nb) || (overlap(V0, nb, d0, nb) && V0 != d0)) return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<S>({n, d0, V0});
    const S* no = nullptr;
    if (sizeof(S) == 4 && precision != PLIC_FP64) {
        if (vec) launch_volume_v<S, S, kVec<S>, true>(n, no, no, d0, V0, count, st);
        else launch_volume_v<S, S, 1, true>(n, no, no, d0, V0, count, st);
    } else {
        if (vec) launch_volume_v<S, double, kVec<S>, true>(n, no, no, d0, V0, count, st);
        else launch_volume_v<S, double, 1, true>(n, no, no, d0, V0, count, st);
    }
    return launch_status();
}

template <class S>
int bwd_rows_entry(const S* n, const S* V0, const S* gd, S* gn, S* gv, int64_t count, int solver, int precision,
                   void* stream) {
    if (count < 0 || count > INT64_MAX / 64 || !valid_solver(solver) || !valid_precision(precision)) return PLIC_EINVAL;
    for (const S* p : {n, V0, gd}) if (!valid_array(p, count)) return PLIC_EINVAL;
    if (!valid_array(gn, count) || !valid_array(gv, count)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(S);
    if (overlap(gn, 3 * nb, n, 3 * nb) || overlap(gn, 3 * nb, V0, nb) || overlap(gn, 3 * nb, gd, nb) ||
        overlap(gn, 3 * nb, gv, nb) || overlap(gv, nb, n, 3 * nb) || overlap(gv, nb, V0, nb) || overlap(gv, nb, gd, nb))
        return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<S>({n, V0, gd, gn, gv});
    const BwdArgs<S> p{n, nullptr, nullptr, V0, gd, gn, nullptr, nullptr, gv, count};
    if constexpr (sizeof(S) == 4) launch_f32<true>(solver, precision, p, vec, st);
    else launch_s<double, double, double, true>(solver, p, vec, st);
    return launch_status();
}

// plane-sphere entry points: in and out may be the same array (each element
// is read and written by the same thread); otherwise they must not overlap
template <int OP, class S>
int sphere_entry(const S* in, S* out, int64_t count, void* stream) {
    if (count < 0 || !valid_array(in, count) || !valid_array(out, count)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(S);
    if (static_cast<const void*>(in) != static_cast<const void*>(out) && overlap(in, nb, out, nb)) return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    launch_sphere<OP, S>(in, out, count, static_cast<hipStream_t>(stream));
    return launch_status();
}

}  // namespace
}  // namespace plic

using namespace plic;

extern "C" {

int plic_offset_f32(const float* nx, const float* ny, const float* nz, const float* V0, float* d0,
                    int64_t count, int solver, int precision, void* stream) {
    if (count < 0 || !valid_solver(solver) || !valid_precision(precision)) return PLIC_EINVAL;
    if (!valid_array(nx, count) || !valid_array(ny, count) || !valid_array(nz, count) ||
        !valid_array(V0, count) || !valid_array(d0, count))
        return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(float);
    if ((overlap(d0, nb, nx, nb) || overlap(d0, nb, ny, nb) || overlap(d0, nb, nz, nb) ||
         overlap(d0, nb, V0, nb)) && d0 != V0)
        return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<float>({nx, ny, nz, V0, d0});
    launch_f32<false>(solver, precision, OffsetArgs<float>{nx, ny, nz, V0, d0, nullptr, count}, vec, st);
    return launch_status();
}

int plic_offset_f64(const double* nx, const double* ny, const double* nz, const double* V0, double* d0,
                    int64_t count, int solver, void* stream) {
    if (count < 0 || !valid_solver(solver)) return PLIC_EINVAL;
    if (!valid_array(nx, count) || !valid_array(ny, count) || !valid_array(nz, count) ||
        !valid_array(V0, count) || !valid_array(d0, count))
        return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(double);
    if ((overlap(d0, nb, nx, nb) || overlap(d0, nb, ny, nb) || overlap(d0, nb, nz, nb) ||
         overlap(d0, nb, V0, nb)) && d0 != V0)
        return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<double>({nx, ny, nz, V0, d0});
    launch_s<double, double, double, false>(solver, OffsetArgs<double>{nx, ny, nz, V0, d0, nullptr, count}, vec, st);
    return launch_status();
}

int plic_volume_f32(const float* nx, const float* ny, const float* nz, const float* d0, float* V0,
                    int64_t count, int precision, void* stream) {
    if (count < 0 || !valid_precision(precision)) return PLIC_EINVAL;
    if (!valid_array(nx, count) || !valid_array(ny, count) || !valid_array(nz, count) ||
        !valid_array(d0, count) || !valid_array(V0, count))
        return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(float);
    if ((overlap(V0, nb, nx, nb) || overlap(V0, nb, ny, nb) || overlap(V0, nb, nz, nb) ||
         overlap(V0, nb, d0, nb)) && V0 != d0)
        return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<float>({nx, ny, nz, d0, V0});
    if (precision == PLIC_FP64) {
        if (vec) launch_volume_v<float, double, 4, false>(nx, ny, nz, d0, V0, count, st);
        else launch_volume_v<float, double, 1, false>(nx, ny, nz, d0, V0, count, st);
    } else {
        if (vec) launch_volume_v<float, float, 4, false>(nx, ny, nz, d0, V0, count, st);
        else launch_volume_v<float, float, 1, false>(nx, ny, nz, d0, V0, count, st);
    }
    return launch_status();
}

int plic_volume_f64(const double* nx, const double* ny, const double* nz, const double* d0, double* V0,
                    int64_t count, void* stream) {
    if (count < 0) return PLIC_EINVAL;
    if (!valid_array(nx, count) || !valid_array(ny, count) || !valid_array(nz, count) ||
        !valid_array(d0, count) || !valid_array(V0, count))
        return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(double);
    if ((overlap(V0, nb, nx, nb) || overlap(V0, nb, ny, nb) || overlap(V0, nb, nz, nb) ||
         overlap(V0, nb, d0, nb)) && V0 != d0)
        return PLIC_EINVAL;
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (all_aligned16<double>({nx, ny, nz, d0, V0})) launch_volume_v<double, double, 2, false>(nx, ny, nz, d0, V0, count, st);
    else launch_volume_v<double, double, 1, false>(nx, ny, nz, d0, V0, count, st);
    return launch_status();
}

int plic_offset_backward_f32(const float* nx, const float* ny, const float* nz, const float* V0,
                             const float* grad_d0, float* grad_nx, float* grad_ny, float* grad_nz,
                             float* grad_V0, int64_t count, int solver, int precision, void* stream) {
    if (count < 0 || !valid_solver(solver) || !valid_precision(precision)) return PLIC_EINVAL;
    const float* ins[5] = {nx, ny, nz, V0, grad_d0};
    float* outs[4] = {grad_nx, grad_ny, grad_nz, grad_V0};
    for (const float* p : ins) if (!valid_array(p, count)) return PLIC_EINVAL;
    for (float* p : outs) if (!valid_array(p, count)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(float);
    for (int a = 0; a < 4; ++a) {
        for (const float* p : ins) if (overlap(outs[a], nb, p, nb)) return PLIC_EINVAL;
        for (int b = a + 1; b < 4; ++b) if (overlap(outs[a], nb, outs[b], nb)) return PLIC_EINVAL;
    }
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<float>({nx, ny, nz, V0, grad_d0, grad_nx, grad_ny, grad_nz, grad_V0});
    launch_f32<false>(solver, precision,
                      BwdArgs<float>{nx, ny, nz, V0, grad_d0, grad_nx, grad_ny, grad_nz, grad_V0, count}, vec, st);
    return launch_status();
}

int plic_offset_backward_f64(const double* nx, const double* ny, const double* nz, const double* V0,
                             const double* grad_d0, double* grad_nx, double* grad_ny, double* grad_nz,
                             double* grad_V0, int64_t count, int solver, void* stream) {
    if (count < 0 || !valid_solver(solver)) return PLIC_EINVAL;
    const double* ins[5] = {nx, ny, nz, V0, grad_d0};
    double* outs[4] = {grad_nx, grad_ny, grad_nz, grad_V0};
    for (const double* p : ins) if (!valid_array(p, count)) return PLIC_EINVAL;
    for (double* p : outs) if (!valid_array(p, count)) return PLIC_EINVAL;
    const size_t nb = static_cast<size_t>(count) * sizeof(double);
    for (int a = 0; a < 4; ++a) {
        for (const double* p : ins) if (overlap(outs[a], nb, p, nb)) return PLIC_EINVAL;
        for (int b = a + 1; b < 4; ++b) if (overlap(outs[a], nb, outs[b], nb)) return PLIC_EINVAL;
    }
    if (count == 0) return PLIC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool vec = all_aligned16<double>({nx, ny, nz, V0, grad_d0, grad_nx, grad_ny, grad_nz, grad_V0});
    launch_s<double, double, double, false>(
        solver, BwdArgs<double>{nx, ny, nz, V0, grad_d0, grad_nx, grad_ny, grad_nz, grad_V0, count}, vec, st);
    return launch_status();
}

int plic_offset_rows_f32(const float* n, const float* V0, float* d0, float* n_copy, int64_t count, int solver,
                         int precision, void* stream) {
    return offset_rows_entry<float>(n, V0, d0, n_copy, count, solver, precision, stream);
}
int plic_offset_rows_f64(const double* n, const double* V0, double* d0, double* n_copy, int64_t count, int solver,
                         void* stream) {
    return offset_rows_entry<double>(n, V0, d0, n_copy, count, solver, PLIC_FP64, stream);
}
int plic_volume_rows_f32(const float* n, const float* d0, float* V0, int64_t count, int precision, void* stream) {
    return volume_rows_entry<float>(n, d0, V0, count, precision, stream);
}
int plic_volume_rows_f64(const double* n, const double* d0, double* V0, int64_t count, void* stream) {
    return volume_rows_entry<double>(n, d0, V0, count, PLIC_FP64, stream);
}
int plic_offset_backward_rows_f32(const float* n, const float* V0, const float* grad_d0, float* grad_n, float* grad_V0,
                                  int64_t count, int solver, int precision, void* stream) {
    return bwd_rows_entry<float>(n, V0, grad_d0, grad_n, grad_V0, count, solver, precision, stream);
}
int plic_offset_backward_rows_f64(const double* n, const double* V0, const double* grad_d0, double* grad_n,
                                  double* grad_V0, int64_t count, int solver, void* stream) {
    return bwd_rows_entry<double>(n, V0, grad_d0, grad_n, grad_V0, count, solver, PLIC_FP64, stream);
}

int plic_sphere_offset_f32(const float* V0, float* d0, int64_t count, void* stream) {
    return sphere_entry<0, float>(V0, d0, count, stream);
}
int plic_sphere_offset_f64(const double* V0, double* d0, int64_t count, void* stream) {
    return sphere_entry<0, double>(V0, d0, count, stream);
}
int plic_sphere_volume_f32(const float* d0, float* V0, int64_t count, void* stream) {
    return sphere_entry<1, float>(d0, V0, count, stream);
}
int plic_sphere_volume_f64(const double* d0, double* V0, int64_t count, void* stream) {
    return sphere_entry<1, double>(d0, V0, count, stream);
}

}  // extern "C"
