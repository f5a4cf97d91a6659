// lbm_device.hpp -- device-side building blocks of the gfx950 library:
// the D3Q19 velocity set, storage traits, the TRT collision of one cell, and
// launch helpers.  Included by every .hip translation unit of the library.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "lbm.h"

namespace lbm {

// ---------------------------------------------------------------------------
// D3Q19.  Populations come in opposite pairs (2k-1, 2k), k = 1..9; the odd
// member's velocity is listed, the even member is its negative.
// ---------------------------------------------------------------------------
constexpr int Q = 19;
constexpr int NPAIR = 9;
// velocity of the odd member 2k-1 of pair k (index k-1)
constexpr int PCX[NPAIR] = {1, 0, 0, 1, 1, 1, 1, 0, 0};
constexpr int PCY[NPAIR] = {0, 1, 0, 1, -1, 0, 0, 1, 1};
constexpr int PCZ[NPAIR] = {0, 0, 1, 0, 0, 1, -1, 1, -1};
// 1/18 for the three axis pairs, 1/36 for the six diagonal pairs
__host__ __device__ constexpr double pair_weight(int k) { return k < 3 ? 1.0 / 18.0 : 1.0 / 36.0; }
constexpr double W0 = 1.0 / 3.0;

__host__ __device__ constexpr int opp(int i) { return i == 0 ? 0 : ((i & 1) ? i + 1 : i - 1); }
__host__ __device__ constexpr int vel_x(int i) { return i == 0 ? 0 : ((i & 1) ? PCX[(i - 1) / 2] : -PCX[(i - 1) / 2]); }
__host__ __device__ constexpr int vel_y(int i) { return i == 0 ? 0 : ((i & 1) ? PCY[(i - 1) / 2] : -PCY[(i - 1) / 2]); }
__host__ __device__ constexpr int vel_z(int i) { return i == 0 ? 0 : ((i & 1) ? PCZ[(i - 1) / 2] : -PCZ[(i - 1) / 2]); }
__host__ __device__ constexpr double weight(int i) { return i == 0 ? W0 : pair_weight((i - 1) / 2); }

// ---------------------------------------------------------------------------
// Storage traits: element type T in memory, arithmetic type A, shift flag.
// ---------------------------------------------------------------------------
template <int ST> struct Storage;
template <> struct Storage<LBM_F64> { using T = double; using A = double; static constexpr bool shifted = false; };
template <> struct Storage<LBM_F64_SHIFTED> { using T = double; using A = double; static constexpr bool shifted = true; };
template <> struct Storage<LBM_F32> { using T = float; using A = float; static constexpr bool shifted = false; };
template <> struct Storage<LBM_F32_SHIFTED> { using T = float; using A = float; static constexpr bool shifted = true; };
template <> struct Storage<LBM_F16_SHIFTED> { using T = _Float16; using A = float; static constexpr bool shifted = true; };

// FP16 holding 2^12 x the value (LBM_F16_SHIFTED_SCALED).  Scaling by a power
// of two is exact in FP32, so loading and storing round exactly as the
// unscaled FP16 form does, only in a range shifted down by 12 binades.
struct Half12 {
    _Float16 bits;
    static constexpr float kUp = 4096.0f, kDown = 1.0f / 4096.0f;
    __host__ __device__ explicit operator float() const { return static_cast<float>(bits) * kDown; }
    __host__ __device__ explicit operator double() const {
        return static_cast<double>(static_cast<float>(bits) * kDown);
    }
};
template <> struct Storage<LBM_F16_SHIFTED_SCALED> { using T = Half12; using A = float; static constexpr bool shifted = true; };

template <class T, class A> __device__ __forceinline__ A ld(const T* p) { return static_cast<A>(*p); }
// Memory policy of a launch, chosen by sweep_launch() from the bytes that a
// step touches.
//  kCached    the state stays in the last-level cache from step to step: plain
//             loads and stores throughout.
//  kStream    larger: rows read once per step (adjacency, 16-bit codes) come
//             in through nontemporal loads, which keeps them from displacing
//             the PDF lines whose partial reuse by neighbouring cells the
//             caches serve; plain stores.
//  kStreamNT  the same with nontemporal stores of the new PDFs.
enum Policy { kCached = 0, kStream = 1, kStreamNT = 2 };

template <int POL, class T> __device__ __forceinline__ T ld_stream(const T* p) {
    if constexpr (POL == kCached)
        return *p;
    else
        return __builtin_nontemporal_load(p);
}
template <int POL> __device__ __forceinline__ Half12 ld_stream(const Half12* p) {
    if constexpr (POL == kCached)
        return *p;
    else
        return Half12{__builtin_nontemporal_load(&p->bits)};
}
// One adjacency code of the two-array sweep.  8-bit codes are read with plain
// loads under every policy: a wave reads half a line of a code row, and the other half is the
// next wave's (sweep of 54 M cells, nontemporal -> plain code loads: FP64
// 3,287 -> 3,258 us, shifted FP32 1,780 -> 1,662, scaled FP16 1,110 -> 1,099;
// 12.7 M cells: 783 -> 759, 437 -> 428, 251 -> 243).  A 16-bit row gives a
// wave a whole line, and 32-bit rows two: those are read once and streamed
// (full list, FP64, 23 M cells: 1,510 us nontemporal, 1,541 plain).
template <int POL, class CT> __device__ __forceinline__ int32_t ld_code(const CT* p) {
    if constexpr (sizeof(CT) == 1)
        return *p;
    else
        return ld_stream<POL>(p);
}
// FP32 -> FP16 conversion rounds to nearest even (IEEE default mode).  The
// value is first rounded to A: device code is built without contraction, so
// no fused product-sum exists that the conversion could absorb, and the empty
// asm hides how the value was computed, so no mixed-precision instruction can
// round an unrounded result straight to FP16 (with contraction on, the
// compiler once did so in one kernel and not in another, and their results
// differed in the last bit).
template <class T, class A, bool NT> __device__ __forceinline__ void st(T* p, A v) {
    if constexpr (!std::is_same_v<T, A>) asm("" : "+v"(v));
    if constexpr (std::is_same_v<T, Half12>) {
        const _Float16 b = static_cast<_Float16>(v * Half12::kUp);  // exact scaling, one rounding
        if constexpr (NT)
            __builtin_nontemporal_store(b, &p->bits);
        else
            p->bits = b;
    } else if constexpr (NT) {
        __builtin_nontemporal_store(static_cast<T>(v), p);
    } else {
        *p = static_cast<T>(v);
    }
}

inline size_t storage_bytes(int st) {
    switch (st) {
    case LBM_F64: case LBM_F64_SHIFTED: return 8;
    case LBM_F32: case LBM_F32_SHIFTED: return 4;
    case LBM_F16_SHIFTED: case LBM_F16_SHIFTED_SCALED: return 2;
    default: return 0;
    }
}

// 16-bit adjacency codes (lbm_compress_adjacency): tiles of 256 list cells,
// one record of 20 int32 words per tile (18 direction offsets, the number of
// escape codes in the tile, the narrow flag of lbm_narrow_codes); reserved
// code values.
constexpr int kCodeTile = 256;
constexpr int kCodeRec = 20;
constexpr int16_t kCodeBounce = -32768;
constexpr int16_t kCodeEscape = -32767;
constexpr int32_t kCodeMin = -32766;
constexpr int32_t kCodeMax = 32767;
// 8-bit form of a tile's codes (lbm_narrow_codes): the same code in one byte,
// bounce-back as -128.
constexpr int8_t kCode8Bounce = -128;
constexpr int32_t kCode8Max = 127;

// ---------------------------------------------------------------------------
// TRT constants of one launch (host-computed in FP64).
// ---------------------------------------------------------------------------
struct TrtConst {
    double sp, sm;       // s+ = 1/tau+, s- = 1/tau-
    double F[NPAIR];     // 3 w c.G for the odd member of each pair
};

// 3 w c.G for the odd member of pair k
__host__ __device__ inline double force_term(int k, const double* force) {
    return 3.0 * pair_weight(k) * (PCX[k] * force[0] + PCY[k] * force[1] + PCZ[k] * force[2]);
}

inline TrtConst make_trt_const(const lbm_params& p) {
    TrtConst c;
    double tau_minus = 0.5 + p.magic / (p.tau_plus - 0.5);
    c.sp = 1.0 / p.tau_plus;
    c.sm = 1.0 / tau_minus;
    for (int k = 0; k < NPAIR; ++k) c.F[k] = force_term(k, p.force);
    return c;
}

// ---------------------------------------------------------------------------
// One cell's TRT collision.  g[19] are the gathered populations (pre-collision),
// in the arithmetic type A.  Writes the post-collision f*[19] into out[] and,
// if PBB, blends with the bounce-back g_opp.  rho/j are returned for callers
// that need them (the adjoint).
// ---------------------------------------------------------------------------
template <class A>
struct CellMoments {
    A rho, jx, jy, jz;
};

template <class A>
__device__ __forceinline__ CellMoments<A> cell_moments(const A* g) {
    CellMoments<A> m;
    A rho = g[0];
    A d[NPAIR];
#pragma unroll
    for (int k = 0; k < NPAIR; ++k) {
        rho += g[2 * k + 1] + g[2 * k + 2];
        d[k] = g[2 * k + 1] - g[2 * k + 2];
    }
    m.rho = rho;
    // j = sum over pairs of c_odd * (g_odd - g_even)
    m.jx = d[0] + d[3] + d[4] + d[5] + d[6];
    m.jy = d[1] + d[3] - d[4] + d[7] + d[8];
    m.jz = d[2] + d[5] - d[6] + d[7] - d[8];
    return m;
}

// The collision of one cell with moments m, one population pair at a time.
template <class A>
struct TrtCell {
    A sp, sm, base;  // base = rho - 3/2 |j|^2
    CellMoments<A> m;
    __device__ __forceinline__ TrtCell(const CellMoments<A>& cm, const TrtConst& c)
        : sp(static_cast<A>(c.sp)), sm(static_cast<A>(c.sm)), m(cm) {
        const A jj = m.jx * m.jx + m.jy * m.jy + m.jz * m.jz;
        base = m.rho - A(1.5) * jj;
    }
    // rest population: g+ = g0, g- = 0, e+ = w0 (rho - 3/2 |j|^2)
    __device__ __forceinline__ A rest(A g0) const {
        return g0 - sp * (g0 - static_cast<A>(W0) * base);
    }
    __device__ __forceinline__ void pair(int k, A ga, A gb, const TrtConst& c, A& fa, A& fb) const {
        const A w = static_cast<A>(pair_weight(k));
        const A cu = A(PCX[k]) * m.jx + A(PCY[k]) * m.jy + A(PCZ[k]) * m.jz;
        const A ep = w * (base + A(4.5) * cu * cu);
        const A em = A(3) * w * cu;
        const A gp = A(0.5) * (ga + gb);
        const A gm = A(0.5) * (ga - gb);
        const A rp = sp * (gp - ep);
        const A rm = sm * (gm - em);
        const A F = static_cast<A>(c.F[k]);
        fa = ga - rp - rm + F;
        fb = gb - rp + rm - F;
    }
};

template <class A, bool PBB>
__device__ __forceinline__ void trt_collide(const A* g, A* out, const TrtConst& c, A ns) {
    const TrtCell<A> t(cell_moments(g), c);
    A f0 = t.rest(g[0]);
    if constexpr (PBB) f0 = (A(1) - ns) * f0 + ns * g[0];
    out[0] = f0;
#pragma unroll
    for (int k = 0; k < NPAIR; ++k) {
        const int a = 2 * k + 1, b = 2 * k + 2;
        A fa, fb;
        t.pair(k, g[a], g[b], c, fa, fb);
        if constexpr (PBB) {
            fa = (A(1) - ns) * fa + ns * g[b];
            fb = (A(1) - ns) * fb + ns * g[a];
        }
        out[a] = fa;
        out[b] = fb;
    }
}

// ---------------------------------------------------------------------------
// One cell update of the pull sweep: gather the 18 upstream populations
// through adj (plus the own rest population), collide, store the 19 results
// to the cell's own column of the destination rows.
// ---------------------------------------------------------------------------
template <int ST, bool PBB, int POL>
__device__ __forceinline__ void update_cell(const typename Storage<ST>::T* __restrict__ src,
                                            typename Storage<ST>::T* __restrict__ dst,
                                            const uint32_t* __restrict__ adj,
                                            const double* __restrict__ ns, int64_t m,
                                            int64_t stride, const TrtConst& c) {
    using T = typename Storage<ST>::T;
    using A = typename Storage<ST>::A;
    uint32_t a[Q - 1];
    const uint32_t* ap = adj + m;
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) a[k] = ld_stream<POL>(ap + k * stride);
    A g[Q];
    g[0] = ld<T, A>(src + m);
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) g[k + 1] = ld<T, A>(src + a[k]);
    A s = A(0);
    if constexpr (PBB) s = static_cast<A>(ns[m]);
    A out[Q];
    trt_collide<A, PBB>(g, out, c, s);
    T* dp = dst + m;
#pragma unroll
    for (int i = 0; i < Q; ++i) st<T, A, POL == kStreamNT>(dp + i * stride, out[i]);
}

// One cell update of an escape-free tile, the slots rebuilt from the 16-bit
// (CT = int16_t) or 8-bit (int8_t) codes in 32-bit arithmetic (every slot is
// below 19 * stride < 2^32).  The per-tile part i * stride + tile * 256 + toff
// is uniform (scalar); per lane it adds the lane and the code.
template <int ST, bool PBB, int POL, class CT>
__device__ __forceinline__ void update_cell_coded(const typename Storage<ST>::T* __restrict__ src,
                                                  typename Storage<ST>::T* __restrict__ dst,
                                                  const CT* __restrict__ codes,
                                                  const int32_t* __restrict__ rec,
                                                  const double* __restrict__ ns, int64_t m,
                                                  int64_t stride, const TrtConst& c) {
    using T = typename Storage<ST>::T;
    using A = typename Storage<ST>::A;
    constexpr int32_t bounce = std::is_same_v<CT, int8_t> ? int32_t(kCode8Bounce)
                                                          : int32_t(kCodeBounce);
    int32_t cd[Q - 1];
    const CT* cp = codes + m;
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) cd[k] = ld_code<POL>(cp + k * stride);
    const uint32_t S = uint32_t(stride);
    const uint32_t mm = uint32_t(m);
    A g[Q];
    g[0] = ld<T, A>(src + m);
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        const uint32_t i = k + 1;
        const uint32_t streamed = i * S + uint32_t(rec[k]) + mm + uint32_t(cd[k]);
        const uint32_t bounced = uint32_t(opp(int(i))) * S + mm;
        g[i] = ld<T, A>(src + (cd[k] == bounce ? bounced : streamed));
    }
    A sf = A(0);
    if constexpr (PBB) sf = static_cast<A>(ns[m]);
    A out[Q];
    trt_collide<A, PBB>(g, out, c, sf);
    T* dp = dst + m;
#pragma unroll
    for (int i = 0; i < Q; ++i) st<T, A, POL == kStreamNT>(dp + i * stride, out[i]);
}

// ---------------------------------------------------------------------------
// Launch geometry.  Workgroups are handed to the 8 XCDs of the MI355X round
// robin (workgroup w runs on XCD w % 8; checked on the device through the
// XCC_ID hardware register), and each XCD has its own L2.  The sweep relabels
// workgroups so that each XCD takes a run of consecutive blocks of the list:
// the gathers of neighbouring blocks share cache lines at block edges, which
// then stay in one L2.
// ---------------------------------------------------------------------------
constexpr int NXCD = 8;

// Runs of `run` consecutive blocks, dealt to the XCDs in turn.  Virtual block v
// of group s = v >> group_shift of 8 runs is block (v >> 3) & mask of XCD
// v % 8's run; a map of one run per XCD has one group (group_shift 31, every
// index bit in mask).  Written without a branch or a division: a sweep of a
// few workgroups waits for this before its first load.  Block indices are
// below 2^31: a list has fewer than 2^32 / 19 cells.
struct XcdMap {
    uint32_t group_shift, run, mask;
    uint32_t flip, off;  // ~0 and the block count: from the last block to the first
};

constexpr XcdMap map_of_runs(int shift) {
    return XcdMap{3u + shift, 1u << shift, (1u << shift) - 1, 0u, 0u};
}
constexpr XcdMap map_of_eighths(int64_t blocks) {
    return XcdMap{31u, uint32_t((blocks + NXCD - 1) / NXCD), ~0u, 0u, 0u};
}

// (Padding blocks of a flipped map wrap to indices above every block.)
__device__ __forceinline__ uint32_t logical_of(uint32_t v, XcdMap map) {
    const uint32_t b = ((v >> map.group_shift) << map.group_shift) + (v & (NXCD - 1)) * map.run +
                       ((v >> 3) & map.mask);
    return (b ^ map.flip) + map.off;
}

__device__ __forceinline__ int64_t logical_block(XcdMap map) { return logical_of(blockIdx.x, map); }

// Virtual blocks of a map over `blocks` blocks (whole groups of NXCD runs).
__host__ __device__ inline int64_t virtual_blocks(int64_t blocks, XcdMap map) {
    const int64_t q = int64_t(NXCD) * map.run;
    return (blocks + q - 1) / q * q;
}

// Launch of a sweep over n cells, one workgroup per 256-cell tile: the memory
// policy and the XCD map.  They follow from the bytes that one step touches
// (cell_bytes per cell) and from the launch hints in the flags:
//  * up to 240 MiB the state stays in the 256 MiB last-level cache: kCached,
//    and one run of an eighth of the blocks per XCD, so that an XCD finds the
//    lines that it wrote itself.  Nontemporal accesses and short runs only cost
//    here (246 MB, us a sweep, this form / nontemporal stores and loads in runs
//    of 1 tile: scaled FP16 over 8-bit codes 40.1 / 57.3, FP64 over 8-bit codes
//    38.7 / 49.3; shifted FP32 over 8-bit codes at 204 MB 32.3 / 48.1; FP64 full
//    list at 165 MB 25.9 / 32.7, at 41 MB 8.0 / 10.6).
//  * that holds for a state that is swept again before others have passed
//    through the cache.  Only the caller knows whether it is, so hints are
//    followed in calls of one sweep; from two on the call itself brings the state
//    in.  Time with hints followed over this form (FP64, shifted FP32, scaled
//    FP16, five forms, 30 to 240 MiB, hints of nontemporal stores and 1, 8, 64
//    tiles or none; smallest / median / largest): one state, calls of 1 or 2
//    sweeps, 0.94 / 1.24 / 1.51 and 1.02 / 1.26 / 1.50; as many states in turn as
//    take 1.2 GB, calls of 1, 2 or 4 sweeps, 0.89 / 0.99 / 1.33, 0.91 / 1.07 /
//    1.33 and 0.98 / 1.16 / 1.44.
//  * from there to SweepRule::whole_runs the cache still holds most of it.
//    Without hints one run per XCD and plain stores; the two-array sweep
//    alternates its direction, so that a sweep begins with what the one before
//    left behind (us, this form / one direction / runs of 8 tiles with
//    nontemporal stores: FP64 full list at 345 MB 56.1 / 56.5 / 67.8, at 435 MB
//    71.8 / 84.9 / 85.5; shifted FP32 full list at 380 MB 58.8 / 59.1 / 68.8, at
//    433 MB 68.2 / 72.7 / 74.8; FP64 over 16-bit codes at 384 MB 69.4 / 76.2 /
//    71.0).  The limit of the full list is 512 MiB (FP64 at 522 MB 93.7 against
//    101.8 in runs of 8 with nontemporal stores, at 601 MB 109.2 against 106.1),
//    of 16-bit codes 384 MiB (FP64 at 436 MB 83.3 against 80.5, scaled FP16 at
//    448 MB 84.3 against 82.3 in runs of 8), and of 8-bit codes 256 MiB (against
//    runs of 8 with nontemporal stores, FP64 at 265 / 303 / 404 MB 43.0 / 62.6 /
//    80.1 and 49.2 / 59.7 / 72.5, shifted FP32 at 257 / 278 / 341 / 397 MB 41.9 /
//    55.5 / 70.0 / 84.4 and 48.4 / 51.6 / 62.8 / 74.4, scaled FP16 at 255 / 299 /
//    376 MB 45.8 / 66.5 / 84.8 and 53.2 / 63.3 / 77.4).
//    The forms that alternate take no hints either in calls of two sweeps and
//    more (the same storages over the list, over 16-bit codes and in place over
//    the list, 2 to 4 sizes each: one state, calls of 2 sweeps, 0.91 / 1.11 /
//    1.23; three states in turn, calls of 2 or of 8 and 20 sweeps, 0.81 / 0.96 /
//    1.08 and 0.89 / 1.08 / 1.24; what is below 0.91 are FP64 over 16-bit codes
//    at 343 MiB and in place at 395 MiB).
//  * beyond it, runs of as many tiles as the LBM_FLAG_XCD_CHUNK bits say, or,
//    without them, of 8 tiles: the XCDs sweep nearby parts of the list together
//    (DRAM pages) and are evenly loaded (FP64 full list, 7.5 M cells: 525 us
//    against 554 with an eighth each; shifted FP32 over codes, 3.6 M: 123
//    against 137).  Runs of 4 to 64 tiles are within 1 % of it.
//  * nontemporal stores with LBM_FLAG_NONTEMPORAL, and beyond that limit also
//    without it where they are faster nearly always: in FP64 (14 random boxes,
//    3 orderings, full list and 16-bit codes: -7 to +0.5 %, median -3.5 %) and
//    over 8-bit codes (narrower storages: -13 to 0 %, median -5 %).  Narrower
//    storages over the other forms go either way (-9 to +7 %).
//  * beyond that limit with plain stores, or over 8-bit codes, every other sweep
//    runs from the last tile to the first, too.  Same boxes: plain -11 to
//    +0.4 %, median -3.5 %; nontemporal over 8-bit codes -4 to +1 %, median -1 %
//    (shifted FP32 612 MB 113.4 -> 108.7 us, FP64 402 MB 77.4 -> 74.0);
//    nontemporal over the other forms -1 to +2 %, so those keep one direction.
constexpr size_t kCachedBytes = size_t(240) << 20;
constexpr int kResidentSweeps = 2;

struct SweepRule {
    size_t whole_runs;     // bytes up to which an XCD takes one run
    bool alternate_whole;  // up to there directions alternate, in calls of several
                           // sweeps whatever the hints
    bool nt;               // nontemporal stores beyond it also without the flag
    bool alternate_nt;     // directions alternate with nontemporal stores too
};

struct SweepLaunch {
    dim3 grid, block;
    XcdMap map;
    int policy;
    bool alternate;  // sweeps towards the lower of two arrays run backwards
    int32_t run;     // list tiles of a run; 0: one run per XCD
    uint32_t blocks;

    XcdMap towards(bool lower) const {
        XcdMap m = map;
        if (alternate && lower) {
            m.flip = ~0u;
            m.off = blocks;
        }
        return m;
    }
};

// n_steps: sweeps of the call; block: list cells per workgroup (a multiple of
// the 256-cell tile).
inline SweepLaunch sweep_launch(int32_t flags, int64_t n, size_t cell_bytes, const SweepRule& rule,
                                int n_steps, int block = kCodeTile) {
    const size_t bytes = size_t(n) * cell_bytes;
    const int64_t blocks = std::max<int64_t>(1, (n + block - 1) / block);
    const bool hinted = flags & (LBM_FLAG_NONTEMPORAL | LBM_FLAG_XCD_CHUNK_MASK);
    const bool resident = !hinted || n_steps >= kResidentSweeps;
    const bool cached = bytes <= kCachedBytes && resident;
    const bool large = bytes > rule.whole_runs;
    const bool whole = !cached && !large && rule.alternate_whole && resident;
    if (cached || whole) flags = 0;
    const int64_t given = (flags & LBM_FLAG_XCD_CHUNK_MASK) >> LBM_FLAG_XCD_CHUNK_SHIFT;
    SweepLaunch l;
    l.blocks = uint32_t(blocks);
    l.run = int32_t(given ? given : large ? 8 : 0);
    if (l.run == 0) {
        l.map = map_of_eighths(blocks);
    } else {
        const int64_t run = int64_t(l.run) * kCodeTile / block;
        int shift = 0;
        while ((int64_t(2) << shift) <= run) ++shift;
        l.map = map_of_runs(shift);
    }
    const bool nt = (flags & LBM_FLAG_NONTEMPORAL) || (large && rule.nt);
    l.policy = cached ? kCached : nt ? kStreamNT : kStream;
    l.alternate = large ? !nt || rule.alternate_nt : whole;
    l.grid = dim3(unsigned(virtual_blocks(blocks, l.map)));
    l.block = dim3(unsigned(block));
    return l;
}

// The two-array sweep of a storage form over the full list or 16- or 8-bit
// codes (code_bytes 4, 2, 1).
template <int ST>
inline SweepLaunch two_array_launch(int32_t flags, int64_t n, size_t code_bytes, int n_steps,
                                    int block = kCodeTile) {
    constexpr size_t T = sizeof(typename Storage<ST>::T);
    const size_t whole_runs = size_t(code_bytes == 4 ? 512 : code_bytes == 2 ? 384 : 256) << 20;
    const SweepRule rule = {whole_runs, true, T == 8 || code_bytes == 1, code_bytes == 1};
    return sweep_launch(flags, n, 2 * Q * T + (Q - 1) * code_bytes, rule, n_steps, block);
}

// The in-place sweep.  Nontemporal stores without the flag in FP64 and over
// 8-bit codes: the local step writes whole lines that it has just read (shifted
// FP32 12.7 / 30.6 M cells 405 / 999 us a sweep against 427 / 1,025 with plain
// stores, scaled FP16 232 / 598 against 248 / 616), the gather-scatter step does
// not mind.  With them both steps run forwards (backwards local steps cost 1 to
// 5 %).
//
// States somewhat larger than the last-level cache, without hints (us a sweep).
// Over 8-bit codes short runs as beyond it: one run per XCD is up to 4 % faster
// for one state of some geometries and up to 17 % slower for others and for
// states stepped in turn (runs of 8 / one run per XCD / plain stores and one run:
// FP64 all-fluid box at 299 MiB 91.4 / 104.8 / 109.7 and, six in turn, 110.4 /
// 128.7 / 116.8; FP64 packing at 308 MiB 101.7 / 107.1 / 117.1 and 116.4 / 130.9 /
// 125.1, at 345 MiB 119.5 / 111.1 / 128.4; shifted FP32 packing at 337 MiB 108.3 /
// 115.3 / 124.3; scaled FP16 packing at 294 MiB 100.9 / 96.7 / 136.7 and 107.3 /
// 107.3 / 140.9).  Over the list plain stores, one run per XCD and alternating
// directions up to 512 MiB (FP64 at 441 / 498 MB 117.1 / 132.0 against 125.9 /
// 141.2 in runs of 8 with nontemporal stores, shifted FP32 at 435 / 502 MB 88.4 /
// 100.7 against 93.2 / 105.9 in runs of 8).
template <int ST>
inline SweepLaunch inplace_launch(int32_t flags, int64_t n, size_t code_bytes, int n_steps) {
    constexpr size_t T = sizeof(typename Storage<ST>::T);
    const size_t whole_runs = size_t(code_bytes == 4 ? 512 : code_bytes == 2 ? 384 : 240) << 20;
    const SweepRule rule = {whole_runs, code_bytes == 4, T == 8 || code_bytes == 1, false};
    return sweep_launch(flags, n, Q * T + (Q - 1) * code_bytes, rule, n_steps);
}

// Calls f(std::integral_constant<int, policy>).
template <class F>
lbm_status with_policy(int policy, F&& f) {
    switch (policy) {
    case kCached: return f(std::integral_constant<int, kCached>{});
    case kStream: return f(std::integral_constant<int, kStream>{});
    default: return f(std::integral_constant<int, kStreamNT>{});
    }
}

}  // namespace lbm
