// moments.hip -- macroscopic fields and FP64 totals (lbm_moments).
//
// Per cell the gathered populations give rho and u = j + G/2 (always in
// FP64, whatever the storage).  Totals per segment are reduced in two fixed
// passes (per-workgroup partials, then one workgroup per segment over its
// partials) with double-double (TwoSum) accumulation, so they are reproducible
// bit for bit and accurate to about 1e-30 relative before the final rounding.
//
// The first pass is bound by its reads (19 populations and 18 adjacency
// entries per cell).  A workgroup takes as many consecutive tiles as leave
// about 8192 workgroups: each thread adds up its cells before the workgroup
// reduces, by wave shifts rather than a tree of barriers, and the second pass
// has few partials.  All segments that fit one argument block share the two
// launches.  us before -> now: totals of 33.9 M cells FP64 / shifted FP32 /
// scaled FP16 1,707 / 1,251 / 1,008 -> 1,392 / 936 / 680 (5.4 TB/s), with fields
// of 7.5 M / 0.95 / 0.41 M cells FP64 451 / 57.7 / 27.7 -> 396 / 52.6 / 24.3.
#include <algorithm>
#include <mutex>

#include "lbm_device.hpp"
#include "lbm_host.hpp"

namespace lbm {

constexpr int kMomBlock = 256;
constexpr int kRedThreads = 1024;
constexpr int kMomSegs = 64;            // segments of one launch
constexpr int64_t kMomParts = 8192;  // workgroups for all segments, about

struct DD {
    double hi, lo;
};

// Knuth's TwoSum, then renormalise: (a.hi + a.lo) + (b.hi + b.lo) in DD.
__device__ __forceinline__ DD dd_add(DD a, DD b) {
    const double s = a.hi + b.hi;
    const double bp = s - a.hi;
    double e = (a.hi - (s - bp)) + (b.hi - bp);
    e += a.lo + b.lo;
    const double hi = s + e;
    return DD{hi, e - (hi - s)};
}

// A value of another lane of the wave, by a pattern that names one for each.
template <int CTRL>
__device__ __forceinline__ DD lane_move(DD v) {
    DD r;
    const uint64_t h = __builtin_bit_cast(uint64_t, v.hi), l = __builtin_bit_cast(uint64_t, v.lo);
    const uint32_t w[4] = {
        uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(h)), CTRL, 0xf, 0xf, true)),
        uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(h >> 32)), CTRL, 0xf, 0xf, true)),
        uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(l)), CTRL, 0xf, 0xf, true)),
        uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(l >> 32)), CTRL, 0xf, 0xf, true))};
    r.hi = __builtin_bit_cast(double, uint64_t(w[1]) << 32 | w[0]);
    r.lo = __builtin_bit_cast(double, uint64_t(w[3]) << 32 | w[2]);
    return r;
}

// The quantity that a lane ends up with in block_reduce4.
__device__ __forceinline__ int quantity_of(int lane) { return (lane & 1) << 1 | ((lane >> 1) & 1); }

// Sum over the 4 lanes of a row of 16 that hold the same quantity, in each.
__device__ __forceinline__ DD row_sum(DD v) {
    v = dd_add(v, lane_move<0x128>(v));  // rotate by 8
    return dd_add(v, lane_move<0x124>(v));  // by 4
}

// Fixed-shape reduction of 4 DD values over a workgroup of WAVES waves.  Lanes
// share the work: a pair of lanes splits the four quantities, a pair of pairs
// splits them again, and each lane then sums one of them over its row of 16
// (5 additions instead of 16); the rows' sums meet in LDS, and the first wave
// adds them up.  Threads 0 to 3 return quantity_of(thread).
template <int WAVES>
__device__ __forceinline__ DD block_reduce4(const DD v[4]) {
    constexpr int kParts = 4 * WAVES;  // rows of 16 lanes
    __shared__ DD row_part[kParts][4];
    const int lane = int(threadIdx.x) & 63;
    const bool odd = lane & 1, upper = lane & 2;
    DD a = odd ? v[2] : v[0], b = odd ? v[3] : v[1];
    a = dd_add(a, lane_move<0xB1>(odd ? v[0] : v[2]));
    b = dd_add(b, lane_move<0xB1>(odd ? v[1] : v[3]));
    DD one = dd_add(upper ? b : a, lane_move<0x4E>(upper ? a : b));
    one = row_sum(one);
    if ((lane & 15) < 4) row_part[threadIdx.x >> 4][lane & 3] = one;
    __syncthreads();
    DD sum{0.0, 0.0};
    if (threadIdx.x < 64) {
        // lane 4 e + j: parts e, e + 16, ... of the quantity in place j
#pragma unroll
        for (int e = 0; e < kParts; e += 16) sum = dd_add(sum, row_part[e + (lane >> 2)][lane & 3]);
        sum = row_sum(sum);
        sum = dd_add(sum, DD{__shfl_xor(sum.hi, 16), __shfl_xor(sum.lo, 16)});
        sum = dd_add(sum, DD{__shfl_xor(sum.hi, 32), __shfl_xor(sum.lo, 32)});
    }
    return sum;
}

// One segment of a launch: its cells, its workgroups and half its force.
struct MomSeg {
    int64_t base, n;
    double half_g[3];
    int32_t first, blocks;
};

// The segments of a launch, up to SEGS of them; a launch of one segment is
// written without the 3 KB of arguments that many take.
template <int SEGS>
struct MomChunk {
    int32_t count;
    int32_t per_block;  // cells of a workgroup
    MomSeg s[SEGS];
};
static_assert(sizeof(MomChunk<kMomSegs>) < 3800, "fits the kernel arguments beside the pointers");

template <int ST, int SEGS, int POL>
__global__ __launch_bounds__(kMomBlock) void k_moments(const typename Storage<ST>::T* __restrict__ f,
                                                       const uint32_t* __restrict__ adj,
                                                       int64_t stride, double* __restrict__ rho,
                                                       double* __restrict__ u, int64_t ld,
                                                       double* __restrict__ partial,
                                                       MomChunk<SEGS> chunk) {
    const int32_t block = int32_t(blockIdx.x);
    int lo = 0, hi = chunk.count - 1;  // the segment of this workgroup
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (chunk.s[mid].first <= block)
            lo = mid;
        else
            hi = mid - 1;
    }
    const MomSeg& seg = chunk.s[lo];
    const double gx = seg.half_g[0], gy = seg.half_g[1], gz = seg.half_g[2];
    const int64_t begin = int64_t(block - seg.first) * chunk.per_block;
    const int64_t end = std::min<int64_t>(seg.n, begin + chunk.per_block);
    const int64_t base = seg.base;
    DD v[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    for (int64_t local = begin + threadIdx.x; local < end; local += kMomBlock) {
        const int64_t m = base + local;
        // the 18 adjacency rows first, then the 18 gathers: both batches in
        // flight at once
        uint32_t a[Q - 1];
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) a[k] = ld_stream<POL>(adj + k * stride + m);
        double g[Q];
        g[0] = static_cast<double>(f[m]);
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) g[k + 1] = static_cast<double>(f[a[k]]);
        const CellMoments<double> cm = cell_moments(g);
        const double r = Storage<ST>::shifted ? 1.0 + cm.rho : cm.rho;
        const double ux = cm.jx + gx, uy = cm.jy + gy, uz = cm.jz + gz;
        if (rho) rho[m] = r;
        if (u) {
            u[m] = ux;
            u[ld + m] = uy;
            u[2 * ld + m] = uz;
        }
        v[0] = dd_add(v[0], DD{r, 0.0});
        v[1] = dd_add(v[1], DD{ux, 0.0});
        v[2] = dd_add(v[2], DD{uy, 0.0});
        v[3] = dd_add(v[3], DD{uz, 0.0});
    }
    if (!partial) return;
    const DD sum = block_reduce4<kMomBlock / 64>(v);
    if (threadIdx.x < 4) {
        double* p = partial + (int64_t(block) * 4 + quantity_of(int(threadIdx.x))) * 2;
        p[0] = sum.hi;
        p[1] = sum.lo;
    }
}

// One workgroup per segment of the launch: totals (4 values) and/or the
// objective (the x total divided by the cell count).
template <int SEGS>
__global__ __launch_bounds__(kRedThreads) void k_reduce_partials(const double* __restrict__ partial,
                                                                 double* __restrict__ totals,
                                                                 double* __restrict__ objective,
                                                                 MomChunk<SEGS> chunk) {
    const MomSeg& seg = chunk.s[SEGS > 1 ? blockIdx.x : 0];
    DD v[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    // thread t sums partials t, t + T, t + 2T, ... in order
    for (int64_t b = threadIdx.x; b < seg.blocks; b += kRedThreads) {
        const double* p = partial + (seg.first + b) * 8;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = dd_add(v[q], DD{p[2 * q], p[2 * q + 1]});
    }
    const DD sum = block_reduce4<kRedThreads / 64>(v);
    if (threadIdx.x < 4) {
        const int q = quantity_of(int(threadIdx.x));
        const double total = sum.hi + sum.lo;
        if (totals) totals[4 * blockIdx.x + q] = total;
        if (objective && q == 1) objective[blockIdx.x] = total / double(seg.n);
    }
}

inline int64_t seg_tiles(int64_t n) { return std::max<int64_t>(1, (n + kMomBlock - 1) / kMomBlock); }

// Launches all segments; `parts` is the number of partials (64 bytes each) that
// `partial` holds, at least min(target, tiles) of the largest segment.
template <int ST, int SEGS>
lbm_status launch_segments(const lbm_params* p, int64_t n, int64_t stride, const uint32_t* adj,
                           const void* f, double* rho, double* u, const lbm_segment* seg,
                           int32_t n_seg, double* totals, double* objective, double* partial,
                           int64_t parts, int64_t target, hipStream_t s) {
    const bool reduce = totals || objective;
    int64_t all_tiles = 0;
    for (int32_t k = 0; k < n_seg; ++k) all_tiles += seg_tiles(seg[k].n);
    const int64_t per = (all_tiles + target - 1) / target;  // tiles of a workgroup
    // a state that fits the last-level cache with its list is read from there
    const bool cached = size_t(all_tiles) * kMomBlock *
                            (Q * sizeof(typename Storage<ST>::T) + (Q - 1) * sizeof(uint32_t)) <= kCachedBytes;
    for (int32_t k0 = 0; k0 < n_seg;) {
        MomChunk<SEGS> ch;
        ch.count = 0;
        ch.per_block = int32_t(per * kMomBlock);
        int64_t blocks = 0;
        int32_t k = k0;
        for (; k < n_seg && ch.count < SEGS; ++k) {
            const int64_t b = (seg_tiles(seg[k].n) + per - 1) / per;
            if (ch.count > 0 && reduce && blocks + b > parts) break;
            const lbm_params& pk = p[seg[k].param_index];
            MomSeg& t = ch.s[ch.count++];
            t.base = seg[k].base;
            t.n = seg[k].n;
            for (int d = 0; d < 3; ++d) t.half_g[d] = 0.5 * pk.force[d];
            t.first = int32_t(blocks);
            t.blocks = int32_t(b);
            blocks += b;
        }
        const auto kernel = cached ? k_moments<ST, SEGS, kCached> : k_moments<ST, SEGS, kStream>;
        kernel<<<dim3(unsigned(blocks)), dim3(kMomBlock), 0, s>>>(
            static_cast<const typename Storage<ST>::T*>(f), adj, stride, rho, u, n,
            reduce ? partial : nullptr, ch);
        if (hipGetLastError() != hipSuccess) return LBM_EHIP;
        if (reduce) {
            // launches run one after another on the stream, so they reuse the partials
            k_reduce_partials<SEGS><<<dim3(unsigned(ch.count)), dim3(kRedThreads), 0, s>>>(
                partial, totals ? totals + 4 * int64_t(k0) : nullptr,
                objective ? objective + k0 : nullptr, ch);
            if (hipGetLastError() != hipSuccess) return LBM_EHIP;
        }
        k0 = k;
    }
    return LBM_OK;
}

template <int ST>
lbm_status launch_moments(const lbm_params* p, int64_t n, int64_t stride, const uint32_t* adj,
                          const void* f, double* rho, double* u, const lbm_segment* seg,
                          int32_t n_seg, double* totals, double* objective, double* partial,
                          int64_t parts, int64_t target, hipStream_t s) {
    const lbm_segment whole{0, n, 0, 0};
    if (!seg || n_seg == 0) {
        seg = &whole;
        n_seg = 1;
    }
    return n_seg == 1 ? launch_segments<ST, 1>(p, n, stride, adj, f, rho, u, seg, 1, totals,
                                               objective, partial, parts, target, s)
                      : launch_segments<ST, kMomSegs>(p, n, stride, adj, f, rho, u, seg, n_seg, totals,
                                                      objective, partial, parts, target, s);
}

// Reads `count` totals back in fixed-size pieces (no allocation) after the
// stream has produced them: LBM_ENONFINITE if one is NaN or infinite.
lbm_status check_totals_finite(const double* totals, int64_t count, hipStream_t s) {
    double buf[64];
    bool finite = true;
    for (int64_t i0 = 0; i0 < count; i0 += 64) {
        const int64_t c = std::min<int64_t>(64, count - i0);
        LBM_TRY_HIP(hipMemcpyAsync(buf, totals + i0, size_t(c) * sizeof(double), hipMemcpyDeviceToHost, s));
        LBM_TRY_HIP(hipStreamSynchronize(s));
        for (int64_t i = 0; i < c; ++i) finite = finite && std::isfinite(buf[i]);
    }
    return finite ? LBM_OK : LBM_ENONFINITE;
}

constexpr size_t kPartBytes = 8 * sizeof(double);

inline size_t moments_bytes(int64_t tiles) {
    return align_up(size_t(std::min<int64_t>(tiles, kMomParts)) * kPartBytes, 256);
}

// Shared by lbm_moments and lbm_objective.
lbm_status moments_call(const lbm_params* p, int32_t n_params, int64_t n, int64_t stride,
                        const uint32_t* adj, const void* f, double* rho, double* u,
                        const lbm_segment* seg, int32_t n_seg, double* totals, double* objective,
                        void* workspace, size_t* ws_bytes, void* stream) {
    if (!p || n_params < 1 || n_params > kMaxParamSets) return LBM_EINVAL;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    if (!valid_segments(seg, n_seg, n, n_params)) return LBM_EINVAL;
    // needed: one partial for every tile of the largest segment (a launch of it
    // uses kMomParts at most); asked for: enough to launch all segments together
    const bool segs = seg && n_seg > 0;
    int64_t largest = segs ? 0 : n, all = segs ? 0 : seg_tiles(n);
    for (int32_t k = 0; segs && k < n_seg; ++k) {
        largest = std::max(largest, seg[k].n);
        all += seg_tiles(seg[k].n);
    }
    const bool reduce = totals || objective;
    const size_t need = reduce ? align_up(size_t(seg_tiles(largest)) * kPartBytes, 256) : 0;
    if (reduce && !workspace) {
        if (!ws_bytes) return LBM_EINVAL;
        *ws_bytes = std::max(need, moments_bytes(all) + (segs ? size_t(std::min<int32_t>(n_seg, kMomSegs)) * kPartBytes : 0));
        return LBM_OK;
    }
    if (reduce && (!ws_bytes || *ws_bytes < need)) return LBM_EWORKSPACE;
    if (!adj || !f) return LBM_EINVAL;
    for (int32_t k = 0; k < n_params; ++k) {
        if (!valid_storage(p[k].storage) || p[k].storage != p[0].storage) return LBM_EINVAL;
        for (int d = 0; d < 3; ++d)
            if (!std::isfinite(p[k].force[d])) return LBM_EINVAL;
    }
    hipStream_t s = as_stream(stream);
    double* partial = static_cast<double*>(workspace);
    const int64_t parts = reduce ? int64_t(*ws_bytes / kPartBytes) : 0;
    lbm_status st;
    switch (p[0].storage) {
    case LBM_F64: st = launch_moments<LBM_F64>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, objective, partial, parts, kMomParts, s); break;
    case LBM_F64_SHIFTED: st = launch_moments<LBM_F64_SHIFTED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, objective, partial, parts, kMomParts, s); break;
    case LBM_F32: st = launch_moments<LBM_F32>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, objective, partial, parts, kMomParts, s); break;
    case LBM_F32_SHIFTED: st = launch_moments<LBM_F32_SHIFTED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, objective, partial, parts, kMomParts, s); break;
    case LBM_F16_SHIFTED: st = launch_moments<LBM_F16_SHIFTED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, objective, partial, parts, kMomParts, s); break;
    case LBM_F16_SHIFTED_SCALED: st = launch_moments<LBM_F16_SHIFTED_SCALED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, objective, partial, parts, kMomParts, s); break;
    default: return LBM_EINVAL;
    }
    if (st != LBM_OK || !totals || !(p[0].flags & LBM_FLAG_CHECK_FINITE)) return st;
    return check_totals_finite(totals, 4 * int64_t(std::max<int32_t>(n_seg, 1)), s);
}

// ---------------------------------------------------------------------------
// lbm_moments_noalloc: the partial sums of the totals live in `scratch`, a
// fixed device array of the library (one copy per GPU, held until the
// process ends), instead of a caller workspace.  Host code never passes the
// array's name to a kernel: it takes the device address from
// hipGetSymbolAddress once per device, with that device current, and uses it.
// ---------------------------------------------------------------------------
constexpr int64_t kNoAllocParts = 4096;  // partial sums, 4 double-doubles each
constexpr int kMaxDevices = 64;
static __device__ __align__(256) double scratch[kNoAllocParts * 8];  // 256 KiB

std::mutex g_scratch_mutex;
double* g_scratch_ptr[kMaxDevices] = {};

// Address of the current device's scratch (looked up on the first call on it).
lbm_status device_scratch(double** out) {
    int dev = -1;
    LBM_TRY_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return LBM_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LBM_EHIP;
        g_scratch_ptr[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return LBM_OK;
}

}  // namespace lbm

using namespace lbm;

extern "C" lbm_status lbm_moments(const lbm_params* p, int32_t n_params, int64_t n,
                                  int64_t stride, const uint32_t* adj, const void* f, double* rho,
                                  double* u, const lbm_segment* seg, int32_t n_seg, double* totals,
                                  void* workspace, size_t* ws_bytes, void* stream) {
    return moments_call(p, n_params, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr,
                        workspace, ws_bytes, stream);
}

extern "C" lbm_status lbm_objective(const lbm_params* p, int32_t n_params, int64_t n,
                                    int64_t stride, const uint32_t* adj, const void* f,
                                    const lbm_segment* seg, int32_t n_seg, double* J,
                                    void* workspace, size_t* ws_bytes, void* stream) {
    if (!J) return LBM_EINVAL;
    return moments_call(p, n_params, n, stride, adj, f, nullptr, nullptr, seg, n_seg, nullptr, J,
                        workspace, ws_bytes, stream);
}

extern "C" lbm_status lbm_moments_noalloc(const lbm_params* p, int32_t n_params, int64_t n,
                                          int64_t stride, const uint32_t* adj, const void* f,
                                          double* rho, double* u, const lbm_segment* seg,
                                          int32_t n_seg, double* totals, void* stream) {
    if (!p || n_params < 1 || n_params > kMaxParamSets || !adj || !f) return LBM_EINVAL;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    if (!valid_segments(seg, n_seg, n, n_params)) return LBM_EINVAL;
    for (int32_t k = 0; k < n_params; ++k) {
        if (!valid_storage(p[k].storage) || p[k].storage != p[0].storage) return LBM_EINVAL;
        for (int d = 0; d < 3; ++d)
            if (!std::isfinite(p[k].force[d])) return LBM_EINVAL;
    }
    double* partial = nullptr;
    if (totals) {
        if (lbm_status st = device_scratch(&partial); st != LBM_OK) return st;
    }
    hipStream_t s = as_stream(stream);
    lbm_status st;
    switch (p[0].storage) {
    case LBM_F64: st = launch_moments<LBM_F64>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr, partial, kNoAllocParts, kNoAllocParts, s); break;
    case LBM_F64_SHIFTED: st = launch_moments<LBM_F64_SHIFTED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr, partial, kNoAllocParts, kNoAllocParts, s); break;
    case LBM_F32: st = launch_moments<LBM_F32>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr, partial, kNoAllocParts, kNoAllocParts, s); break;
    case LBM_F32_SHIFTED: st = launch_moments<LBM_F32_SHIFTED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr, partial, kNoAllocParts, kNoAllocParts, s); break;
    case LBM_F16_SHIFTED: st = launch_moments<LBM_F16_SHIFTED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr, partial, kNoAllocParts, kNoAllocParts, s); break;
    case LBM_F16_SHIFTED_SCALED: st = launch_moments<LBM_F16_SHIFTED_SCALED>(p, n, stride, adj, f, rho, u, seg, n_seg, totals, nullptr, partial, kNoAllocParts, kNoAllocParts, s); break;
    default: return LBM_EINVAL;
    }
    if (st != LBM_OK || !totals || !(p[0].flags & LBM_FLAG_CHECK_FINITE)) return st;
    return check_totals_finite(totals, 4 * int64_t(std::max<int32_t>(n_seg, 1)), s);
}
