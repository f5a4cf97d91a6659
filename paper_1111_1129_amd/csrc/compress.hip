// compress.hip -- 16-bit and 8-bit adjacency codes and the sweeps that read
// them (lbm_compress_adjacency, lbm_step_c16, lbm_narrow_codes, lbm_step_c8).
//
// The adjacency list is 72 of the 376 bytes a FP64 cell update moves (49 %
// of the 148 bytes in shifted FP16).  In a locality-preserving ordering the
// 256 cells of a tile pull a given direction from a nearby run of cells, so
// each entry is stored as
//   code  = src - m - toff[tile][k]   (-32766..32767) for a streaming entry,
//   code  = BOUNCE (-32768)           for the implicit bounce-back,
//   code  = ESCAPE (-32767)           if the difference does not fit,
// with one int32 offset toff per tile and direction (the midpoint of the
// tile's smallest and largest src - m).  A tile record holds the 18 offsets,
// the number of escapes in the tile and a flag word, 0 until lbm_narrow_codes
// sets it (80 bytes, two scalar loads).  The sweep rebuilds the exact slot i*stride + src from the codes
// (bounce-back: opp(i)*stride + m) in a tile without escapes, and reads the
// full list in a tile with any: the choice is uniform over the workgroup, so
// neither path branches per lane and every gather of a cell is in flight at
// once.  Results are bit-identical to the uncompressed sweep; the adjacency
// traffic of an escape-free tile drops from 72 to 36.3 bytes per cell.
//
// 8-bit codes (lbm_narrow_codes, lbm_step_c8): in a tile whose 16-bit codes
// all lie in -127..127 or are bounce-backs (most tiles of a lexicographic
// order: the offsets of a tile spread over little more than the fluid count
// of one row) the same codes fit one byte each, with -128 for bounce-back.
// Word 19 of the tile record marks such a tile; the sweep then reads 18 bytes
// of codes per cell instead of 36, and the other tiles as before.
#include <algorithm>
#include <type_traits>

#include "lbm_device.hpp"
#include "lbm_host.hpp"

namespace lbm {

constexpr int kCTile = kCodeTile;  // cells per tile = workgroup size of the sweep
constexpr int kRec = kCodeRec;

// Smallest / largest of a value over the wave, uniform.
__device__ __forceinline__ int32_t wave_max(int32_t v) {
#define LBM_DPP_MAX(ctrl) v = max(v, __builtin_amdgcn_update_dpp(v, v, ctrl, 0xf, 0xf, false))
    LBM_DPP_MAX(0xB1);   // exchange neighbours, pairs, halves of 8, halves of a row of 16
    LBM_DPP_MAX(0x4E);
    LBM_DPP_MAX(0x141);
    LBM_DPP_MAX(0x140);
    LBM_DPP_MAX(0x142);  // lane 15 of a row to the next row, lane 31 to the upper half
    LBM_DPP_MAX(0x143);
#undef LBM_DPP_MAX
    return __builtin_amdgcn_readlane(v, 63);
}

// Four consecutive elements of a row at p: one access with VEC, else four.
template <bool VEC, class T>
__device__ __forceinline__ void load4(const T* p, T* v) {
    typedef T V4 __attribute__((ext_vector_type(4)));
    if constexpr (VEC) {
        const V4 q = *reinterpret_cast<const V4*>(p);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = q[j];
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = p[j];
    }
}

// ... the first `live` of them stored
template <bool VEC, class T>
__device__ __forceinline__ void store4(T* p, const T* v, int live) {
    typedef T V4 __attribute__((ext_vector_type(4)));
    if (VEC && live == 4) {
        *reinterpret_cast<V4*>(p) = V4{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < live) p[j] = v[j];
    }
}

// The code kernels take one wave per tile and four consecutive cells per lane.
// They stream whole rows, and what bounds them is the number of memory
// instructions: with one cell per lane a wave moved 64 to 256 bytes with each.
// 30.6 M cells, one cell per lane -> four: k_compress (108 bytes per cell) 793
// -> 616 us, 5.3 TB/s, its tile minima by wave shifts instead of through LDS;
// k_narrow (54 bytes) 317 -> 306 us.  4.8 M cells: 158 -> 111, 52 -> 48 us.
// VEC: rows start on a multiple of four elements of an aligned array.
struct LaneCells {
    int64_t m;  // first cell; lanes past the list take cells 0.. and are ignored
    int live;   // cells of this lane in the list
};

__device__ __forceinline__ LaneCells lane_cells(int64_t tile, int lane, int64_t n) {
    const int64_t m = tile * kCTile + 4 * lane;
    return LaneCells{m < n ? m : 0, int(m < n ? (n - m < 4 ? n - m : 4) : 0)};
}

constexpr int kCodeBlock = 256;  // 4 waves, 4 tiles

inline bool rows_of_4(int64_t stride, const void* p, size_t element) {
    return stride % 4 == 0 && reinterpret_cast<uintptr_t>(p) % (4 * element) == 0;
}

__device__ __forceinline__ int64_t wave_tile() {
    return int64_t(blockIdx.x) * (kCodeBlock / 64) +
           __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
}

template <bool VEC>
__global__ __launch_bounds__(kCodeBlock) void k_compress(const uint32_t* __restrict__ adj, int64_t n,
                                                         int64_t stride, int64_t tiles,
                                                         int16_t* __restrict__ codes,
                                                         int32_t* __restrict__ rec) {
    const int64_t tile = wave_tile();
    if (tile >= tiles) return;
    const int lane = int(threadIdx.x) & 63;
    const LaneCells c = lane_cells(tile, lane, n);
    uint32_t slot[Q - 1][4];
    if (VEC || c.live == 4) {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) load4<VEC>(adj + k * stride + c.m, slot[k]);
    } else {
        // the list's last cells: not past the end of the last row
#pragma unroll
        for (int k = 0; k < Q - 1; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) slot[k][j] = adj[k * stride + (j < c.live ? c.m + j : 0)];
    }
    const uint32_t S = uint32_t(stride);
    int32_t word = 0;  // of the tile record, lanes 0 to 19
    uint32_t esc = 0;
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        // streaming entries lie in row k + 1: offset from the cell itself, the
        // tile's smallest and largest, their midpoint (0 if nothing streams)
        int32_t d[4], lo = INT32_MAX, hi = INT32_MIN;
        bool st[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t col = slot[k][j] - uint32_t(k + 1) * S;
            st[j] = j < c.live && col < S;
            d[j] = int32_t(col - uint32_t(c.m + j));
            lo = st[j] ? min(lo, d[j]) : lo;
            hi = st[j] ? max(hi, d[j]) : hi;
        }
        hi = wave_max(hi);
        lo = ~wave_max(~lo);
        const int32_t base = lo <= hi ? lo + int32_t((uint32_t(hi) - uint32_t(lo)) / 2) : 0;
        word = lane == k ? base : word;
        int16_t code[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t r = d[j] - base;  // |d|, |base| < stride < 2^28
            const bool fits = r >= kCodeMin && r <= kCodeMax;
            code[j] = !st[j] ? kCodeBounce : fits ? int16_t(r) : kCodeEscape;
            esc += st[j] && !fits ? 1u : 0u;
        }
        store4<VEC>(codes + k * stride + c.m, code, c.live);
    }
    for (int off = 32; off > 0; off >>= 1) esc += __shfl_xor(esc, off);
    word = lane == Q - 1 ? int32_t(esc) : word;
    if (lane < kRec) rec[tile * kRec + lane] = word;
}

// Sum of one word over all tile records in two passes: up to kSumParts
// workgroups each total a strided share of the tiles, then one workgroup adds
// the partial sums (the per-tile counts are totalled here rather than by a
// global atomic per tile, which the 8 XCDs would serialise on one address).
constexpr int kSumBlock = 256;
constexpr int kSumParts = 256;
constexpr size_t kSumWorkspace = (kSumParts + 1) * sizeof(unsigned long long);

__device__ __forceinline__ unsigned long long block_sum(unsigned long long v) {
    __shared__ unsigned long long part[kSumBlock / 64];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = v;
    __syncthreads();
    unsigned long long total = 0;
    for (int w = 0; w < kSumBlock / 64; ++w) total += part[w];
    return total;
}

__global__ __launch_bounds__(kSumBlock) void k_sum_records(const int32_t* __restrict__ rec,
                                                           int64_t tiles, int word,
                                                           unsigned long long* __restrict__ parts) {
    unsigned long long s = 0;
    const int64_t step = int64_t(gridDim.x) * kSumBlock;
    for (int64_t t = int64_t(blockIdx.x) * kSumBlock + threadIdx.x; t < tiles; t += step)
        s += uint32_t(rec[t * kRec + word]);
    const unsigned long long total = block_sum(s);
    if (threadIdx.x == 0) parts[blockIdx.x] = total;
}

__global__ __launch_bounds__(kSumBlock) void k_sum_parts(const unsigned long long* __restrict__ parts,
                                                         int n_parts,
                                                         unsigned long long* __restrict__ out) {
    const unsigned long long total = block_sum(threadIdx.x < n_parts ? parts[threadIdx.x] : 0ull);
    if (threadIdx.x == 0) *out = total;
}

// Launches the two passes; the total lands in ws[kSumParts].
lbm_status sum_records(const int32_t* rec, int64_t tiles, int word, unsigned long long* ws,
                       hipStream_t s) {
    const int parts = int(std::min<int64_t>(kSumParts, (tiles + kSumBlock - 1) / kSumBlock));
    k_sum_records<<<parts, kSumBlock, 0, s>>>(rec, tiles, word, ws);
    if (hipGetLastError() != hipSuccess) return LBM_EHIP;
    k_sum_parts<<<1, kSumBlock, 0, s>>>(ws, parts, ws + kSumParts);
    return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EHIP;
}

// The tile is narrow if every live cell's 18 codes fit (a tile with escapes
// never does).  Codes of a wide tile are stored as 0.
template <bool VEC>
__global__ __launch_bounds__(kCodeBlock) void k_narrow(const int16_t* __restrict__ codes, int64_t n,
                                                       int64_t stride, int64_t tiles,
                                                       int32_t* __restrict__ rec,
                                                       int8_t* __restrict__ codes8) {
    const int64_t tile = wave_tile();
    if (tile >= tiles) return;
    const int lane = int(threadIdx.x) & 63;
    const LaneCells c = lane_cells(tile, lane, n);
    int16_t cd[Q - 1][4];
    if (VEC || c.live == 4) {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) load4<VEC>(codes + k * stride + c.m, cd[k]);
    } else {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) cd[k][j] = codes[k * stride + (j < c.live ? c.m + j : 0)];
    }
    bool fits = true;
#pragma unroll
    for (int k = 0; k < Q - 1; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t v = cd[k][j];
            fits = fits && (j >= c.live || v == kCodeBounce || (v >= -kCode8Max && v <= kCode8Max));
        }
    const bool narrow = __all(fits);
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        int8_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[j] = !narrow ? int8_t(0) : cd[k][j] == kCodeBounce ? kCode8Bounce : int8_t(cd[k][j]);
        store4<VEC>(codes8 + k * stride + c.m, v, c.live);
    }
    if (lane == 0) rec[tile * kRec + Q] = narrow ? 1 : 0;
}

template <int ST, bool PBB, int POL>
__global__ __launch_bounds__(kCTile) void k_trt_c16(const typename Storage<ST>::T* __restrict__ src,
                                                    typename Storage<ST>::T* __restrict__ dst,
                                                    const int16_t* __restrict__ codes,
                                                    const int32_t* __restrict__ tile_rec,
                                                    const uint32_t* __restrict__ adj,
                                                    const double* __restrict__ ns, int64_t n,
                                                    int64_t stride, TrtConst c, XcdMap map) {
    const int64_t tile = logical_block(map);
    const int64_t m = tile * kCTile + threadIdx.x;
    if (m >= n) return;
    const int32_t* rec = tile_rec + tile * kRec;  // uniform over the workgroup
    if (rec[Q - 1] != 0)
        update_cell<ST, PBB, POL>(src, dst, adj, ns, m, stride, c);
    else
        update_cell_coded<ST, PBB, POL, int16_t>(src, dst, codes, rec, ns, m, stride, c);
}

// Three-way, uniform over the workgroup: narrow tile -> 8-bit codes, tile
// with escapes -> full list, otherwise 16-bit codes.
template <int ST, bool PBB, int POL>
__global__ __launch_bounds__(kCTile) void k_trt_c8(const typename Storage<ST>::T* __restrict__ src,
                                                   typename Storage<ST>::T* __restrict__ dst,
                                                   const int8_t* __restrict__ codes8,
                                                   const int16_t* __restrict__ codes,
                                                   const int32_t* __restrict__ tile_rec,
                                                   const uint32_t* __restrict__ adj,
                                                   const double* __restrict__ ns, int64_t n,
                                                   int64_t stride, TrtConst c, XcdMap map) {
    const int64_t tile = logical_block(map);
    const int64_t m = tile * kCTile + threadIdx.x;
    if (m >= n) return;
    const int32_t* rec = tile_rec + tile * kRec;
    if (rec[Q] != 0)
        update_cell_coded<ST, PBB, POL, int8_t>(src, dst, codes8, rec, ns, m, stride, c);
    else if (rec[Q - 1] != 0)
        update_cell<ST, PBB, POL>(src, dst, adj, ns, m, stride, c);
    else
        update_cell_coded<ST, PBB, POL, int16_t>(src, dst, codes, rec, ns, m, stride, c);
}

// codes8 == nullptr: the 16-bit sweep (k_trt_c16); else the 8-bit one.
template <int ST, bool PBB>
lbm_status launch_coded(const lbm_params& p, int64_t n, int64_t stride, const int8_t* codes8,
                        const int16_t* codes, const int32_t* toff, const uint32_t* adj,
                        const double* ns, void* fa, void* fb, int n_steps, hipStream_t s) {
    using T = typename Storage<ST>::T;
    T* a = static_cast<T*>(fa);
    T* b = static_cast<T*>(fb);
    const TrtConst c = make_trt_const(p);
    const SweepLaunch l = two_array_launch<ST>(p.flags, n, codes8 ? 1 : 2, n_steps);
    return with_policy(l.policy, [&](auto pol) -> lbm_status {
        const auto steps = [&](auto&& sweep) -> lbm_status {
            for (int k = 0; k < n_steps; ++k) {
                const T* src = (k & 1) ? b : a;
                T* dst = (k & 1) ? a : b;
                if (lbm_status st = sweep(src, dst, l.towards(dst < src)); st != LBM_OK) return st;
            }
            return LBM_OK;
        };
        if (codes8) {
            const BoundKernel kernel(k_trt_c8<ST, PBB, pol>, l.grid, l.block, s);
            return steps([&](const T* src, T* dst, XcdMap map) {
                return kernel(src, dst, codes8, codes, toff, adj, ns, n, stride, c, map);
            });
        }
        const BoundKernel kernel(k_trt_c16<ST, PBB, pol>, l.grid, l.block, s);
        return steps([&](const T* src, T* dst, XcdMap map) {
            return kernel(src, dst, codes, toff, adj, ns, n, stride, c, map);
        });
    });
}

template <int ST>
lbm_status dispatch_coded(const lbm_params& p, int64_t n, int64_t stride, const int8_t* codes8,
                          const int16_t* codes, const int32_t* toff, const uint32_t* adj,
                          const double* ns, void* fa, void* fb, int n_steps, hipStream_t s) {
    return ns ? launch_coded<ST, true>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s)
              : launch_coded<ST, false>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
}

lbm_status step_coded(const lbm_params& p, int64_t n, int64_t stride, const int8_t* codes8,
                      const int16_t* codes, const int32_t* toff, const uint32_t* adj,
                      const double* ns, void* fa, void* fb, int n_steps, hipStream_t s) {
    switch (p.storage) {
    case LBM_F64: return dispatch_coded<LBM_F64>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
    case LBM_F64_SHIFTED: return dispatch_coded<LBM_F64_SHIFTED>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
    case LBM_F32: return dispatch_coded<LBM_F32>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
    case LBM_F32_SHIFTED: return dispatch_coded<LBM_F32_SHIFTED>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
    case LBM_F16_SHIFTED: return dispatch_coded<LBM_F16_SHIFTED>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
    case LBM_F16_SHIFTED_SCALED: return dispatch_coded<LBM_F16_SHIFTED_SCALED>(p, n, stride, codes8, codes, toff, adj, ns, fa, fb, n_steps, s);
    default: return LBM_EINVAL;
    }
}

}  // namespace lbm

using namespace lbm;

extern "C" lbm_status lbm_compress_adjacency(int64_t n, int64_t stride, const uint32_t* adj,
                                             int16_t* codes, int32_t* tile_records,
                                             int64_t* n_escapes, void* workspace,
                                             size_t* ws_bytes, void* stream) {
    if (!ws_bytes) return LBM_EINVAL;
    if (!workspace) {
        *ws_bytes = kSumWorkspace;
        return LBM_OK;
    }
    if (*ws_bytes < kSumWorkspace) return LBM_EWORKSPACE;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    if (!adj || !codes || !tile_records || !n_escapes || n <= 0) return LBM_EINVAL;
    hipStream_t s = as_stream(stream);
    auto* ws = static_cast<unsigned long long*>(workspace);
    const int64_t tiles = (n + kCTile - 1) / kCTile;
    const unsigned grid = unsigned((tiles + kCodeBlock / 64 - 1) / (kCodeBlock / 64));
    if (rows_of_4(stride, adj, sizeof(*adj)) && rows_of_4(stride, codes, sizeof(*codes)))
        k_compress<true><<<grid, kCodeBlock, 0, s>>>(adj, n, stride, tiles, codes, tile_records);
    else
        k_compress<false><<<grid, kCodeBlock, 0, s>>>(adj, n, stride, tiles, codes, tile_records);
    if (hipGetLastError() != hipSuccess) return LBM_EHIP;
    if (lbm_status st = sum_records(tile_records, tiles, Q - 1, ws, s); st != LBM_OK) return st;
    unsigned long long e = 0;
    LBM_TRY_HIP(hipMemcpyAsync(&e, ws + kSumParts, sizeof(e), hipMemcpyDeviceToHost, s));
    LBM_TRY_HIP(hipStreamSynchronize(s));
    *n_escapes = int64_t(e);
    return LBM_OK;
}

extern "C" lbm_status lbm_step_c16(const lbm_params* p, int64_t n, int64_t stride,
                                   const int16_t* codes, const int32_t* tile_records,
                                   const uint32_t* adj, const double* ns, void* f_a, void* f_b,
                                   int32_t n_steps, void* stream) {
    if (!valid_params(p) || !codes || !tile_records || !adj || !f_a || !f_b || n_steps < 0)
        return LBM_EINVAL;
    if (f_a == f_b) return LBM_EINVAL;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    if (n == 0 || n_steps == 0) return LBM_OK;
    return step_coded(*p, n, stride, nullptr, codes, tile_records, adj, ns, f_a, f_b, n_steps,
                      as_stream(stream));
}

extern "C" lbm_status lbm_narrow_codes(int64_t n, int64_t stride, const int16_t* codes,
                                       int32_t* tile_records, int8_t* codes8,
                                       int64_t* n_narrow_tiles, void* workspace,
                                       size_t* ws_bytes, void* stream) {
    if (!ws_bytes) return LBM_EINVAL;
    if (!workspace) {
        *ws_bytes = kSumWorkspace;
        return LBM_OK;
    }
    if (*ws_bytes < kSumWorkspace) return LBM_EWORKSPACE;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    if (!codes || !tile_records || !codes8 || !n_narrow_tiles || n <= 0) return LBM_EINVAL;
    hipStream_t s = as_stream(stream);
    auto* ws = static_cast<unsigned long long*>(workspace);
    const int64_t tiles = (n + kCTile - 1) / kCTile;
    const unsigned grid = unsigned((tiles + kCodeBlock / 64 - 1) / (kCodeBlock / 64));
    if (rows_of_4(stride, codes, sizeof(*codes)) && rows_of_4(stride, codes8, sizeof(*codes8)))
        k_narrow<true><<<grid, kCodeBlock, 0, s>>>(codes, n, stride, tiles, tile_records, codes8);
    else
        k_narrow<false><<<grid, kCodeBlock, 0, s>>>(codes, n, stride, tiles, tile_records, codes8);
    if (hipGetLastError() != hipSuccess) return LBM_EHIP;
    if (lbm_status st = sum_records(tile_records, tiles, Q, ws, s); st != LBM_OK) return st;
    unsigned long long t = 0;
    LBM_TRY_HIP(hipMemcpyAsync(&t, ws + kSumParts, sizeof(t), hipMemcpyDeviceToHost, s));
    LBM_TRY_HIP(hipStreamSynchronize(s));
    *n_narrow_tiles = int64_t(t);
    return LBM_OK;
}

extern "C" lbm_status lbm_step_c8(const lbm_params* p, int64_t n, int64_t stride,
                                  const int8_t* codes8, const int16_t* codes,
                                  const int32_t* tile_records, const uint32_t* adj,
                                  const double* ns, void* f_a, void* f_b, int32_t n_steps,
                                  void* stream) {
    if (!valid_params(p) || !codes8 || !codes || !tile_records || !adj || !f_a || !f_b ||
        n_steps < 0)
        return LBM_EINVAL;
    if (f_a == f_b) return LBM_EINVAL;
    if (lbm_status st = check_layout(n, stride); st != LBM_OK) return st;
    if (n == 0 || n_steps == 0) return LBM_OK;
    return step_coded(*p, n, stride, codes8, codes, tile_records, adj, ns, f_a, f_b, n_steps,
                      as_stream(stream));
}
