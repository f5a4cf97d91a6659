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

// The code kernels take one wave per tile and four consecutive cells per lane:
// they stream whole rows, and with one cell per lane a wave moves 64 to 256
// bytes with each memory instruction.  Rows may begin anywhere (a row stride or
// an array of the caller's): the accesses ask for an element's alignment only.
// Small lists give a SIMD one wave or none, which then waits for its own
// instructions, so these are few and without branches: values that neither the
// largest nor the smallest sees instead of conditions, 16-bit pairs in one
// operation, and reductions in which four directions share the lanes.
// us over random boxes of 2.4 k / 0.53 M / 10 M / 34 M cells: k_compress (108
// bytes per cell) 5.3 / 12.6 / 199 / 668 against 6.9 / 21.6 / 250 / 835 with one
// cell per lane, and 5.3 / 13.2 / 226 / 761 against 7.1 / 21.5 / 257 / 842 where
// rows begin off their vectors; k_narrow (54 bytes) 4.0 / 7.3 / 96 / 315 against
// 3.2 / 7.8 / 96 / 332, off their vectors 3.8 / 7.8 / 112 / 374 against 3.4 / 8.4 /
// 127 / 442.
constexpr int kCodeBlock = 256;  // 4 waves, 4 tiles

// LDS that a launch asks for and nothing uses: it holds lists that the caches
// cannot hold to two workgroups per CU.  Five to seven spread the rows that are
// read and written together over more places of the memory (k_compress / k_narrow
// with two and with all that fit: 30.6 M cells of a packing 639 / 299 and 658 /
// 327 us, 10 M of a random box 199 / 96 and 206 / 103; but 4.2 M 89 / 45.5 and
// 90 / 44.4, 1.3 M 23.8 / 13.8 and 23.4 / 12.5).
constexpr int64_t kCodeStreamCells = int64_t(8) << 20;
inline unsigned code_lds(int64_t n) { return n > kCodeStreamCells ? 64u << 10 : 0u; }

typedef int16_t Pair __attribute__((ext_vector_type(2)));

// Four elements, and the same at any element's address.
template <class T> struct Four {
    typedef T V __attribute__((ext_vector_type(4)));
    typedef V Any __attribute__((aligned(alignof(T))));
};
using Slots4 = Four<uint32_t>::V;
using Codes4 = Four<int16_t>::V;
using Bytes4 = Four<int8_t>::V;

// The four cells of a lane.
struct LaneCells {
    int64_t m;    // first cell
    int64_t n;    // cells of the list
    bool whole;   // the tile's 256 cells are all in the list (uniform)
    __device__ __forceinline__ LaneCells(int64_t tile, int lane, int64_t cells)
        : m(tile * kCTile + 4 * lane), n(cells), whole((tile + 1) * kCTile <= cells) {}
};

__device__ __forceinline__ int64_t wave_tile() {
    return int64_t(blockIdx.x) * (kCodeBlock / 64) +
           __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
}

// Four consecutive entries of every row of [18][stride] at a lane's cells;
// `none` in place of cells past the list (which read cell 0: no branches
// between the loads of the last tile, which a list of a few tiles waits for).
template <class T>
__device__ __forceinline__ void load_rows(const T* __restrict__ rows, int64_t stride, LaneCells c, T none,
                                          typename Four<T>::V* v) {
    if (c.whole) {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k)
            v[k] = *reinterpret_cast<const typename Four<T>::Any*>(rows + k * stride + c.m);
    } else {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool live = c.m + j < c.n;
                const T x = rows[k * stride + (live ? c.m + j : 0)];
                v[k][j] = live ? x : none;
            }
    }
}

template <class T>
__device__ __forceinline__ void store_rows(T* __restrict__ rows, int64_t stride, LaneCells c,
                                           const typename Four<T>::V* v) {
    if (c.whole) {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k)
            *reinterpret_cast<typename Four<T>::Any*>(rows + k * stride + c.m) = v[k];
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (c.m + j < c.n) {
#pragma unroll
                for (int k = 0; k < Q - 1; ++k) rows[k * stride + c.m + j] = v[k][j];
            }
    }
}

template <int CTRL>
__device__ __forceinline__ uint32_t row_lane(uint32_t x) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), CTRL, 0xf, 0xf, true));
}

// Reduction of four values over the wave at once: the 16 lanes of row q return
// that of v[q].
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce4(const uint32_t* v, Op op) {
    const auto halves = [&](uint32_t a, uint32_t b) {  // lower half: a, upper half: b
        const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        return op(s[0], s[1]);
    };
    const auto s = __builtin_amdgcn_permlane16_swap(halves(v[0], v[2]), halves(v[1], v[3]), false, false);
    uint32_t r = op(s[0], s[1]);
    // exchange neighbours, pairs, halves of 8, halves of the row
    r = op(r, row_lane<0xB1>(r));
    r = op(r, row_lane<0x4E>(r));
    r = op(r, row_lane<0x141>(r));
    return op(r, row_lane<0x140>(r));
}

__global__ __launch_bounds__(kCodeBlock) void k_compress(const uint32_t* __restrict__ adj, int64_t n,
                                                         int64_t stride, int64_t tiles,
                                                         int16_t* __restrict__ codes,
                                                         int32_t* __restrict__ rec) {
    const int64_t tile = wave_tile();
    if (tile >= tiles) return;
    const int lane = int(threadIdx.x) & 63;
    const LaneCells c(tile, lane, n);
    const uint32_t S = uint32_t(stride);
    // An entry that streams (it lies in row k + 1) is kept as its offset from the
    // cell plus kZero, between 0 and 2^29 since strides are below 2^28; any
    // other as kNone, which is below those as a signed and above them as an
    // unsigned number.  A slot past the list lies in no row.
    constexpr uint32_t kZero = 1u << 28, kNone = 1u << 31;
    constexpr int kGroups = (Q - 1 + 3) / 4;
    Slots4 e[Q - 1];
    load_rows(adj, stride, c, ~0u, e);
    // per direction the midpoint of the tile's smallest and largest offset (0 if
    // nothing streams); lanes 16 q + g hold that of direction 4 g + q
    uint32_t base[kGroups], word = 0;
    bool wide = false;  // an offset of the tile may not fit its code
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 4 * g + q;
            hi[q] = lo[q] = kNone;
#pragma unroll
            for (int j = 0; j < 4 && k < Q - 1; ++j) {
                const uint32_t col = e[k][j] - uint32_t(k + 1) * S;
                e[k][j] = col < S ? col - (uint32_t(c.m) + j - kZero) : kNone;
                hi[q] = uint32_t(max(int32_t(hi[q]), int32_t(e[k][j])));
                lo[q] = min(lo[q], e[k][j]);
            }
        }
        const uint32_t top = wave_reduce4(hi, [](uint32_t a, uint32_t b) {
            return uint32_t(max(int32_t(a), int32_t(b)));
        });
        const uint32_t low = wave_reduce4(lo, [](uint32_t a, uint32_t b) { return min(a, b); });
        const uint32_t span = low < kNone ? top - low : 0u;
        base[g] = low < kNone ? low + span / 2 : kZero;
        wide = wide || span > uint32_t(kCodeMax - kCodeMin);
        word = (lane & 15) == g ? base[g] - kZero : word;
    }
    wide = __any(wide);
    uint32_t esc = 0;
    Codes4 code[Q - 1];
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        const uint32_t b = uint32_t(__builtin_amdgcn_readlane(int(base[k / 4]), 16 * (k % 4)));
        uint32_t r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = int32_t(e[k][j]) < 0 ? uint32_t(kCodeBounce) : e[k][j] - b;
        if (wide) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool escape = int32_t(e[k][j]) >= 0 && r[j] - uint32_t(kCodeMin) > uint32_t(kCodeMax - kCodeMin);
                r[j] = escape ? uint32_t(kCodeEscape) : r[j];
                esc += escape ? 1u : 0u;
            }
        }
        code[k] = Codes4{int16_t(r[0]), int16_t(r[1]), int16_t(r[2]), int16_t(r[3])};
    }
    store_rows(codes, stride, c, code);
    if (wide)
        for (int off = 32; off > 0; off >>= 1) esc += __shfl_xor(esc, off);
    // the record: word 4 g + q from lane 16 q + g, then the escapes and 0
    const int at = 4 * (lane & 15) + (lane >> 4);
    if (at < kRec) rec[tile * kRec + at] = int32_t(at < Q - 1 ? word : at == Q - 1 ? esc : 0u);
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
__global__ __launch_bounds__(kCodeBlock) void k_narrow(const int16_t* __restrict__ codes, int64_t n,
                                                       int64_t stride, int64_t tiles,
                                                       int32_t* __restrict__ rec,
                                                       int8_t* __restrict__ codes8) {
    const int64_t tile = wave_tile();
    if (tile >= tiles) return;
    const int lane = int(threadIdx.x) & 63;
    const LaneCells c(tile, lane, n);
    Codes4 cd[Q - 1];
    load_rows(codes, stride, c, kCodeBounce, cd);
    // the largest of every code and its negative; the code of a bounce-back,
    // -2^15, is its own negative in 16 bits
    Pair size = {0, 0};
    const auto grow = [&](Pair v) {
        typedef uint16_t Bits __attribute__((ext_vector_type(2)));
        const Pair neg = __builtin_bit_cast(Pair, Bits{0, 0} - __builtin_bit_cast(Bits, v));
        size = __builtin_elementwise_max(size, __builtin_elementwise_max(v, neg));
    };
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        grow(cd[k].xy);
        grow(cd[k].zw);
    }
    const bool narrow = __all(max(size.x, size.y) <= kCode8Max);
    // the low byte of a code, of -128 for a bounce-back
    const auto bytes_of = [](Pair v) {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, Pair{kCode8Bounce, kCode8Bounce}));
    };
    Bytes4 bytes[Q - 1];
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        const uint32_t four = __builtin_amdgcn_perm(bytes_of(cd[k].zw), bytes_of(cd[k].xy), 0x06040200u);
        bytes[k] = __builtin_bit_cast(Bytes4, narrow ? four : 0u);
    }
    store_rows(codes8, stride, c, bytes);
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
            const BoundKernel kernel(k_trt_c8<ST, PBB, pol>, l.grid, l.block, s, n_steps);
            return steps([&](const T* src, T* dst, XcdMap map) {
                return kernel(src, dst, codes8, codes, toff, adj, ns, n, stride, c, map);
            });
        }
        const BoundKernel kernel(k_trt_c16<ST, PBB, pol>, l.grid, l.block, s, n_steps);
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
    k_compress<<<grid, kCodeBlock, code_lds(n), s>>>(adj, n, stride, tiles, codes, tile_records);
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
    k_narrow<<<grid, kCodeBlock, code_lds(n), s>>>(codes, n, stride, tiles, tile_records, codes8);
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
