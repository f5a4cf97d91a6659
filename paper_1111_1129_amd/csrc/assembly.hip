// assembly.hip -- assembly of the sparse representation on the GPU
// (lbm_build_adjacency).
//
// The paper's preprocessor (Sec. 3) numbers every box cell with an injective
// key, removes the gaps left by solid cells to get the contiguous index I_c,
// then finds each fluid cell's neighbours in the full representation.  Its
// distributed octree merge of incell runs computes, for every fluid cell, the
// number of fluid cells with a smaller key.  On one GPU that is an exclusive
// prefix count of fluid flags taken in key order, done here as a three-pass
// stream compaction:
//   1. count:  walk key positions in order, decode each to a box cell, test
//              its flag; ballot + popcount, one total per wave;
//   2. scan:   exclusive scan of those totals (one workgroup);
//   3. emit:   walk again; a lane's rank = wave offset + running total +
//              fluid lanes before it (mbcnt over the ballot mask); write
//              cell_of[rank] and index_of[cell];
//   4. adjacency: one thread per fluid cell, 18 neighbour lookups in index_of.
// A large lexicographic list (kTableBox) looks its neighbours up in rank words,
// a bit mask and a rank for every 32 cells: pass 3 writes those and cell_of, and
// index_of is written by another walk after the adjacency, if the caller wants it.
// All counts are exact integers, so the result does not depend on tile size
// or workgroup count (Sec. 8: the same sparse representation always).
//
// Key positions: lexicographic and blocked orders are walked through a
// gap-free "compact" position that decodes directly to the cell holding that
// rank among box cells; the Z curves, the Hilbert curve and the random order
// walk their own key space (a power of two, at most 8x the cube around the
// box) and skip positions that decode outside the box.
//
// The walk is bound by the decode wherever that is done per position in 64
// bits, so it is split: 4096 consecutive positions (a tile) of a Z or Hilbert
// curve are a 16^3 cube and 64 (a row, one wave load) a 4^3 cube, so the upper
// digits of the key are decoded once per tile, the next two per row, both
// uniform over the wave, and a lane adds its own two; aligned cubes outside the
// box are passed over whole.  The blocked order finds the block of a row once
// and divides by multiplication (box indices fit 31 bits).  Every wave walks
// its own run of positions, 16 rows at a time with all 16 flag loads in flight
// before the first ballot, and needs no barrier.  us for count / emit, before
// -> now: lexicographic, 75 M box cells 95 / 172 -> 24 / 97 (emit moves 0.5 GB,
// 5.2 TB/s); Hilbert curve over a 500 x 100 x 100 box, 134 M positions 718 /
// 758 -> 48 / 58.
#include <algorithm>

#include "lbm_device.hpp"
#include "lbm_host.hpp"

namespace lbm {

constexpr int kWalkBlock = 256;
constexpr int kWalkWaves = kWalkBlock / 64;
constexpr int kRow = 64;                     // positions of one wave load
constexpr int kRows = 16;                    // rows of a unit, in flight together
constexpr int kUnit = kRows * kRow;          // 1024 positions
constexpr int kTileUnits = 4;                // units of a tile (4096 positions)
constexpr int64_t kMaxGroups = 32768;        // waves of a walk
constexpr int kScanThreads = 1024;
constexpr uint64_t kMaxPositions = uint64_t(1) << 34;

// n / d for n < 2^31 by multiplication: with l = ceil(log2 d) and
// mul = ceil(2^(31 + l) / d) < 2^32 the error mul * d - 2^(31 + l) is below
// d <= 2^l, so n times it stays below 2^(31 + l) and the quotient is exact.
struct FastDiv {
    uint32_t mul, shift, d;
};

inline FastDiv make_div(uint64_t d) {
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    return FastDiv{uint32_t(((uint64_t(1) << (31 + l)) + d - 1) / d), l, uint32_t(d)};
}

// (quotient, remainder) in place: n becomes the remainder
__device__ __forceinline__ uint32_t div_rem(uint32_t& n, FastDiv f) {
    const uint32_t q = __umulhi(n << 1, f.mul) >> f.shift;
    n -= q * f.d;
    return q;
}

__device__ __forceinline__ FastDiv pick(bool second, FastDiv a, FastDiv b) {
    return FastDiv{second ? b.mul : a.mul, second ? b.shift : a.shift, second ? b.d : a.d};
}

// Blocked order: sizes of a whole block and of the last one in each direction
// ([0] whole, [1] last), as divisors.
struct BlockDivs {
    uint32_t b, last_x, last_y, last_z;  // block edge; block indices of the last blocks
    FastDiv slab;                        // cells of a slab of whole blocks in z
    FastDiv row[2];                      // cells of a row of blocks, by z block
    FastDiv blk[2][2];                   // cells of a block, by z and y block
    FastDiv bx[2], by[2];                // cells of a block's x row; its rows per plane
    uint32_t whole_bz, last_bz;          // its planes
};

struct KeySpace {
    int order;
    int h;             // random order: half width
    uint32_t nx, ny, nz;
    uint64_t seed;     // random order
    int groups;        // Z and Hilbert curves: number of 1-bit or 2-bit (MORTON2) groups
    uint64_t positions;
    BlockDivs blocks;  // blocked order
};

__host__ __device__ inline uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Inverse of the 4-round Feistel bijection used as the random ordering's key
// (forward round r: (L, R) -> (R, L ^ F_r(R))).
__device__ inline uint64_t feistel_inverse(uint64_t seed, int h, uint64_t v) {
    const uint64_t mask = (uint64_t(1) << h) - 1;
    uint64_t L = (v >> h) & mask, R = v & mask;
    for (int r = 3; r >= 0; --r) {
        const uint64_t prevR = L;
        const uint64_t prevL = R ^ (splitmix64(seed ^ (uint64_t(r) << 32) ^ prevR) & mask);
        L = prevL;
        R = prevR;
    }
    return (L << h) | R;
}

struct Vec3 {
    uint32_t x, y, z;
};

__device__ __forceinline__ int32_t linear_in_box(const KeySpace& ks, Vec3 c) {
    return c.x < ks.nx && c.y < ks.ny && c.z < ks.nz ? int32_t(c.x + ks.nx * (c.y + ks.ny * c.z)) : -1;
}

// Coordinates from interleaved groups of GB bits, `count` groups.
template <int GB>
__device__ __forceinline__ Vec3 deinterleave(uint64_t p, int count) {
    constexpr uint32_t mask = (1u << GB) - 1;
    Vec3 c{0u, 0u, 0u};
    for (int k = 0; k < count; ++k) {
        const uint32_t digit = uint32_t(p >> (3 * GB * k));
        c.x |= (digit & mask) << (GB * k);
        c.y |= ((digit >> GB) & mask) << (GB * k);
        c.z |= ((digit >> (2 * GB)) & mask) << (GB * k);
    }
    return c;
}

// One level of the inverse of Skilling's coordinates-to-index transform: with
// `bits` the three words' bits of this level, every word's lower bits (mask
// `low`) are reflected or exchanged.
__device__ __forceinline__ void hilbert_level(Vec3& v, Vec3 bits, uint32_t low) {
    if (bits.z) {
        v.x ^= low;
    } else {
        const uint32_t t = (v.x ^ v.z) & low;
        v.x ^= t;
        v.z ^= t;
    }
    if (bits.y) {
        v.x ^= low;
    } else {
        const uint32_t t = (v.x ^ v.y) & low;
        v.x ^= t;
        v.y ^= t;
    }
    if (bits.x) v.x ^= low;
}

// Cell of `levels` Hilbert digits p: split into the three transposed words
// (x's bit the most significant of each 3-bit digit), undo the Gray code
// (`carry`: z's bit of the digit above, 0 at the top), then undo the
// reflections and exchanges of these levels from the lowest up.  gray gets the
// words before that, whose bits decide what the levels do to the bits below
// (a level touches lower bits only, so the decisions are not changed on the
// way and a lower part of the key can be decoded by itself).
__device__ __forceinline__ Vec3 hilbert_digits(uint64_t p, int levels, uint32_t carry, Vec3& gray) {
    Vec3 v{0u, 0u, 0u};
    for (int j = 0; j < levels; ++j) {
        const uint32_t digit = uint32_t(p >> (3 * j));
        v.x |= ((digit >> 2) & 1u) << j;
        v.y |= ((digit >> 1) & 1u) << j;
        v.z |= (digit & 1u) << j;
    }
    const uint32_t t = (v.z | (carry << levels)) >> 1;
    v.z ^= v.y;
    v.y ^= v.x;
    v.x ^= t;
    gray = v;
    for (int j = 1; j < levels; ++j)
        hilbert_level(v, Vec3{(gray.x >> j) & 1u, (gray.y >> j) & 1u, (gray.z >> j) & 1u},
                      (1u << j) - 1);
    return v;
}

// What the levels above a part of a Hilbert key do to it: an exchange of the
// words and a reflection of each, found by passing marked words through them.
struct Orient {
    uint32_t px, py, pz;  // which word each coordinate comes from
    uint32_t rx, ry, rz;  // ~0: reflected
};

__device__ __forceinline__ uint32_t word_of(Vec3 v, uint32_t which) {
    return which == 0 ? v.x : which == 1 ? v.y : v.z;
}

__device__ __forceinline__ Vec3 oriented(const Orient& o, Vec3 v, uint32_t low) {
    return Vec3{word_of(v, o.px) ^ (o.rx & low), word_of(v, o.py) ^ (o.ry & low),
                word_of(v, o.pz) ^ (o.rz & low)};
}

__device__ __forceinline__ Orient orientation(Vec3 gray, int levels) {
    // bits [0, 3): the word's mark; the same value reflected reads 7 - mark
    Vec3 v{0u, 1u, 2u};
    for (int j = 0; j < levels; ++j)
        hilbert_level(v, Vec3{(gray.x >> j) & 1u, (gray.y >> j) & 1u, (gray.z >> j) & 1u}, 7u);
    Orient o;
    o.rx = v.x > 2 ? ~0u : 0u;
    o.ry = v.y > 2 ? ~0u : 0u;
    o.rz = v.z > 2 ? ~0u : 0u;
    o.px = v.x > 2 ? 7u - v.x : v.x;
    o.py = v.y > 2 ? 7u - v.y : v.y;
    o.pz = v.z > 2 ? 7u - v.z : v.z;
    return o;
}

// Walk over the positions of one order, in tiles of 4096.  tile() is called
// with the index of a tile (uniform over the wave) and returns 0, or how many
// tiles from this one on are known to hold no cell of the box.  row() is called
// for a row of the tile (uniform) and cell() gives the box cell (linear index)
// at a lane of it, -1 for a gap.
template <int ORDER> struct Walk;

template <> struct Walk<LBM_ORDER_LEX> {
    uint64_t p0, p;
    __device__ explicit Walk(int) {}
    __device__ __forceinline__ uint32_t tile(const KeySpace&, uint32_t t) {
        p0 = uint64_t(t) * (kTileUnits * kUnit);
        return 0;
    }
    __device__ __forceinline__ void row(const KeySpace&, int r) { p = p0 + uint32_t(r * kRow); }
    __device__ __forceinline__ int32_t cell(const KeySpace& ks, int lane) const {
        return p + uint32_t(lane) < ks.positions ? int32_t(uint32_t(p) + uint32_t(lane)) : -1;
    }
};

template <> struct Walk<LBM_ORDER_BLOCKED> {
    uint64_t p0;
    uint32_t p;                // first position of the row
    bool whole;                // the row lies in one block
    uint32_t rest;             // its first position's place in that block
    uint32_t bx, by, bz;       // indices of the block
    bool lx, ly, lz;           // it is the last one in x, y, z
    __device__ explicit Walk(int) {}
    __device__ __forceinline__ uint32_t tile(const KeySpace&, uint32_t t) {
        p0 = uint64_t(t) * (kTileUnits * kUnit);
        return 0;
    }
    // block of position r; r becomes the place in it
    __device__ __forceinline__ static void block_of(const BlockDivs& d, uint32_t& r, uint32_t& X,
                                                    uint32_t& Y, uint32_t& Z) {
        Z = div_rem(r, d.slab);
        const bool lz = Z == d.last_z;
        Y = div_rem(r, pick(lz, d.row[0], d.row[1]));
        X = div_rem(r, block_cells(d, Y == d.last_y, lz));
    }
    __device__ __forceinline__ static FastDiv block_cells(const BlockDivs& d, bool ly, bool lz) {
        return pick(ly, pick(lz, d.blk[0][0], d.blk[1][0]), pick(lz, d.blk[0][1], d.blk[1][1]));
    }
    __device__ __forceinline__ static int32_t in_block(const KeySpace& ks, uint32_t r, uint32_t X,
                                                       uint32_t Y, uint32_t Z) {
        const BlockDivs& d = ks.blocks;
        uint32_t t = div_rem(r, pick(X == d.last_x, d.bx[0], d.bx[1]));     // r: x in the block
        const uint32_t z = div_rem(t, pick(Y == d.last_y, d.by[0], d.by[1]));  // t: y in it
        return int32_t((X * d.b + r) + ks.nx * ((Y * d.b + t) + ks.ny * (Z * d.b + z)));
    }
    __device__ __forceinline__ void row(const KeySpace& ks, int r) {
        const uint64_t first = p0 + uint32_t(r * kRow);
        whole = false;
        if (first >= ks.positions) {
            p = ~0u;
            return;
        }
        p = uint32_t(first);
        rest = p;
        block_of(ks.blocks, rest, bx, by, bz);
        // cells of this block (bx.d of a last block in x over the whole one's)
        const BlockDivs& d = ks.blocks;
        const uint32_t cells = (bx == d.last_x ? d.bx[1].d : d.bx[0].d) *
                               (by == d.last_y ? d.by[1].d : d.by[0].d) *
                               (bz == d.last_z ? d.last_bz : d.whole_bz);
        whole = rest + kRow <= cells;
    }
    __device__ __forceinline__ int32_t cell(const KeySpace& ks, int lane) const {
        if (whole) return in_block(ks, rest + uint32_t(lane), bx, by, bz);
        const uint64_t q = uint64_t(p) + uint32_t(lane);
        if (q >= ks.positions) return -1;
        uint32_t r = uint32_t(q), X, Y, Z;
        block_of(ks.blocks, r, X, Y, Z);
        return in_block(ks, r, X, Y, Z);
    }
};

// A curve's aligned cubes are aligned runs of positions.  `digits` is the
// number of binary digits of a tile's coordinates; the first two, decoded by
// themselves, already show most of the tiles outside a box that is much
// smaller than its cube.  decode(p, n): the cube of n leading digits p.
// Returns the tiles left in that cube if it lies outside the box, else 0.
template <class F>
__device__ __forceinline__ uint32_t coarse_tiles_outside(const KeySpace& ks, uint32_t t, int digits,
                                                         F&& decode) {
    if (digits <= 2) return 0;
    const int rest = digits - 2;
    const Vec3 c = decode(t >> (3 * rest), 2);
    const bool out = (c.x << (rest + 4)) >= ks.nx || (c.y << (rest + 4)) >= ks.ny ||
                     (c.z << (rest + 4)) >= ks.nz;
    const uint32_t run = 1u << (3 * rest);
    return out ? run - (t & (run - 1)) : 0u;
}

// The same for the cubes of 64, 8 and 1 tiles that begin at t; c is any cell of
// tile t.
__device__ __forceinline__ uint32_t tiles_outside(const KeySpace& ks, uint32_t t, Vec3 c) {
    for (int s = 2; s >= 0; --s) {
        const uint32_t run = 1u << (3 * s), edge = 16u << s;
        const Vec3 o{c.x & ~(edge - 1), c.y & ~(edge - 1), c.z & ~(edge - 1)};
        if ((t & (run - 1)) == 0 && (o.x >= ks.nx || o.y >= ks.ny || o.z >= ks.nz)) return run;
    }
    return 0;
}

template <int GB> struct ZWalk {
    Vec3 lane_c, tile_c, row_c;
    __device__ explicit ZWalk(int lane) : lane_c(deinterleave<GB>(uint64_t(lane), 2 / GB)) {}
    __device__ __forceinline__ uint32_t tile(const KeySpace& ks, uint32_t t) {
        const uint32_t skip = coarse_tiles_outside(
            ks, t, ks.groups * GB - 4,
            [](uint32_t p, int n) { return deinterleave<GB>(p, n / GB); });
        if (skip) return skip;
        tile_c = deinterleave<GB>(t, ks.groups - 4 / GB);
        tile_c = Vec3{tile_c.x << 4, tile_c.y << 4, tile_c.z << 4};
        return tiles_outside(ks, t, tile_c);
    }
    __device__ __forceinline__ void row(const KeySpace&, int r) {
        row_c = deinterleave<GB>(uint64_t(r), 2 / GB);
        row_c = Vec3{tile_c.x + 4 * row_c.x, tile_c.y + 4 * row_c.y, tile_c.z + 4 * row_c.z};
    }
    __device__ __forceinline__ int32_t cell(const KeySpace& ks, int) const {
        // a position past the key space has a coordinate past its cube
        return linear_in_box(ks, Vec3{row_c.x + lane_c.x, row_c.y + lane_c.y, row_c.z + lane_c.z});
    }
};
template <> struct Walk<LBM_ORDER_MORTON1> : ZWalk<1> { using ZWalk<1>::ZWalk; };
template <> struct Walk<LBM_ORDER_MORTON2> : ZWalk<2> { using ZWalk<2>::ZWalk; };

template <> struct Walk<LBM_ORDER_HILBERT> {
    Vec3 lane_c[2];  // the lane's two digits, by the carry from the row's last digit
    Vec3 tile_c, row_c, row_gray;
    Orient tile_o;
    uint32_t t, r;
    __device__ explicit Walk(int lane) {
        Vec3 g;
        lane_c[0] = hilbert_digits(uint64_t(lane), 2, 0u, g);
        lane_c[1] = hilbert_digits(uint64_t(lane), 2, 1u, g);
    }
    __device__ __forceinline__ uint32_t tile(const KeySpace& ks, uint32_t tile) {
        t = tile;
        if (ks.groups < 4) return 0;
        Vec3 g;
        uint32_t skip = coarse_tiles_outside(
            ks, t, ks.groups - 4, [&](uint32_t p, int n) { return hilbert_digits(p, n, 0u, g); });
        if (skip) return skip;
        tile_c = hilbert_digits(t, ks.groups - 4, 0u, g);
        tile_c = Vec3{tile_c.x << 4, tile_c.y << 4, tile_c.z << 4};
        skip = tiles_outside(ks, t, tile_c);
        if (skip == 0) tile_o = orientation(g, ks.groups - 4);
        return skip;
    }
    __device__ __forceinline__ void row(const KeySpace& ks, int row) {
        r = uint32_t(row);
        if (ks.groups < 4) return;
        // carry into the row's digits: z's bit of the tile's last digit
        const uint32_t carry = ks.groups > 4 ? t & 1u : 0u;
        const Vec3 c = oriented(tile_o, hilbert_digits(r, 2, carry, row_gray), 3u);
        row_c = Vec3{tile_c.x + 4 * c.x, tile_c.y + 4 * c.y, tile_c.z + 4 * c.z};
    }
    __device__ __forceinline__ int32_t cell(const KeySpace& ks, int lane) const {
        if (ks.groups < 4) {  // the whole curve is shorter than a tile
            const uint64_t p = uint64_t(r) * kRow + uint32_t(lane);
            Vec3 g;
            return p < ks.positions ? linear_in_box(ks, hilbert_digits(p, ks.groups, 0u, g)) : -1;
        }
        Vec3 l = (r & 1) ? lane_c[1] : lane_c[0];
        hilbert_level(l, Vec3{row_gray.x & 1u, row_gray.y & 1u, row_gray.z & 1u}, 3u);
        hilbert_level(l, Vec3{row_gray.x >> 1, row_gray.y >> 1, row_gray.z >> 1}, 3u);
        l = oriented(tile_o, l, 3u);
        return linear_in_box(ks, Vec3{row_c.x + l.x, row_c.y + l.y, row_c.z + l.z});
    }
};

template <> struct Walk<LBM_ORDER_RANDOM> {
    uint64_t p0, p;
    __device__ explicit Walk(int) {}
    __device__ __forceinline__ uint32_t tile(const KeySpace&, uint32_t t) {
        p0 = uint64_t(t) * (kTileUnits * kUnit);
        return 0;
    }
    __device__ __forceinline__ void row(const KeySpace&, int r) { p = p0 + uint32_t(r * kRow); }
    __device__ __forceinline__ int32_t cell(const KeySpace& ks, int lane) const {
        const uint64_t q = p + uint32_t(lane);
        if (q >= ks.positions) return -1;
        const uint64_t lin = feistel_inverse(ks.seed, ks.h, q);
        return lin < uint64_t(ks.nx) * ks.ny * ks.nz ? int32_t(lin) : -1;
    }
};

// Calls unit(cells, masks) for each unit in [u0, u1) that may hold a cell of
// the box: the box cells at its 16 rows and their fluid masks.
template <int ORDER, class F>
__device__ __forceinline__ void walk_units(const KeySpace& ks, const uint8_t* __restrict__ flag,
                                           uint32_t u0, uint32_t u1, int lane, F&& unit) {
    Walk<ORDER> walk(lane);
    uint32_t u = u0;
    bool fresh = true;  // the tile of u has not been decoded
    while (u < u1) {
        if (fresh || u % kTileUnits == 0) {
            const uint32_t skip = walk.tile(ks, u / kTileUnits);
            fresh = skip != 0;
            if (skip) {
                u = (u / kTileUnits + skip) * kTileUnits;
                continue;
            }
        }
        int32_t lin[kRows];
        uint8_t fl[kRows];
        uint64_t mask[kRows];
        const int r0 = int(u % kTileUnits) * kRows;
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            walk.row(ks, r0 + j);
            lin[j] = walk.cell(ks, lane);
        }
#pragma unroll
        for (int j = 0; j < kRows; ++j) fl[j] = flag[lin[j] < 0 ? 0 : lin[j]];
#pragma unroll
        for (int j = 0; j < kRows; ++j) mask[j] = __ballot(lin[j] >= 0 && fl[j] != 0);
        unit(lin, mask);
        ++u;
    }
}

// Wave g of the launch (a "group") walks units [g * per, (g + 1) * per).
__device__ __forceinline__ uint32_t wave_group() {
    return blockIdx.x * kWalkWaves + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
}

template <int ORDER>
__global__ __launch_bounds__(kWalkBlock) void k_count(KeySpace ks, const uint8_t* __restrict__ flag,
                                                      uint32_t units, uint32_t per, uint32_t groups,
                                                      uint32_t* __restrict__ group_count) {
    const uint32_t g = wave_group();
    if (g >= groups) return;
    const int lane = int(threadIdx.x) & 63;
    uint32_t mine = 0;
    walk_units<ORDER>(ks, flag, g * per, min(units, (g + 1) * per), lane,
                      [&](const int32_t*, const uint64_t* mask) {
#pragma unroll
                          for (int j = 0; j < kRows; ++j) mine += __popcll(mask[j]);
                      });
    if (lane == 0) group_count[g] = mine;
}

// Exclusive scan of n <= kMaxGroups counts in place (room for a multiple of 4),
// total written to *total.  One workgroup: each thread takes a run of counts,
// four to a load.
__global__ __launch_bounds__(kScanThreads) void k_scan(uint32_t* __restrict__ v, int n,
                                                       int64_t* __restrict__ total) {
    constexpr int kMaxQuads = int(kMaxGroups) / kScanThreads / 4;
    __shared__ uint32_t wave_tot[kScanThreads / 64];
    const int tid = threadIdx.x;
    const int quads = (n + 4 * kScanThreads - 1) / (4 * kScanThreads);  // of each thread
    uint4* const q = reinterpret_cast<uint4*>(v) + int64_t(tid) * quads;
    uint4 c[kMaxQuads];
    uint32_t local = 0;
#pragma unroll
    for (int i = 0; i < kMaxQuads; ++i) {
        c[i] = uint4{0u, 0u, 0u, 0u};
        const int at = 4 * (tid * quads + i);
        if (i < quads && at < n) {
            c[i] = q[i];
            if (at + 1 >= n) c[i].y = 0u;
            if (at + 2 >= n) c[i].z = 0u;
            if (at + 3 >= n) c[i].w = 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < kMaxQuads; ++i) local += c[i].x + c[i].y + c[i].z + c[i].w;
    // inclusive scan of `local` across the workgroup (a box has < 2^31 cells)
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t x = local;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    uint32_t run = x - local;  // exclusive prefix of this thread's counts
    for (int w = 0; w < wave; ++w) run += wave_tot[w];
#pragma unroll
    for (int i = 0; i < kMaxQuads; ++i) {
        if (i < quads && 4 * (tid * quads + i) < n) {
            uint4 o;
            o.x = run;
            o.y = o.x + c[i].x;
            o.z = o.y + c[i].y;
            o.w = o.z + c[i].z;
            q[i] = o;
        }
        run += c[i].x + c[i].y + c[i].z + c[i].w;
    }
    if (tid == kScanThreads - 1) *total = int64_t(run);
}

// Lexicographic order: the fluid cells among 32 consecutive box cells and the
// rank of the first of them.  A table of these holds all that index_of does in
// a sixteenth of the bytes.  Entry w + 1 covers cells [32 w, 32 w + 32); the
// first and the last kRankGuard entries are empty.
struct RankWord {
    uint32_t mask, rank;
};
constexpr int64_t kRankGuard = 2;

// Entries of a table over so many units: a guard, the words, two more guards.
constexpr int64_t rank_words(int64_t units) { return 1 + units * (kUnit / 32) + kRankGuard; }

// Smallest box for the rank words: below it index_of stays in the last-level
// cache between the two kernels, and reading it costs less than a second pass
// over the flags (whole call, index / words: 320^3 273 / 281 us and, with
// porosity 0.8, 426 / 452; 384^3 634 / 460 and 1,084 / 765).  The words fit in
// the index: a quarter of it, and a unit's worth and the guards beyond that.
constexpr int64_t kTableBox = int64_t(40) << 20;
static_assert(rank_words(kTableBox / kUnit + 1) * sizeof(RankWord) <= kTableBox * sizeof(int32_t),
              "rank words fit in the index");

// Which of its results a k_emit launch writes: the list and the index, the list
// and the rank words, or the index.
enum EmitPart { kEmitAll = 0, kEmitList = 1, kEmitIndex = 2 };

template <int ORDER, int PART>
__global__ __launch_bounds__(kWalkBlock) void k_emit(KeySpace ks, const uint8_t* __restrict__ flag,
                                                     uint32_t units, uint32_t per, uint32_t groups,
                                                     const uint32_t* __restrict__ group_offset,
                                                     int32_t* __restrict__ index_of,
                                                     int32_t* __restrict__ cell_of,
                                                     RankWord* __restrict__ table) {
    const uint32_t g = wave_group();
    if (PART == kEmitList && g == 0 && threadIdx.x <= kRankGuard)
        table[threadIdx.x == 0 ? 0 : rank_words(units) - threadIdx.x] = RankWord{0u, 0u};
    if (g >= groups) return;
    const int lane = int(threadIdx.x) & 63;
    uint32_t r = group_offset[g];
    uint32_t u = g * per;  // lexicographic order: the unit at hand (none is passed over)
    walk_units<ORDER>(ks, flag, g * per, min(units, (g + 1) * per), lane,
                      [&](const int32_t* lin, const uint64_t* mask) {
        if constexpr (PART == kEmitList) {
            // lane 2 j + h writes half h of row j
            uint64_t m = 0;
            uint32_t first = 0, before = r;
#pragma unroll
            for (int j = 0; j < kRows; ++j) {
                const bool mine = (lane >> 1) == j;
                m = mine ? mask[j] : m;
                first = mine ? before : first;
                before += __popcll(mask[j]);
            }
            const uint32_t lo = uint32_t(m), hi = uint32_t(m >> 32);
            if (lane < 2 * kRows)
                table[1 + int64_t(u) * (kUnit / 32) + lane] =
                    (lane & 1) ? RankWord{hi, first + uint32_t(__popc(lo))} : RankWord{lo, first};
            ++u;
        }
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            // fluid lanes below this one in the row
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                uint32_t(mask[j] >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask[j]), 0u));
            const bool fluid = (mask[j] >> lane) & 1u;
            if (PART != kEmitIndex && fluid) cell_of[r + below] = lin[j];
            if (PART != kEmitList && lin[j] >= 0) index_of[lin[j]] = fluid ? int32_t(r + below) : -1;
            r += __popcll(mask[j]);
        }
    });
}

struct AdjGeom {
    FastDiv nx, ny;
    uint32_t nz, periodic;
    uint32_t base, stride;
};

// What a step of one cell against velocity component c (index c + 1) along
// one dimension adds to the linear index, and whether it leaves the box.
struct Steps {
    uint32_t add[3];
    bool out[3];
};

__device__ __forceinline__ Steps steps_along(uint32_t x, uint32_t n, uint32_t pitch, bool wrap) {
    const bool lo = x == 0, hi = x == n - 1;
    Steps s;
    s.add[0] = hi ? (1u - n) * pitch : pitch;  // c = -1: upstream is x + 1
    s.add[1] = 0u;
    s.add[2] = lo ? (n - 1u) * pitch : 0u - pitch;
    s.out[0] = hi && !wrap;
    s.out[1] = false;
    s.out[2] = lo && !wrap;
    return s;
}

// Ranks (-1: solid) of box cells at - 1, at and at + 1.
struct Triple {
    int32_t v[3];
};

__device__ __forceinline__ int32_t rank_in(RankWord w, uint32_t bit) {
    return (w.mask >> bit) & 1u ? int32_t(w.rank + __popc(w.mask & ((1u << bit) - 1))) : -1;
}

// Where the ranks come from: index_of, or the rank words of a lexicographic
// list (the words of at - 1 and the one after it in one access).
struct FromIndex {
    const int32_t* __restrict__ index_of;
    __device__ __forceinline__ int32_t one(uint32_t at) const { return index_of[at]; }
    __device__ __forceinline__ Triple three(uint32_t at) const {
        return *reinterpret_cast<const Triple*>(index_of + at - 1);
    }
};

struct FromTable {
    const RankWord* __restrict__ table;
    __device__ __forceinline__ int32_t one(uint32_t at) const {
        return rank_in(table[(at >> 5) + 1], at & 31u);
    }
    __device__ __forceinline__ Triple three(uint32_t at) const {
        struct Two {
            RankWord w[2];
        };
        const uint32_t first = at + 31u;  // cell at - 1, counted from the table's first word
        const Two two = *reinterpret_cast<const Two*>(table + (first >> 5));
        const uint32_t bit = first & 31u;
        const uint64_t mask = two.w[0].mask | uint64_t(two.w[1].mask) << 32;
        const uint32_t bits = uint32_t(mask >> bit);  // of the three cells, from the lowest
        // the second word's rank is the first's plus its fluid cells
        uint32_t r = two.w[0].rank + __popc(two.w[0].mask & ((1u << bit) - 1));
        Triple t;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            t.v[j] = (bits >> j) & 1u ? int32_t(r) : -1;
            r += (bits >> j) & 1u;
        }
        return t;
    }
};

// One thread per fluid cell.  Its rank lookups are all in flight at once (a
// neighbour outside a non-periodic face reads the cell's own entry and is then
// discarded).  What bounds them is the address unit, which takes a gather's
// cache lines one by one: 64 consecutive fluid cells of a packing lie on about
// six lines of a box row of index_of.  The 14 neighbours on the five rows (y,
// z), (y +- 1, z), (y, z +- 1) are therefore read three along x at a time, 9
// gathers for 18; only cells on the box's x faces read them one by one.  The
// rows written (72 of the 80 bytes a cell moves) go past the caches, which are
// left to the ranks.  6.9 M cells of a 256^3 packing: 97 us, 5.7 TB/s (153 with
// cached stores); 4.8 M cells of a Hilbert-ordered channel 69 us (121 with 18
// gathers and cached stores).  30.6 M cells of a 384 x 384 x 512 packing, whose
// index_of does not fit the last-level cache: the gathers wait about 2,100
// cycles for memory that the stores keep busy, 690 us, of which the stores by
// themselves take 437; a large lexicographic list reads rank words instead (381
// us).  Runs of consecutive blocks per XCD: 8 or 32, 3 to 6 % faster than one
// eighth each.
// STREAM: cell_of comes in through nontemporal loads; see the launch.
template <bool STREAM, class Ranks>
__global__ __launch_bounds__(256) void k_adjacency(const int32_t* __restrict__ cell_of, Ranks ranks,
                                                   int64_t nf, AdjGeom g, XcdMap map,
                                                   uint32_t* __restrict__ adj) {
    const int64_t m = logical_block(map) * 256 + threadIdx.x;
    if (m >= nf) return;
    const uint32_t lin = uint32_t(STREAM ? __builtin_nontemporal_load(cell_of + m) : cell_of[m]);
    uint32_t x = lin;
    uint32_t y = div_rem(x, g.nx);
    const uint32_t z = div_rem(y, g.ny);
    const Steps sx = steps_along(x, g.nx.d, 1u, g.periodic & 1u);
    const Steps sy = steps_along(y, g.ny.d, g.nx.d, g.periodic & 2u);
    const Steps sz = steps_along(z, g.nz, g.nx.d * g.ny.d, g.periodic & 4u);
    int32_t up[Q - 1];
    if (x > 0 && x + 1 < g.nx.d) {
        Triple row[3][3];  // by the y and z components + 1; the diagonal rows: v[1] only
#pragma unroll
        for (int cy = 0; cy < 3; ++cy)
#pragma unroll
            for (int cz = 0; cz < 3; ++cz) {
                const uint32_t at = sy.out[cy] || sz.out[cz] ? lin : lin + sy.add[cy] + sz.add[cz];
                if (cy == 1 || cz == 1)
                    row[cy][cz] = ranks.three(at);
                else
                    row[cy][cz].v[1] = ranks.one(at);
            }
#pragma unroll
        for (int k = 0; k < Q - 1; ++k)
            up[k] = row[vel_y(k + 1) + 1][vel_z(k + 1) + 1].v[1 - vel_x(k + 1)];
    } else {
#pragma unroll
        for (int k = 0; k < Q - 1; ++k) {
            const int cx = vel_x(k + 1) + 1, cy = vel_y(k + 1) + 1, cz = vel_z(k + 1) + 1;
            const bool out = sx.out[cx] || sy.out[cy] || sz.out[cz];
            up[k] = ranks.one(out ? lin : lin + sx.add[cx] + sy.add[cy] + sz.add[cz]);
        }
    }
    const uint32_t self = g.base + uint32_t(m);
#pragma unroll
    for (int k = 0; k < Q - 1; ++k) {
        const int i = k + 1;
        const bool out = sx.out[vel_x(i) + 1] || sy.out[vel_y(i) + 1] || sz.out[vel_z(i) + 1];
        const uint32_t slot = !out && up[k] >= 0 ? uint32_t(i) * g.stride + g.base + uint32_t(up[k])
                                                 : uint32_t(opp(i)) * g.stride + self;
        __builtin_nontemporal_store(slot, adj + int64_t(k) * g.stride + self);
    }
}

static int bits_for(int64_t n) {
    int b = 0;
    while ((int64_t(1) << b) < n) ++b;
    return b;
}

static int feistel_half_bits(uint64_t n_box) {
    int h = 1;
    while (h < 31 && (uint64_t(1) << (2 * h)) < n_box) ++h;
    return h;
}

// Divisors of the blocked order with block edge b.  A slab or row that is
// larger than the box never divides anything: its quotient is 0 for every
// position, which any divisor above the last position gives.
static BlockDivs make_blocks(const lbm_geom& g, int64_t b) {
    const int64_t n_box = int64_t(g.nx) * g.ny * g.nz;
    BlockDivs d;
    d.b = uint32_t(b);
    const int64_t dims[3] = {g.nx, g.ny, g.nz};
    int64_t last[3], size[3][2];  // index of the last block; cells of a whole and of the last block
    for (int k = 0; k < 3; ++k) {
        last[k] = (dims[k] - 1) / b;
        size[k][0] = std::min<int64_t>(b, dims[k]);
        size[k][1] = dims[k] - last[k] * b;
    }
    d.last_x = uint32_t(last[0]);
    d.last_y = uint32_t(last[1]);
    d.last_z = uint32_t(last[2]);
    d.slab = make_div(std::min<int64_t>(b * dims[0] * dims[1], n_box));
    if (last[2] == 0) d.slab = make_div(n_box);
    for (int z = 0; z < 2; ++z) {
        d.row[z] = make_div(std::min<int64_t>(size[1][0] * dims[0] * size[2][z], n_box));
        for (int y = 0; y < 2; ++y)
            d.blk[z][y] = make_div(size[0][0] * size[1][y] * size[2][z]);
    }
    for (int e = 0; e < 2; ++e) {
        d.bx[e] = make_div(size[0][e]);
        d.by[e] = make_div(size[1][e]);
    }
    d.whole_bz = uint32_t(size[2][0]);
    d.last_bz = uint32_t(size[2][1]);
    return d;
}

// Fills ks; returns LBM_OK or an error for unusable geometry/order.
static lbm_status make_keyspace(const lbm_geom& g, KeySpace& ks) {
    ks = KeySpace{};
    ks.order = g.order;
    ks.nx = uint32_t(g.nx);
    ks.ny = uint32_t(g.ny);
    ks.nz = uint32_t(g.nz);
    const int64_t n_box = int64_t(g.nx) * g.ny * g.nz;
    const int64_t dmax = std::max<int64_t>({g.nx, g.ny, g.nz});
    switch (g.order) {
    case LBM_ORDER_LEX:
        ks.positions = uint64_t(n_box);
        break;
    case LBM_ORDER_BLOCKED:
        if (g.order_param == 0) return LBM_EINVAL;
        // blocks wider than the box order cells exactly like blocks as wide as it
        ks.blocks = make_blocks(g, std::min<int64_t>(int64_t(g.order_param), dmax));
        ks.positions = uint64_t(n_box);
        break;
    case LBM_ORDER_MORTON1:
    case LBM_ORDER_HILBERT: {
        ks.groups = bits_for(dmax);
        if (3 * ks.groups > 62) return LBM_EOVERFLOW;
        ks.positions = uint64_t(1) << (3 * ks.groups);
        break;
    }
    case LBM_ORDER_MORTON2: {
        ks.groups = (bits_for(dmax) + 1) / 2;
        if (6 * ks.groups > 62) return LBM_EOVERFLOW;
        ks.positions = uint64_t(1) << (6 * ks.groups);
        break;
    }
    case LBM_ORDER_RANDOM:
        ks.h = feistel_half_bits(uint64_t(n_box));
        ks.seed = g.order_param;
        ks.positions = uint64_t(1) << (2 * ks.h);
        break;
    default:
        return LBM_EINVAL;
    }
    if (ks.positions > kMaxPositions) return LBM_EOVERFLOW;
    return LBM_OK;
}

// Calls f(std::integral_constant<int, order>).
template <class F>
static void with_order(int order, F&& f) {
    switch (order) {
    case LBM_ORDER_LEX: return f(std::integral_constant<int, LBM_ORDER_LEX>{});
    case LBM_ORDER_BLOCKED: return f(std::integral_constant<int, LBM_ORDER_BLOCKED>{});
    case LBM_ORDER_MORTON1: return f(std::integral_constant<int, LBM_ORDER_MORTON1>{});
    case LBM_ORDER_MORTON2: return f(std::integral_constant<int, LBM_ORDER_MORTON2>{});
    case LBM_ORDER_HILBERT: return f(std::integral_constant<int, LBM_ORDER_HILBERT>{});
    default: return f(std::integral_constant<int, LBM_ORDER_RANDOM>{});
    }
}

}  // namespace lbm

using namespace lbm;

extern "C" lbm_status lbm_build_adjacency(const lbm_geom* g, const uint8_t* flag, int64_t base,
                                          int64_t stride, int32_t* index_of, int32_t* cell_of,
                                          uint32_t* adj, int64_t cap, int64_t* n_fluid,
                                          void* workspace, size_t* ws_bytes, void* stream) {
    if (!g || !ws_bytes) return LBM_EINVAL;
    if (g->nx <= 0 || g->ny <= 0 || g->nz <= 0) return LBM_EINVAL;
    const int64_t n_box = int64_t(g->nx) * g->ny * g->nz;
    if (n_box >= kBoxLimit) return LBM_EOVERFLOW;
    KeySpace ks;
    if (lbm_status st = make_keyspace(*g, ks); st != LBM_OK) return st;
    // units are dealt in equal runs to at most kMaxGroups waves
    const int64_t units = int64_t((ks.positions + kUnit - 1) / kUnit);
    const int64_t per = (units + kMaxGroups - 1) / kMaxGroups;
    const int64_t groups = (units + per - 1) / per;
    const dim3 walk_grid{unsigned((groups + kWalkWaves - 1) / kWalkWaves)};

    // workspace: wave counts | total | index_of scratch (only if index_of is NULL)
    const size_t off_total = align_up(size_t(groups) * sizeof(uint32_t), 256);
    const size_t off_index = off_total + 256;
    const size_t need = off_index + (index_of ? 0 : align_up(size_t(n_box) * sizeof(int32_t), 256));
    if (!workspace) {
        *ws_bytes = need;
        return LBM_OK;
    }
    if (*ws_bytes < need) return LBM_EWORKSPACE;
    if (!flag || !n_fluid) return LBM_EINVAL;
    if (base < 0 || cap < 0) return LBM_EINVAL;
    if (adj && !stride_fits(stride)) return LBM_EOVERFLOW;

    char* ws = static_cast<char*>(workspace);
    uint32_t* group_count = reinterpret_cast<uint32_t*>(ws);
    int64_t* total = reinterpret_cast<int64_t*>(ws + off_total);
    int32_t* idx = index_of ? index_of : reinterpret_cast<int32_t*>(ws + off_index);
    hipStream_t s = as_stream(stream);

    with_order(ks.order, [&](auto order) {
        k_count<order><<<walk_grid, dim3(kWalkBlock), 0, s>>>(
            ks, flag, uint32_t(units), uint32_t(per), uint32_t(groups), group_count);
    });
    if (hipGetLastError() != hipSuccess) return LBM_EHIP;
    k_scan<<<1, kScanThreads, 0, s>>>(group_count, int(groups), total);
    if (hipGetLastError() != hipSuccess) return LBM_EHIP;
    int64_t nf = 0;
    LBM_TRY_HIP(hipMemcpyAsync(&nf, total, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    LBM_TRY_HIP(hipStreamSynchronize(s));
    *n_fluid = nf;
    if (!cell_of) return LBM_OK;  // count-only pass
    if (nf > cap) return LBM_ECAPACITY;
    if (adj && stride < base + nf) return LBM_EINVAL;

    // A large lexicographic list with adjacency: the rank words lie in idx until
    // the adjacency has been found, and the index is written over them.
    RankWord* table = ks.order == LBM_ORDER_LEX && adj && nf > 0 && n_box >= kTableBox &&
                              reinterpret_cast<uintptr_t>(idx) % sizeof(RankWord) == 0
                          ? reinterpret_cast<RankWord*>(idx) : nullptr;
    const auto emit = [&](auto order, auto part) {
        k_emit<order, part><<<walk_grid, dim3(kWalkBlock), 0, s>>>(
            ks, flag, uint32_t(units), uint32_t(per), uint32_t(groups), group_count, idx, cell_of, table);
        return after_launch();
    };
    constexpr auto lex = std::integral_constant<int, LBM_ORDER_LEX>{};
    lbm_status st = LBM_OK;
    if (table)
        st = emit(lex, std::integral_constant<int, kEmitList>{});
    else
        with_order(ks.order, [&](auto order) { st = emit(order, std::integral_constant<int, kEmitAll>{}); });
    if (st != LBM_OK) return st;
    if (adj && nf > 0) {
        const AdjGeom ag{make_div(uint64_t(g->nx)), make_div(uint64_t(g->ny)), uint32_t(g->nz),
                         g->periodic, uint32_t(base), uint32_t(stride)};
        const int64_t blocks = (nf + 255) / 256;
        const XcdMap map = map_of_runs(table ? 3 : 5);
        const dim3 grid{unsigned(virtual_blocks(blocks, map))};
        // Flags, list and rank words that fit the last-level cache are still
        // there; if they do not, the list is kept from displacing the words
        // (54 M cells of a 512^3 box, whole call 1,406 -> 1,221 us, 45.5 M of
        // 384 x 384 x 512 907 -> 807; 30.6 M cells of that box 573, 595 if
        // streamed).
        const bool stream = n_box + n_box / 4 + 4 * nf > int64_t(kCachedBytes);
        if (!table)
            k_adjacency<false><<<grid, dim3(256), 0, s>>>(cell_of, FromIndex{idx}, nf, ag, map, adj);
        else if (stream)
            k_adjacency<true><<<grid, dim3(256), 0, s>>>(cell_of, FromTable{table}, nf, ag, map, adj);
        else
            k_adjacency<false><<<grid, dim3(256), 0, s>>>(cell_of, FromTable{table}, nf, ag, map, adj);
        if (hipGetLastError() != hipSuccess) return LBM_EHIP;
    }
    if (table && index_of) return emit(lex, std::integral_constant<int, kEmitIndex>{});
    return LBM_OK;
}
