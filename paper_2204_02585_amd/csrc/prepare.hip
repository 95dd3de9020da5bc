// Create-time preparation of the position planes: for each plane j a mask of
// the texels whose samples may have sigma > 0, the Chebyshev (L-infinity)
// distance in texels from every texel to the nearest such texel (capped at
// kDistCap), and a record that packs the distance next to the value the
// render kernel reads.
//
// Eq. 4: sigma = sigma^xy sigma^yz sigma^zx vanishes wherever one factor
// does, so a texel is live unless its sigma^j compares equal to zero (NaN
// counts as live).
//
// Eq. 5 (linear decoder): sigma = max(0, W_sigma concat(sigma^j) + b_sigma)
// is evaluated as ((s^xy + s^yz) + s^zx) + b_sigma from per-plane partial
// sums s^j (a chain of fused multiply-adds over the channels of plane j).
// The partial sums are folded here, once, into the records.  A texel of plane
// j is dead when the same expression with the other two partial sums replaced
// by their maxima over the samples that can share this texel (a row or column
// of the other planes) is <= 0: binary32 addition is monotone, so every such
// sample then has a sum <= 0 or NaN, i.e. sigma = 0.
//
// A sample whose plane-j texel has distance D > 0 is empty, and so is every
// sample whose plane-j texel stays within Chebyshev distance D - 1 of it: the
// render kernel leaps over such runs.  L-infinity distance is separable: with
// f(a, b) the distance along row a from column b to the nearest live texel of
// that row, dist(a, b) = min over a' of max(|a - a'|, f(a', b)).  Every pass
// takes the three planes in one launch: one for the rows, one for the columns
// and the packing (Eq. 4); Eq. 5 folds its channels first and builds a grid of
// empty cells beside it.
#include <math.h>

#include "sqn_internal.h"

namespace sqn {
namespace {

__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(_Float16 x) { return static_cast<float>(x); }

// ---- row pass --------------------------------------------------------------

// One workgroup takes 16 rows x 256 columns of a plane.  Its waves turn the
// texels of those columns and of the 256 on either side (a capped distance
// reaches no further) into 64-bit masks, one ballot per 64 texels, and each
// thread then finds the nearest set bit on either side of four neighbouring
// columns in four rows.  Bound by latency: 1.5 KB of masks replaces a sweep
// of one thread along each row, whose 2 n_p dependent, uncoalesced steps took
// 395 us a plane at n_p = 1024; here the three planes take about 9 us.
constexpr int32_t kRowTile = 16;       // rows per workgroup, and per block minimum
constexpr int32_t kColTile = 256;      // columns per workgroup
constexpr int32_t kMaskWords = 12;     // (256 + 256 + 256) / 64
static_assert(kDistCap == 255, "a distance is one byte and reaches at most 255 texels");

int32_t row_pitch(int32_t n_p) { return (n_p + 3) / 4 * 4; }

// Eq. 4 planes: live unless sigma^j == 0.
template <typename ST>
struct ProductLive {
    const ST* plane[3];
    struct Row {
        const ST* p;
    };
    __device__ __forceinline__ Row row(int32_t j, int32_t a, int32_t n_p) const
    {
        const ST* p = j == 0 ? plane[0] : (j == 1 ? plane[1] : plane[2]);
        return {p + static_cast<uint32_t>(a) * static_cast<uint32_t>(n_p)};
    }
    // the two values a texel's test takes, loaded apart from it
    static __device__ __forceinline__ float2 load(const Row& r, int32_t b)
    {
        return make_float2(static_cast<float>(r.p[b]), 0.0f);
    }
    __device__ __forceinline__ bool live(const Row&, int32_t, float2 v) const { return !(v.x == 0.0f); }
};

// Eq. 5 planes (partial sums s, [3][n_p][n_p]).  maxima[2k] / maxima[2k + 1]
// are the row / column maxima of plane k (planes xy = [x][y], yz = [y][z],
// zx = [z][x]); the texel (a, b) of plane j shares samples with
//   xy (x=a, y=b): s^yz over row y, s^zx over column x
//   yz (y=a, z=b): s^xy over column y, s^zx over row z
//   zx (z=a, x=b): s^xy over row x, s^yz over column z
// and the bound keeps the evaluation order ((s^xy + s^yz) + s^zx) + b.
struct LinearLive {
    const float* s;
    const float* maxima;
    float b_sigma;
    struct Row {
        const float *p, *along;   // s of the row; the maxima that follow its columns
        float fixed;              // the maximum of the whole row's other partner
    };
    __device__ __forceinline__ Row row(int32_t j, int32_t a, int32_t n_p) const
    {
        const int32_t along = j == 0 ? 2 : (j == 1 ? 4 : 0), fixed = j == 0 ? 5 : (j == 1 ? 1 : 3);
        return {s + static_cast<size_t>(j) * n_p * n_p + static_cast<size_t>(a) * n_p,
                maxima + static_cast<size_t>(along) * n_p, maxima[static_cast<size_t>(fixed) * n_p + a]};
    }
    static __device__ __forceinline__ float2 load(const Row& r, int32_t b) { return make_float2(r.p[b], r.along[b]); }
    __device__ __forceinline__ bool live(const Row& r, int32_t j, float2 v) const
    {
        const float s_xy = j == 0 ? v.x : (j == 1 ? r.fixed : v.y);
        const float s_yz = j == 0 ? v.y : (j == 1 ? v.x : r.fixed);
        const float s_zx = j == 0 ? r.fixed : (j == 1 ? v.y : v.x);
        float bound = s_xy + s_yz;
        bound = bound + s_zx;
        bound = bound + b_sigma;
        return !(bound <= 0.0f);
    }
};

// f[j][a][b]: distance along row a of plane j from column b to the nearest
// live texel of the row, capped at kDistCap (rows of `pitch` bytes, rows past
// n_p filled with kDistCap up to a multiple of 16); f_min[j][a / 16][b]: its
// minimum over the 16 rows.
template <typename Live>
__global__ __launch_bounds__(256) void row_distance(const Live live, uint8_t* __restrict__ f,
                                                    uint8_t* __restrict__ f_min, int32_t n_p, int32_t pitch)
{
    __shared__ uint64_t mask[kRowTile][kMaskWords];
    __shared__ int32_t beside[kRowTile][4][2];
    __shared__ uint32_t part[4][64];
    const int32_t j = blockIdx.z, c0 = blockIdx.x * kColTile, a0 = blockIdx.y * kRowTile;
    const int32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int32_t q = 0; q < 4; ++q) {
        const int32_t r = 4 * wave + q, a = a0 + r;
        // texels off the plane read its edge and count as empty: loads
        // without branches, so that a row's twelve are in flight together
        const typename Live::Row row = live.row(j, min(a, n_p - 1), n_p);
        float2 v[kMaskWords];
#pragma unroll
        for (int32_t w = 0; w < kMaskWords; ++w)
            v[w] = Live::load(row, min(max(c0 - 256 + 64 * w + lane, 0), n_p - 1));
        uint64_t m = 0;
#pragma unroll
        for (int32_t w = 0; w < kMaskWords; ++w) {
            const int32_t b = c0 - 256 + 64 * w + lane;
            const uint64_t x
                = __builtin_amdgcn_ballot_w64(live.live(row, j, v[w]) & (a < n_p) & (b >= 0) & (b < n_p));
            m = lane == w ? x : m;
        }
        if (lane < kMaskWords)
            mask[r][lane] = m;
    }
    __syncthreads();
    // the nearest live bit before and after each word, relative to its first
    // bit, among the four words on either side
    if (threadIdx.x < 2 * 4 * kRowTile) {
        const int32_t r = threadIdx.x >> 3, w = threadIdx.x & 3, after = (threadIdx.x >> 2) & 1;
        uint64_t x[4];
#pragma unroll
        for (int32_t k = 0; k < 4; ++k)
            x[k] = mask[r][4 + w + (after ? k + 1 : -k - 1)];
        int32_t at = after ? 1 << 20 : -(1 << 20);
#pragma unroll
        for (int32_t k = 3; k >= 0; --k)
            if (x[k] != 0)
                at = after ? __builtin_ctzll(x[k]) + 64 * (k + 1) : 63 - __builtin_clzll(x[k]) - 64 * (k + 1);
        beside[r][w][after] = at;
    }
    __syncthreads();
    const int32_t b = c0 + 4 * lane;
    const int32_t w = lane >> 4, bit = 4 * (lane & 15);
    const size_t rows = static_cast<size_t>((n_p + kRowTile - 1) / kRowTile) * kRowTile;
    uint32_t least[4] = {255u, 255u, 255u, 255u};
#pragma unroll
    for (int32_t q = 0; q < 4; ++q) {
        const int32_t r = 4 * wave + q;
        const uint64_t m = mask[r][4 + w];
        // nearest live bit before and after the four columns, relative to
        // the first of this word
        const uint64_t below = m & ((1ull << bit) - 1ull);
        const uint64_t above = (m >> bit) >> 4;
        int32_t last = below != 0 ? 63 - __builtin_clzll(below) : beside[r][w][0];
        int32_t next = above != 0 ? bit + 4 + __builtin_ctzll(above) : beside[r][w][1];
        uint32_t d[4];
        const uint32_t nib = static_cast<uint32_t>(m >> bit);
#pragma unroll
        for (int32_t i = 0; i < 4; ++i) {
            last = ((nib >> i) & 1u) ? bit + i : last;
            d[i] = static_cast<uint32_t>(min(kDistCap, bit + i - last));
        }
#pragma unroll
        for (int32_t i = 3; i >= 0; --i) {
            next = ((nib >> i) & 1u) ? bit + i : next;
            d[i] = min(d[i], static_cast<uint32_t>(min(kDistCap, next - (bit + i))));
            least[i] = min(least[i], d[i]);
        }
        if (b < pitch)
            *reinterpret_cast<uint32_t*>(f + (j * rows + a0 + r) * pitch + b)
                = d[0] | (d[1] << 8) | (d[2] << 16) | (d[3] << 24);
    }
    part[wave][lane] = least[0] | (least[1] << 8) | (least[2] << 16) | (least[3] << 24);
    __syncthreads();
    if (wave == 0 && b < pitch) {
        uint32_t out = 0;
#pragma unroll
        for (int32_t i = 0; i < 4; ++i) {
            uint32_t v = 255u;
#pragma unroll
            for (int32_t w = 0; w < 4; ++w)
                v = min(v, (part[w][lane] >> (8 * i)) & 255u);
            out |= v << (8 * i);
        }
        *reinterpret_cast<uint32_t*>(f_min + (j * (rows / kRowTile) + blockIdx.y) * pitch + b) = out;
    }
}

// ---- column pass and packing -------------------------------------------------

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef short short2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ ushort2v pair(uint32_t x) { return __builtin_bit_cast(ushort2v, x); }
__device__ __forceinline__ uint32_t word(ushort2v x) { return __builtin_bit_cast(uint32_t, x); }

// blocks of 16 rows on either side that a distance under the cap can reach
// (the nearest row of block k lies at least 16 k - 15 rows off)
constexpr int32_t kReach = (kDistCap + kRowTile - 1) / kRowTile;
constexpr int32_t kNear = 2 * kReach + 1;

struct PackArgs {
    const void* value[3];     // [n_p][n_p] sigma^j (binary16 or binary32) or partial sums
    void* packed[3];
    int32_t quads;            // 1: four values of a row load as one aligned vector
};

// dist(a, b) = min over a' of max(|a - a'|, f(a', b)) and the packed record
// of the texel.  binary16 sigma -> one 32-bit word (sigma bits | dist << 16);
// binary32 sigma -> two words (sigma bits, dist).  Record (a, b) of a plane
// lands at (a & ~3) n_p + 4 b + (a & 3): four rows interleaved, so that a
// 64-byte segment holds a 4 x 4 block of texels (4 x 2 with two-word
// records), which a quad's four samples along a ray share far more often
// than a run of one row (row_part in render.hip); rows are padded to a
// multiple of four.
//
// One thread takes 4 rows x 4 columns, the 64 (128) bytes of one such run of
// records: a row of f serves its sixteen distances with one 4-byte load and
// packed 16-bit minima.  The minima of blocks of 16 rows (f_min) give a first
// bound on the distances and say which blocks' rows can lower it; only those
// are read.  (Reading every block that could lower the distances found so
// far, without the bound, with a wave over 4 rows x 256 columns: 31 us for the
// three planes at n_p = 1024, bound by vector-ALU issue; a wave over 16 rows x
// 64 columns shares more of its blocks: 19 us.  One thread per texel and one
// row per step took 72 us a plane, the packing 6 us more.)
template <typename VT>
__global__ __launch_bounds__(256) void column_pack(const PackArgs A, const uint8_t* __restrict__ f,
                                                   const uint8_t* __restrict__ f_min, int32_t n_p, int32_t pitch)
{
    __shared__ uint32_t near_min[kNear][64];
    const int32_t j = blockIdx.z, tile_b = blockIdx.x;
    // a wave takes the 16 rows of block `home` in 64 columns: lane = strip of
    // four rows x four columns
    const int32_t home = blockIdx.y;
    const int32_t group = 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
    const int32_t a = kRowTile * home + 4 * ((threadIdx.x >> 4) & 3);
    const int32_t b = 4 * (tile_b * 64 + group);
    const int32_t blocks = (n_p + kRowTile - 1) / kRowTile;
    // minima of the blocks a capped distance can reach, edge blocks repeated
    // past the plane: the bounds below walk them from LDS
    const uint8_t* mj = f_min + static_cast<size_t>(j) * blocks * pitch;
    const int32_t bc = min(b, pitch - 4);
    {
        const int32_t c = min(4 * (tile_b * 64 + static_cast<int32_t>(threadIdx.x & 63)), pitch - 4);
#pragma unroll
        for (int32_t i = 0; i < kNear; i += 4) {
            const int32_t k = i + (threadIdx.x >> 6);
            const int32_t blk = min(max(home - kReach + k, 0), blocks - 1);
            if (k < kNear)
                near_min[k][threadIdx.x & 63]
                    = *reinterpret_cast<const uint32_t*>(mj + static_cast<size_t>(blk) * pitch + c);
        }
    }
    // the sixteen values first: they wait for HBM while the distances form
    const VT* value = static_cast<const VT*>(j == 0 ? A.value[0] : (j == 1 ? A.value[1] : A.value[2]));
    VT val[4][4];
    if (A.quads) {
#pragma unroll
        for (int32_t r = 0; r < 4; ++r) {
            typedef VT quad __attribute__((ext_vector_type(4)));
            const quad q = *reinterpret_cast<const quad*>(
                value + static_cast<uint32_t>(min(a + r, n_p - 1)) * static_cast<uint32_t>(n_p) + bc);
#pragma unroll
            for (int32_t i = 0; i < 4; ++i)
                val[r][i] = q[i];
        }
    } else {
#pragma unroll
        for (int32_t r = 0; r < 4; ++r)
#pragma unroll
            for (int32_t i = 0; i < 4; ++i)
                val[r][i] = value[static_cast<uint32_t>(min(a + r, n_p - 1)) * static_cast<uint32_t>(n_p)
                                  + min(b + i, n_p - 1)];
    }
    __syncthreads();
    if (b >= pitch || a >= n_p)
        return;
    const uint8_t* fj = f + static_cast<size_t>(j) * blocks * kRowTile * pitch;
    // minima over the rows of a block, columns 0 and 2, and 1 and 3
    auto minima = [&](int32_t blk, ushort2v& v0, ushort2v& v1) {
        const uint32_t v = near_min[blk - home + kReach][group];
        v0 = pair(v & 0x00ff00ffu);
        v1 = pair((v >> 8) & 0x00ff00ffu);
    };
    // rows between the strip and the nearest row of block home -+ k
    auto below_by = [&](int32_t k) { return a - ((home - k) * kRowTile + kRowTile - 1); };
    auto above_by = [&](int32_t k) { return (home + k) * kRowTile - (a + 3); };
    // First a bound per column: some row of a block has its minimum, so no
    // distance of the strip exceeds max(rows to the far end of the block,
    // minimum).
    ushort2v most0, most1;
    minima(home, most0, most1);
    most0 = __builtin_elementwise_max(most0, pair(0x000f000fu));
    most1 = __builtin_elementwise_max(most1, pair(0x000f000fu));
    int32_t most;
    auto largest = [&]() {
        const ushort2v m = __builtin_elementwise_max(most0, most1);
        most = max(static_cast<int32_t>(m.x), static_cast<int32_t>(m.y));
    };
    auto bound = [&](int32_t blk, int32_t by) {
        ushort2v v0, v1;
        minima(blk, v0, v1);
        const ushort2v kk = pair(static_cast<uint32_t>(by + 18) * 0x00010001u);
        most0 = __builtin_elementwise_min(most0, __builtin_elementwise_max(v0, kk));
        most1 = __builtin_elementwise_min(most1, __builtin_elementwise_max(v1, kk));
    };
    largest();
    for (int32_t k = 1; k <= kReach; ++k) {
        const int32_t down = below_by(k), up = above_by(k);
        if (!((home - k >= 0 && down + 18 < most) || (home + k < blocks && up + 18 < most)))
            break;
        if (home - k >= 0)
            bound(home - k, down);
        if (home + k < blocks)
            bound(home + k, up);
        largest();
    }
    // Then the rows of the blocks that can go below the bounds, nearest
    // first: a block that lies `by` rows off and has minimum v gives no
    // distance under max(by, v).
    ushort2v best[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        best[r][0] = most0;
        best[r][1] = most1;
    }
    auto helps = [&](int32_t blk, int32_t by) {
        ushort2v v0, v1;
        minima(blk, v0, v1);
        const ushort2v kk = pair(static_cast<uint32_t>(max(by, 0)) * 0x00010001u);
        v0 = __builtin_elementwise_max(v0, kk);
        v1 = __builtin_elementwise_max(v1, kk);
        return (v0.x < most0.x) | (v0.y < most0.y) | (v1.x < most1.x) | (v1.y < most1.y);
    };
    // the rows of a block that starts `at` rows from the strip's first one
    auto take = [&](int32_t blk, int32_t at) {
        const uint8_t* p = fj + static_cast<size_t>(blk) * kRowTile * pitch;
        uint32_t v[kRowTile];
#pragma unroll
        for (int32_t i = 0; i < kRowTile; ++i)
            v[i] = *reinterpret_cast<const uint32_t*>(p + static_cast<uint32_t>(i * pitch + b));
        // kk[i - r + 3] = |row i of the block - row r of the strip|
        short2v kk[kRowTile + 3];
#pragma unroll
        for (int32_t i = 0; i < kRowTile + 3; ++i) {
            const short x = static_cast<short>(at + i - 3);
            const short2v d = {x, x};
            kk[i] = __builtin_elementwise_max(d, -d);
        }
#pragma unroll
        for (int32_t i = 0; i < kRowTile; ++i) {
            const ushort2v v0 = pair(v[i] & 0x00ff00ffu), v1 = pair((v[i] >> 8) & 0x00ff00ffu);
#pragma unroll
            for (int32_t r = 0; r < 4; ++r) {
                const ushort2v k = __builtin_bit_cast(ushort2v, kk[i - r + 3]);
                best[r][0] = __builtin_elementwise_min(best[r][0], __builtin_elementwise_max(v0, k));
                best[r][1] = __builtin_elementwise_min(best[r][1], __builtin_elementwise_max(v1, k));
            }
        }
        most0 = __builtin_elementwise_max(__builtin_elementwise_max(best[0][0], best[1][0]),
                                          __builtin_elementwise_max(best[2][0], best[3][0]));
        most1 = __builtin_elementwise_max(__builtin_elementwise_max(best[0][1], best[1][1]),
                                          __builtin_elementwise_max(best[2][1], best[3][1]));
        largest();
    };
    if (helps(home, 0))
        take(home, kRowTile * home - a);
    for (int32_t k = 1; k <= kReach; ++k) {
        const int32_t down = below_by(k), up = above_by(k);
        const bool go_down = home - k >= 0 && down < most, go_up = home + k < blocks && up < most;
        if (!go_down && !go_up)
            break;
        const int32_t ks = __builtin_amdgcn_readfirstlane(k);   // the same in every lane
        if (go_down && helps(home - ks, down))
            take(home - ks, kRowTile * (home - ks) - a);
        if (go_up && helps(home + ks, up))
            take(home + ks, kRowTile * (home + ks) - a);
    }
    void* packed = j == 0 ? A.packed[0] : (j == 1 ? A.packed[1] : A.packed[2]);
#pragma unroll
    for (int32_t i = 0; i < 4; ++i) {
        if (b + i >= n_p)
            break;
        uint32_t dist[4];
#pragma unroll
        for (int32_t r = 0; r < 4; ++r)
            dist[r] = (word(best[r][i & 1]) >> (i >= 2 ? 16 : 0)) & 0xffffu;
        const uint32_t at = static_cast<uint32_t>(a) * static_cast<uint32_t>(n_p) + 4u * (b + i);
        if constexpr (sizeof(VT) == 2) {
            static_cast<uint4*>(packed)[at >> 2] = make_uint4(val[0][i] | (dist[0] << 16), val[1][i] | (dist[1] << 16),
                                                              val[2][i] | (dist[2] << 16), val[3][i] | (dist[3] << 16));
        } else {
            uint4* out = static_cast<uint4*>(packed) + (at >> 1);
            out[0] = make_uint4(val[0][i], dist[0], val[1][i], dist[1]);
            out[1] = make_uint4(val[2][i], dist[2], val[3][i], dist[3]);
        }
    }
}

// Row and column pass over the three planes, `value` of 2 or 4 bytes.
template <typename Live>
hipError_t distance_and_pack(const Live& live, const void* const value[3], bool value16, int32_t n_p,
                             void* const packed[3], const PrepareWork& work, hipStream_t stream)
{
    const int32_t pitch = row_pitch(n_p);
    row_distance<Live><<<dim3((n_p + kColTile - 1) / kColTile, (n_p + kRowTile - 1) / kRowTile, 3), 256, 0, stream>>>(
        live, work.f, work.f_min, n_p, pitch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    PackArgs args;
    args.quads = n_p % 4 == 0;
    for (int j = 0; j < 3; ++j) {
        args.value[j] = value[j];
        args.packed[j] = packed[j];
        args.quads = args.quads && reinterpret_cast<uintptr_t>(value[j]) % (value16 ? 8 : 16) == 0;
    }
    const dim3 grid((pitch / 4 + 63) / 64, (n_p + kRowTile - 1) / kRowTile, 3);
    if (value16)
        column_pack<uint16_t><<<grid, 256, 0, stream>>>(args, work.f, work.f_min, n_p, pitch);
    else
        column_pack<uint32_t><<<grid, 256, 0, stream>>>(args, work.f, work.f_min, n_p, pitch);
    return hipGetLastError();
}

// ---- linear decoder -------------------------------------------------------

struct FoldArgs {
    const void* sigma[3];
    float w[3 * kMaxSigma];   // density weights, plane by plane
};

// Partial sums s[j][a][b] of plane j: an fma chain over the d_sigma channels
// from zero, in channel order (the evaluation order of the density, see the
// file head), with the maxima of 64-texel runs of each row (row_part
// [3][tiles][n_p]) and of 16-texel runs of each column (col_part
// [3][n_p / 16][n_p]).  fmaxf skips NaN, whose samples have zero density
// anyway; an all-NaN run gives -inf.  A wave loads the channels of 64 texels
// of a row as one run and takes them back from LDS, one texel per lane.
template <typename ST>
__global__ __launch_bounds__(256) void fold_partials(const FoldArgs A, int32_t ds, int32_t n_p, float* __restrict__ s,
                                                     float* __restrict__ row_part, float* __restrict__ col_part)
{
    extern __shared__ __align__(16) unsigned char fold_lds[];
    __shared__ float col_lds[4][64];
    const int32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t j = blockIdx.z, c0 = blockIdx.x * 64, a0 = blockIdx.y * kRowTile;
    const int32_t waves = blockDim.x >> 6;
    ST* stage = reinterpret_cast<ST*>(fold_lds) + wave * 64 * ds;
    const ST* sigma = static_cast<const ST*>(j == 0 ? A.sigma[0] : (j == 1 ? A.sigma[1] : A.sigma[2]));
    const float* w = A.w + j * ds;
    const int32_t texels = min(64, n_p - c0), b = c0 + lane;
    const size_t n = static_cast<size_t>(n_p) * n_p;
    float col = -INFINITY;
    for (int32_t r = wave; r < kRowTile; r += waves) {
        const int32_t a = a0 + r;
        if (a >= n_p)
            break;
        const ST* src = sigma + (static_cast<size_t>(a) * n_p + c0) * ds;
        for (int32_t i = lane; i < texels * ds; i += 64)
            stage[i] = src[i];
        // written and read by this wave alone, whose LDS operations complete
        // in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float row = -INFINITY;
        if (lane < texels) {
            float v = 0.0f;
            for (int32_t c = 0; c < ds; ++c)
                v = __builtin_fmaf(w[c], widen(stage[lane * ds + c]), v);
            s[j * n + static_cast<size_t>(a) * n_p + b] = v;
            row = fmaxf(row, v);
            col = fmaxf(col, v);
        }
#pragma unroll
        for (int32_t k = 32; k > 0; k >>= 1)
            row = fmaxf(row, __shfl_xor(row, k));
        if (lane == 0)
            row_part[(static_cast<size_t>(j) * gridDim.x + blockIdx.x) * n_p + a] = row;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    col_lds[wave][lane] = col;
    __syncthreads();
    if (wave == 0 && lane < texels) {
        for (int32_t k = 1; k < waves; ++k)
            col = fmaxf(col, col_lds[k][lane]);
        col_part[(static_cast<size_t>(j) * gridDim.y + blockIdx.y) * n_p + b] = col;
    }
}

// maxima[2j][a] over the row parts, maxima[2j + 1][b] over the column parts
// (blockIdx.y = 2j or 2j + 1).
__global__ void reduce_maxima(const float* __restrict__ row_part, const float* __restrict__ col_part,
                              float* __restrict__ maxima, int32_t n_p, int32_t row_tiles, int32_t col_tiles)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t y = blockIdx.y, j = y >> 1;
    if (i >= n_p)
        return;
    const int32_t tiles = (y & 1) ? col_tiles : row_tiles;
    const float* part = ((y & 1) ? col_part : row_part) + static_cast<size_t>(j) * tiles * n_p + i;
    float m = -INFINITY;
#pragma unroll 8
    for (int32_t k = 0; k < tiles; ++k)
        m = fmaxf(m, part[static_cast<size_t>(k) * n_p]);
    maxima[static_cast<size_t>(y) * n_p + i] = m;
}

// ---- cell grid of the linear decoder ---------------------------------------

// max of s^j over the g x g texels of each cell of plane j = blockIdx.z
// (cells [3][m][m]).
__global__ void cell_max(const float* __restrict__ s, int32_t n_p, int32_t shift, int32_t m, float* __restrict__ out)
{
    const int32_t cb = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t ca = blockIdx.y, j = blockIdx.z;
    if (cb >= m)
        return;
    const float* p = s + static_cast<size_t>(j) * n_p * n_p;
    const int32_t g = 1 << shift;
    const int32_t a1 = min(n_p, (ca + 1) * g), b1 = min(n_p, (cb + 1) * g);
    float mx = -INFINITY;
    for (int32_t a = ca * g; a < a1; ++a)
        for (int32_t b = cb * g; b < b1; ++b)
            mx = fmaxf(mx, p[static_cast<size_t>(a) * n_p + b]);
    out[(static_cast<size_t>(j) * m + ca) * m + cb] = mx;
}

constexpr int32_t kCells = 128;        // most cells per axis
constexpr int32_t kSlabZ = 32;         // cells along z per workgroup
constexpr int32_t kSlabGroups = kSlabZ / 4;
constexpr int32_t kSlabThreads = 1024;   // one item of the pass per thread at m = 128

// Separable Chebyshev pass along the first axis of a slab [m][32] of
// distances in LDS: out(p, z) = min over q of max(|p - q|, slab(q, z)), four
// z per thread; `store` takes the position, the first z (in the slab) and the
// four bytes.
template <typename Store>
__device__ __forceinline__ void slab_pass(const uint32_t* slab, int32_t m, const Store& store)
{
    for (int32_t i = threadIdx.x; i < m * kSlabGroups; i += kSlabThreads) {
        const int32_t p = i / kSlabGroups, g = i % kSlabGroups;
        const uint32_t v = slab[p * kSlabGroups + g];
        ushort2v b0 = pair(v & 0x00ff00ffu), b1 = pair((v >> 8) & 0x00ff00ffu);
        for (int32_t k = 1; k < m; ++k) {
            const ushort2v most = __builtin_elementwise_max(b0, b1);
            if (k >= max(static_cast<int32_t>(most.x), static_cast<int32_t>(most.y)))
                break;
            const ushort2v kk = pair(static_cast<uint32_t>(k) * 0x00010001u);
            // positions off the grid repeat the edge, which is nearer than k
            const uint32_t d = slab[max(p - k, 0) * kSlabGroups + g], u = slab[min(p + k, m - 1) * kSlabGroups + g];
            const ushort2v l0 = __builtin_elementwise_min(pair(d & 0x00ff00ffu), pair(u & 0x00ff00ffu));
            const ushort2v l1 = __builtin_elementwise_min(pair((d >> 8) & 0x00ff00ffu), pair((u >> 8) & 0x00ff00ffu));
            b0 = __builtin_elementwise_min(b0, __builtin_elementwise_max(l0, kk));
            b1 = __builtin_elementwise_min(b1, __builtin_elementwise_max(l1, kk));
        }
        store(p, 4 * g, word(b0) | (word(b1) << 8));
    }
}

// Cells [cx = blockIdx.x][cy][cz], 32 cz from 32 blockIdx.y: live when the
// bound ((M_xy + M_yz) + M_zx) + b is not <= 0; distance along cz from ballots
// (m <= 128: two words per row), then along cy in LDS, to part[cx][cy][cz]
// (rows of 128 bytes; 255: none).  The z range is cut so that the 512
// workgroups of m = 128 fill the chip; each takes its rows' ballots anew,
// which cost little beside the pass.  n_p = 512 (m = 128): 20 us, and 10 us
// for cell_dist_x, where five passes over the 2 M cells took 157 us.
__global__ __launch_bounds__(kSlabThreads) void cell_dist_zy(const float* __restrict__ cmax, int32_t m, float b_sigma,
                                                             uint8_t* __restrict__ part)
{
    __shared__ uint32_t slab[kCells * kSlabGroups];
    const int32_t cx = blockIdx.x, z0 = kSlabZ * blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float* mxy = cmax;
    const float* myz = cmax + m * m;
    const float* mzx = cmax + 2 * m * m;
    uint8_t* bytes = reinterpret_cast<uint8_t*>(slab);
    const float zx0 = mzx[min(lane, m - 1) * m + cx], zx1 = mzx[min(64 + lane, m - 1) * m + cx];
    // the wave's rows cy = wave, wave + 16, ..., all their loads in flight
    constexpr int32_t kRows = kCells / (kSlabThreads / 64);
    float xy[kRows], yz0[kRows], yz1[kRows];
#pragma unroll
    for (int32_t i = 0; i < kRows; ++i) {
        const int32_t cy = min(wave + i * (kSlabThreads / 64), m - 1);
        xy[i] = mxy[cx * m + cy];
        yz0[i] = myz[cy * m + min(lane, m - 1)];
        yz1[i] = myz[cy * m + min(64 + lane, m - 1)];
    }
#pragma unroll
    for (int32_t i = 0; i < kRows; ++i) {
        const int32_t cy = wave + i * (kSlabThreads / 64);
        float bound0 = xy[i] + yz0[i], bound1 = xy[i] + yz1[i];
        bound0 = bound0 + zx0;
        bound1 = bound1 + zx1;
        bound0 = bound0 + b_sigma;
        bound1 = bound1 + b_sigma;
        const uint64_t live0 = __builtin_amdgcn_ballot_w64(!(bound0 <= 0.0f) & (lane < m));
        const uint64_t live1 = __builtin_amdgcn_ballot_w64(!(bound1 <= 0.0f) & (64 + lane < m));
        // lanes 0..31: the slab's z, bit k of word w
        const int32_t w = z0 >> 6, k = (z0 & 63) + (lane & 31);
        const uint64_t own = w == 0 ? live0 : live1;
        const uint64_t upto = own & (~0ull >> (63 - k)), from = own >> k;
        int32_t d = 255;
        if (upto != 0)
            d = k - (63 - __builtin_clzll(upto));
        else if (w == 1 && live0 != 0)
            d = k + 64 - (63 - __builtin_clzll(live0));
        if (from != 0)
            d = min(d, __builtin_ctzll(from));
        else if (w == 0 && live1 != 0)
            d = min(d, 64 - k + __builtin_ctzll(live1));
        if (lane < kSlabZ && cy < m)
            bytes[cy * kSlabZ + lane] = static_cast<uint8_t>(d);
    }
    __syncthreads();
    slab_pass(slab, m, [&](int32_t cy, int32_t z, uint32_t v) {
        *reinterpret_cast<uint32_t*>(part + (static_cast<size_t>(cx) * m + cy) * kCells + z0 + z) = v;
    });
}

// The pass along cx, cy = blockIdx.x: dist[(cx m + cy) m + cz].
__global__ __launch_bounds__(kSlabThreads) void cell_dist_x(const uint8_t* __restrict__ part, int32_t m,
                                                            uint8_t* __restrict__ dist)
{
    __shared__ uint32_t slab[kCells * kSlabGroups];
    const int32_t cy = blockIdx.x, z0 = kSlabZ * blockIdx.y;
    for (int32_t i = threadIdx.x; i < m * kSlabGroups; i += kSlabThreads) {
        const int32_t cx = i / kSlabGroups, g = i % kSlabGroups;
        slab[i] = *reinterpret_cast<const uint32_t*>(part + (static_cast<size_t>(cx) * m + cy) * kCells + z0 + 4 * g);
    }
    __syncthreads();
    slab_pass(slab, m, [&](int32_t cx, int32_t z, uint32_t v) {
        uint8_t* out = dist + (static_cast<size_t>(cx) * m + cy) * m + z0 + z;
        if ((m & 3) == 0) {
            if (z0 + z < m)
                *reinterpret_cast<uint32_t*>(out) = v;
        } else {
            for (int32_t k = 0; k < 4 && z0 + z + k < m; ++k)
                out[k] = static_cast<uint8_t>(v >> (8 * k));
        }
    });
}

}  // namespace

size_t prepare_f_bytes(int32_t n_p)
{
    const size_t rows = static_cast<size_t>((n_p + kRowTile - 1) / kRowTile) * kRowTile;
    return 3 * rows * row_pitch(n_p);
}

size_t prepare_f_min_bytes(int32_t n_p)
{
    return 3 * static_cast<size_t>((n_p + kRowTile - 1) / kRowTile) * row_pitch(n_p);
}

size_t prepare_part_floats(int32_t n_p)
{
    return 3 * (static_cast<size_t>((n_p + 63) / 64) + (n_p + kRowTile - 1) / kRowTile) * n_p;
}

hipError_t prepare_sigma_planes(const void* const sigma[3], int sigma_dtype, int32_t n_p, void* const packed[3],
                                const PrepareWork& work, hipStream_t stream)
{
    if (sigma_dtype == SQN_F16) {
        ProductLive<_Float16> live;
        for (int j = 0; j < 3; ++j)
            live.plane[j] = static_cast<const _Float16*>(sigma[j]);
        return distance_and_pack(live, sigma, true, n_p, packed, work, stream);
    }
    ProductLive<float> live;
    for (int j = 0; j < 3; ++j)
        live.plane[j] = static_cast<const float*>(sigma[j]);
    return distance_and_pack(live, sigma, false, n_p, packed, work, stream);
}

hipError_t prepare_linear_planes(const void* const sigma[3], int sigma_dtype, int32_t n_p, int32_t d_sigma,
                                 const float* w_sigma, float b_sigma, void* const packed[3], int32_t cell_shift, int32_t m,
                                 uint8_t* cell_dist, const PrepareWork& work, hipStream_t stream)
{
    FoldArgs fa;
    for (int j = 0; j < 3; ++j)
        fa.sigma[j] = sigma[j];
    for (int32_t k = 0; k < 3 * d_sigma; ++k)
        fa.w[k] = w_sigma[k];
    const int32_t row_tiles = (n_p + 63) / 64, col_tiles = (n_p + kRowTile - 1) / kRowTile;
    const dim3 tiles(row_tiles, col_tiles, 3);
    float* row_part = work.part;
    float* col_part = work.part + 3 * static_cast<size_t>(row_tiles) * n_p;
    // four waves a workgroup while their channels leave room for others on
    // the compute unit, one (at most 16 KiB) otherwise
    const size_t wave_lds = 64 * static_cast<size_t>(d_sigma) * (sigma_dtype == SQN_F16 ? 2 : 4);
    const uint32_t waves = 4 * wave_lds <= 32768 ? 4 : 1;
    if (sigma_dtype == SQN_F16)
        fold_partials<_Float16><<<tiles, 64 * waves, waves * wave_lds, stream>>>(fa, d_sigma, n_p, work.s, row_part,
                                                                                 col_part);
    else
        fold_partials<float><<<tiles, 64 * waves, waves * wave_lds, stream>>>(fa, d_sigma, n_p, work.s, row_part,
                                                                              col_part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    reduce_maxima<<<dim3((n_p + 255) / 256, 6), 256, 0, stream>>>(row_part, col_part, work.maxima, n_p, row_tiles,
                                                                  col_tiles);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    LinearLive live;
    live.s = work.s;
    live.maxima = work.maxima;
    live.b_sigma = b_sigma;
    const size_t n = static_cast<size_t>(n_p) * n_p;
    const void* const value[3] = {work.s, work.s + n, work.s + 2 * n};
    if ((e = distance_and_pack(live, value, false, n_p, packed, work, stream)) != hipSuccess)
        return e;
    cell_max<<<dim3((m + 63) / 64, m, 3), 64, 0, stream>>>(work.s, n_p, cell_shift, m, work.cell_max);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    cell_dist_zy<<<dim3(m, (m + kSlabZ - 1) / kSlabZ), kSlabThreads, 0, stream>>>(work.cell_max, m, b_sigma, work.cell_part);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    cell_dist_x<<<dim3(m, (m + kSlabZ - 1) / kSlabZ), kSlabThreads, 0, stream>>>(work.cell_part, m, cell_dist);
    return hipGetLastError();
}

}  // namespace sqn
