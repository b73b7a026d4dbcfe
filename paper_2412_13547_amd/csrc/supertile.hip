// Tile-Gaussian pairs in (tile id, depth) order and per-tile ranges (stage
// (b)) in two levels: Gaussians into supertiles of 8 x 8 tiles, then the
// supertiles' lists into the tiles' lists.
//
// The Gaussians come in depth order (stable, so equal depths keep ascending
// index).  A Gaussian's tile rectangle covers few supertiles (6.4 on average
// against 172 tiles at 3M Gaussians on a 120 x 68 tile grid), so the stable
// scatter into them is cheap, and inside a supertile the order of a tile's
// list is the order of the supertile's list restricted to the Gaussians whose
// rectangle holds the tile: a compaction, which a wavefront does with one
// ballot per tile and 64 entries and writes with consecutive stores.
//   1. super_count: per block of 512 consecutive Gaussians and per supertile,
//      how many of them touch it; the block's pairs.  An exclusive scan over
//      (supertile, block) gives every block's first entry in every list; one
//      block of it adds up the pairs (added by every block to one word they
//      took a third of step 1: 39 -> 27 us at 3M Gaussians).
//   2. super_emit: the block's Gaussians of a supertile, a bit each, are those
//      that reach its column and its row of supertiles (a ballot for each
//      column and row, lanes_reaching); the prefix of their population counts
//      is a stable rank.  A Gaussian's entry in the supertile's list is (id,
//      column mask << 24 | row mask) of the tiles it covers.  One more block
//      cuts the lists into chunks of equal length.
//   3. super_tile_count: per chunk, the entries covering each of the 64 tiles.
//   4. super_chunk_scan, super_ranges: every chunk's first place in every
//      tile, every tile's [start, end).
//   5. super_expand: per chunk, one wavefront per tile row keeps the entries
//      of its row and appends their ids to the row's eight tiles.
// The pair count is on the device after 1; above the capacity the later
// kernels write nothing and the ranges come out empty, so no step waits for
// the host.  A list entry holds at least one pair, so a list buffer of the
// pair capacity always fits.
//
// Small views are binned directly instead (direct_kernel).
//
// What bounds it: the 4 bytes written per pair in step 5.  The earlier form
// (rows, then a counting sort by column of 4096-pair slices in LDS; still used
// above kSuperMax supertiles, binning.hip) wrote a run of ~34 pairs per
// column and slice; here a run is a chunk's part of a tile's list.
#include "common.hpp"
#include "wave.hpp"

#include <algorithm>

namespace tgs {
namespace {

constexpr int kSuperWaves = kSuperGauss / 64;
constexpr int kDirectTiles = 16;                           // tiles (wavefronts) per block of the direct binning
constexpr int kChunkMin = 256;                             // entries of the shortest chunk
constexpr int kScanNT = 256, kScanPer = 16;                // table scan
constexpr int kScanBlock = kScanNT * kScanPer;

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t prefix_bits(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
}

// Block-wide exclusive scan, one value per thread.
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t* s_w, uint32_t& total) {
    const int wv = int(threadIdx.x >> 6);
    uint32_t wt;
    const uint32_t ex = wave_exclusive_sum(x, wt);
    if (__lane_id() == 0) s_w[wv] = wt;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
    for (int w = 0; w < NT / 64; ++w) {
        if (w < wv) before += s_w[w];
        total += s_w[w];
    }
    __syncthreads();
    return before + ex;
}

// The supertiles [x0, x1) x [y0, y1) of a tile rectangle; empty for an empty one.
struct SuperRect { int x0, x1, y0, y1; };

__device__ __forceinline__ SuperRect super_rect(const Rect& r) {
    if (r.xlo >= r.xhi || r.ylo >= r.yhi) return SuperRect{0, 0, 0, 0};
    return SuperRect{r.xlo >> 3, (r.xhi + 7) >> 3, r.ylo >> 3, (r.yhi + 7) >> 3};
}

// The tiles [lo, hi) of the 8 of a supertile from tile `first` on, as a bit
// each: rows from bit 0 up, columns from bit 31 down (so that doubling the
// word carries out one column after the other).
__device__ __forceinline__ uint32_t cover_rows(int lo, int hi, int first) {
    return (0xFFu >> (8 - min(hi - first, 8))) & (0xFFu << max(lo - first, 0));
}
__device__ __forceinline__ uint32_t cover_cols(int lo, int hi, int first) {
    return ((0xFFu >> max(lo - first, 0)) & (0xFFu << (8 - min(hi - first, 8)))) << 24;
}

// Per wavefront and supertile column (then row) the lanes whose rectangle
// reaches it, [sx + sy][kSuperWaves]: those reaching supertile (x, y) are the
// intersection of two of these words.  (sx + sy ballots; a bit or a count set
// by atomics per Gaussian and supertile took as long as its largest rectangle.)
// The caller's barrier follows.
__device__ __forceinline__ void lanes_reaching(const SuperRect& q, int sx, int sy, uint64_t* mask) {
    const int wv = int(threadIdx.x >> 6), lane = __lane_id();
    auto fill = [&](int lo, int hi, int count, uint64_t* out) {
        for (int x0 = 0; x0 < count; x0 += 64) {
            uint64_t mine = 0;
            const int top = min(64, count - x0);
            for (int x = 0; x < top; ++x) {
                const uint64_t m = __ballot(lo <= x0 + x && x0 + x < hi);
                if (lane == x) mine = m;
            }
            if (lane < top) out[(x0 + lane) * kSuperWaves + wv] = mine;
        }
    };
    fill(q.x0, q.x1, sx, mask);
    fill(q.y0, q.y1, sy, mask + sx * kSuperWaves);
}

__global__ void __launch_bounds__(kSuperGauss)
super_count_kernel(const uint2* __restrict__ rects, const uint32_t* __restrict__ order, int64_t n,
                   const uint32_t* __restrict__ dcount, int sx, int sy, uint32_t* __restrict__ table,
                   uint2* __restrict__ srect, uint32_t* __restrict__ block_pairs) {
    extern __shared__ uint64_t mask[];
    __shared__ uint32_t s_w[kSuperGauss / 64];
    const int64_t s = int64_t(blockIdx.x) * kSuperGauss + threadIdx.x;
    const uint32_t id = s < n ? order[s] : 0u;                 // (before m arrives)
    const int64_t m = min(n, int64_t(*dcount));
    const uint32_t nb = uint32_t((m + kSuperGauss - 1) / kSuperGauss);
    if (blockIdx.x >= nb) return;
    uint2 packed = make_uint2(0u, 0u);
    if (s < m) {
        packed = rects[id];
        srect[s] = packed;
    }
    const Rect rc = unpack_rect(packed);
    lanes_reaching(super_rect(rc), sx, sy, mask);
    uint32_t total;                                            // < 2^31: 512 rectangles of < 2^22
    (void)block_scan<kSuperGauss>(uint32_t(rc.xhi - rc.xlo) * uint32_t(rc.yhi - rc.ylo), s_w, total);
    if (threadIdx.x == 0) block_pairs[blockIdx.x] = total;
    for (int k = threadIdx.x; k < sx * sy; k += kSuperGauss) {
        const int y = k / sx, x = k - y * sx;
        const uint64_t* mx = mask + x * kSuperWaves;
        const uint64_t* my = mask + (sx + y) * kSuperWaves;
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kSuperWaves; ++w) c += uint32_t(__popcll(mx[w] & my[w]));
        table[uint64_t(k) * nb + blockIdx.x] = c;
    }
}

// Exclusive scan of the table's S * nb words in place (nb known on the
// device): tile sums, then each tile after the sums before it; the total
// follows the last word.
__device__ __forceinline__ uint32_t table_words(int64_t n, const uint32_t* dcount, int S) {
    const int64_t m = min(n, int64_t(*dcount));
    return uint32_t((m + kSuperGauss - 1) / kSuperGauss) * uint32_t(S);
}

__global__ void __launch_bounds__(kScanNT)
super_scan_reduce(const uint32_t* __restrict__ table, int64_t n, const uint32_t* __restrict__ dcount,
                  int S, uint32_t* __restrict__ sums) {
    __shared__ uint32_t s_w[kScanNT / 64];
    const uint32_t count = table_words(n, dcount, S);
    const uint32_t base = blockIdx.x * uint32_t(kScanBlock);
    if (base >= count) return;
    uint32_t v[kScanPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const uint32_t i = base + uint32_t(k) * kScanNT + threadIdx.x;
        v[k] = i < count ? table[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) sum += v[k];
    uint32_t total;
    (void)block_scan<kScanNT>(sum, s_w, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kScanNT)
super_scan_down(uint32_t* __restrict__ table, int64_t n, const uint32_t* __restrict__ dcount, int S,
                const uint32_t* __restrict__ sums, const uint32_t* __restrict__ block_pairs,
                unsigned long long* __restrict__ pairs, uint32_t* __restrict__ pair_count) {
    __shared__ uint32_t s_w[kScanNT / 64];
    if (blockIdx.x == gridDim.x - 1) {                         // one block more: the pair count
        __shared__ unsigned long long s_p[kScanNT / 64];
        const uint32_t nb = table_words(n, dcount, 1);
        unsigned long long p = 0;
        for (uint32_t b = threadIdx.x; b < nb; b += kScanNT) p += block_pairs[b];
        for (int o = 32; o > 0; o >>= 1) p += __shfl_xor(p, o);
        if ((threadIdx.x & 63) == 0) s_p[threadIdx.x >> 6] = p;
        __syncthreads();
        if (threadIdx.x == 0) {
            p = s_p[0] + s_p[1] + s_p[2] + s_p[3];
            *pairs = p;
            *pair_count = uint32_t(min(p, 0xFFFFFFFFull));
        }
        return;
    }
    const uint32_t count = table_words(n, dcount, S);
    const uint32_t base = blockIdx.x * uint32_t(kScanBlock) + threadIdx.x * uint32_t(kScanPer);
    if (blockIdx.x * uint32_t(kScanBlock) >= count) {
        if (count == 0 && blockIdx.x == 0 && threadIdx.x == 0) table[0] = 0u;
        return;
    }
    uint32_t before = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kScanNT) before += sums[b];
    uint32_t v[kScanPer], sum = 0;
    if (base + kScanPer <= count) {                            // (16-byte aligned)
#pragma unroll
        for (int k = 0; k < kScanPer; k += 4) {
            const uint4 w = *reinterpret_cast<const uint4*>(table + base + k);
            v[k] = w.x; v[k + 1] = w.y; v[k + 2] = w.z; v[k + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; ++k) v[k] = base + uint32_t(k) < count ? table[base + k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) sum += v[k];
    uint32_t carry, total;
    (void)block_scan<kScanNT>(before, s_w, carry);
    uint32_t run = carry + block_scan<kScanNT>(sum, s_w, total);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const uint32_t x = v[k];
        v[k] = run;
        run += x;
    }
    if (base + kScanPer <= count) {
#pragma unroll
        for (int k = 0; k < kScanPer; k += 4)
            *reinterpret_cast<uint4*>(table + base + k) = make_uint4(v[k], v[k + 1], v[k + 2], v[k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; ++k)
            if (base + uint32_t(k) < count) table[base + k] = v[k];
    }
    if (threadIdx.x == 0 && blockIdx.x == (count - 1) / kScanBlock) table[count] = carry + total;
}

// Chunks: the lists cut into pieces of one length (a multiple of 64, about
// kChunkTarget pieces in all, none shorter than kChunkMin but a list's last),
// so that steps 3 and 5 have equal pieces whatever the lists' lengths.
// desc[c] = (supertile, first entry, end entry); first[s] the supertile's
// first chunk.  One block.
__device__ void super_setup(const uint32_t* table, uint32_t nb, int S, int gy, bool fits,
                            uint32_t* first, uint4* desc, uint32_t* nchunks, uint32_t* row_total,
                            uint32_t* s_w, uint32_t* lds) {
    const uint32_t tid = threadIdx.x;
    for (int r = int(tid); r < gy; r += kSuperGauss) row_total[r] = 0u;
    constexpr int per = kSuperMax / kSuperGauss;
    uint32_t* s_first = lds;                                   // [S + 1]
    uint32_t* s_start = lds + S + 1;                           // [S + 1] first entry of every list
    const uint32_t total = fits ? table[uint64_t(S) * nb] : 0u;
    const uint32_t len = max(uint32_t(kChunkMin), ((total + kChunkTarget - 1) / kChunkTarget + 63u) & ~63u);
    uint32_t nc[per], sum = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int s = int(tid) * per + k;
        const uint32_t a = fits && s < S ? table[uint64_t(s) * nb] : 0u;
        const uint32_t b = fits && s < S ? table[uint64_t(s + 1) * nb] : 0u;
        if (s < S) s_start[s] = a;
        nc[k] = (b - a + len - 1) / len;
        sum += nc[k];
    }
    uint32_t all;
    uint32_t at = block_scan<kSuperGauss>(sum, s_w, all);
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int s = int(tid) * per + k;
        if (s < S) {
            first[s] = at;
            s_first[s] = at;
        }
        at += nc[k];
    }
    if (tid == 0) {
        s_first[S] = all;
        s_start[S] = total;
    }
    __syncthreads();
    for (uint32_t c = tid; c < all; c += kSuperGauss) {
        int lo = 0, hi = S;                                    // the last s with s_first[s] <= c
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_first[mid] <= c) lo = mid;
            else hi = mid;
        }
        const uint32_t e = s_start[lo] + (c - s_first[lo]) * len;
        desc[c] = make_uint4(uint32_t(lo), e, min(e + len, s_start[lo + 1]), 0u);
    }
    if (tid == 0) {
        first[S] = all;
        *nchunks = all;
    }
}

__global__ void __launch_bounds__(kSuperGauss)
super_emit_kernel(const uint2* __restrict__ srect, const uint32_t* __restrict__ order, int64_t n,
                  const uint32_t* __restrict__ dcount, int sx, int S, int gy, uint32_t capacity,
                  const unsigned long long* __restrict__ pairs, const uint32_t* __restrict__ table,
                  uint2* __restrict__ list, uint32_t* __restrict__ first, uint4* __restrict__ desc,
                  uint32_t* __restrict__ nchunks, uint32_t* __restrict__ row_total) {
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t s_w[kSuperGauss / 64];
    const int tid = int(threadIdx.x);
    const int64_t m = min(n, int64_t(*dcount));
    const uint32_t nb = uint32_t((m + kSuperGauss - 1) / kSuperGauss);
    const bool fits = *pairs <= capacity;
    if (blockIdx.x == 0) {
        super_setup(table, nb, S, gy, fits && m > 0, first, desc, nchunks, row_total, s_w, lds);
        return;
    }
    const uint32_t blk = blockIdx.x - 1;
    if (blk >= nb || !fits) return;                            // block-uniform
    uint2* ent = reinterpret_cast<uint2*>(lds);                // [kSuperGauss] rectangles
    uint32_t* ids = lds + 2 * kSuperGauss;                     // [kSuperGauss]
    uint64_t* mask = reinterpret_cast<uint64_t*>(ids + kSuperGauss);
    const int64_t s = int64_t(blk) * kSuperGauss + tid;
    uint2 packed = make_uint2(0u, 0u);
    uint32_t id = 0;
    if (s < m) {
        packed = srect[s];
        id = order[s];
    }
    // a wavefront takes four supertiles at a time, 16 lanes each and 32
    // Gaussians to a lane (one supertile, 64 lanes and 8 Gaussians, where there
    // are too few for all wavefronts): the lanes list their Gaussians' entries in
    // LDS, and all of them write what is listed, an entry each.  Bound by these
    // instructions; with a thread writing one Gaussian's entries after the other
    // few lanes had any left after the first and each wrote a line of its own:
    // 164 -> 88 us at 3M Gaussians on 510 supertiles, 39 -> 36 on 135, 37 -> 23 at
    // 1M on 240 (3.4 -> 4.1 at 2K on one).
    static_assert(kSuperWaves == 8, "512 Gaussians are 16 words of 32");
    __shared__ uint16_t s_item[kSuperWaves][4 * kSuperGauss];
    __shared__ uint2 s_row[kSuperWaves][4];
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = __lane_id();
    const int rows = S < 4 * kSuperWaves ? 1 : 4;
    const int row = rows == 4 ? lane >> 4 : 0, first_g = (rows * lane & 63) * 8;
    const uint32_t part = rows == 4 ? 0xFFFFFFFFu : 0xFFu;
    const uint32_t* half = reinterpret_cast<const uint32_t*>(mask) + (first_g >> 5);
    uint16_t* item = s_item[wv];
    int k = wv * rows + row;
    uint32_t base = k < S ? table[uint64_t(k) * nb + blk] : 0u;
    ent[tid] = packed;
    ids[tid] = id;
    lanes_reaching(super_rect(unpack_rect(packed)), sx, S / sx, mask);
    __syncthreads();
    for (int k0 = wv * rows; k0 < S; k0 += rows * kSuperWaves) {
        const int next = k + rows * kSuperWaves;
        const uint32_t base_next = next < S ? table[uint64_t(next) * nb + blk] : 0u;
        const int y = k / sx, x = k - y * sx;
        uint32_t w = k < S ? half[x * (2 * kSuperWaves)] & half[(sx + y) * (2 * kSuperWaves)] : 0u;
        w = (w >> (first_g & 31)) & part;
        uint32_t total;
        uint32_t at = wave_exclusive_sum(uint32_t(__popc(w)), total);
        if (first_g == 0) s_row[wv][row] = make_uint2(base - at, uint32_t(y) << 16 | uint32_t(x));
        const uint32_t tag = uint32_t(row) << 9 | uint32_t(first_g);
        while (w != 0u) {
            item[at++] = uint16_t(tag + uint32_t(__builtin_ctz(w)));
            w &= w - 1u;
        }
        wave_sync();
        for (uint32_t e = uint32_t(lane); e < total; e += 64u) {
            const uint32_t it = item[e], g = it & (kSuperGauss - 1);
            const uint2 to = s_row[wv][it >> 9];
            const Rect rc = unpack_rect(ent[g]);
            list[to.x + e] = make_uint2(ids[g], cover_rows(rc.ylo, rc.yhi, 8 * int(to.y >> 16)) |
                                                    cover_cols(rc.xlo, rc.xhi, 8 * int(to.y & 0xFFFFu)));
        }
        wave_sync();
        k = next;
        base = base_next;
    }
}

constexpr uint32_t kCountStage = 2048;

// Per chunk (a wavefront) the entries covering each of the supertile's 64
// tiles: a lane counts its entries in bytes, 4 tiles to a word
// (kCountStage entries at a time, 32 to a lane), and the lanes' bytes
// are summed through LDS.
__global__ void __launch_bounds__(256)
super_tile_count(const uint2* __restrict__ list, const uint4* __restrict__ desc,
                 const uint32_t* __restrict__ nchunks, uint32_t* __restrict__ tcnt) {
    constexpr int kRow = 68;                                   // words: 16-byte rows, no conflicts
    __shared__ __align__(16) uint32_t s_acc[4][16 * kRow];
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = __lane_id();
    const uint32_t c = blockIdx.x * 4u + uint32_t(wv);
    if (c >= *nchunks) return;                                 // wavefront-uniform, no barriers
    const uint4 d = desc[c];
    uint32_t* acc_l = s_acc[wv];
    uint32_t total = 0;
    for (uint32_t e0 = d.y; e0 < d.z; e0 += kCountStage) {
        const uint32_t e1 = min(d.z, e0 + kCountStage);
        uint32_t acc[16] = {};
        auto add = [&](uint32_t mk) {
            // columns 0-3 and 4-7, the first in the top byte
            const uint32_t lo = ((mk >> 28) * 0x00204081u) & 0x01010101u;
            const uint32_t hi = (((mk >> 24) & 15u) * 0x00204081u) & 0x01010101u;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t on = uint32_t(int32_t(mk << (31 - r)) >> 31);   // bit r
                acc[2 * r] += lo & on;
                acc[2 * r + 1] += hi & on;
            }
        };
        uint32_t e = e0 + uint32_t(lane);
        for (; e - uint32_t(lane) + 256u <= e1; e += 256u) {     // four loads in flight
            uint32_t mk[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) mk[u] = list[e + 64u * uint32_t(u)].y;
#pragma unroll
            for (int u = 0; u < 4; ++u) add(mk[u]);
        }
        for (; e < e1; e += 64u) add(list[e].y);
#pragma unroll
        for (int k = 0; k < 16; ++k) acc_l[k * kRow + lane] = acc[k];
        wave_sync();
        const uint32_t* row = acc_l + (lane >> 2) * kRow;
        const uint32_t pick = 1u << (8 * (3 - (lane & 3)));
#pragma unroll
        for (int k = 0; k < 64; k += 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(row + k);
            total = __builtin_amdgcn_udot4(v.x, pick, total, false);
            total = __builtin_amdgcn_udot4(v.y, pick, total, false);
            total = __builtin_amdgcn_udot4(v.z, pick, total, false);
            total = __builtin_amdgcn_udot4(v.w, pick, total, false);
        }
        wave_sync();
    }
    tcnt[uint64_t(c) * 64 + lane] = total;
}

// One block per supertile: the chunks' counts of each tile become the chunk's
// first place in the tile, and the tile's total goes to ranges[2 tile + 1]
// and into its row's.
__global__ void __launch_bounds__(1024)
super_chunk_scan(uint32_t* __restrict__ tcnt, const uint32_t* __restrict__ first, int sx, Grid grid,
                 uint32_t* __restrict__ row_total, uint32_t* __restrict__ ranges) {
    constexpr int kSegs = 16, kLoads = 8;
    __shared__ uint32_t s_seg[kSegs][64];
    const int t = int(threadIdx.x & 63u), g = int(threadIdx.x >> 6);
    const uint32_t f0 = first[blockIdx.x], nc = first[blockIdx.x + 1] - f0;
    const uint32_t seg = (nc + kSegs - 1) / kSegs;
    const uint32_t k0 = min(nc, uint32_t(g) * seg), k1 = min(nc, k0 + seg);
    uint32_t* col = tcnt + uint64_t(f0) * 64 + t;
    uint32_t sum = 0;
    for (uint32_t k = k0; k < k1; k += kLoads) {
        uint32_t v[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) v[q] = col[uint64_t(min(k + q, k1 - 1)) * 64];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) sum += k + q < k1 ? v[q] : 0u;
    }
    s_seg[g][t] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
    for (int q = 0; q < kSegs; ++q) {
        const uint32_t v = s_seg[q][t];
        if (q < g) run += v;
        total += v;
    }
    for (uint32_t k = k0; k < k1; k += kLoads) {
        uint32_t v[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) v[q] = col[uint64_t(min(k + q, k1 - 1)) * 64];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            if (k + q < k1) col[uint64_t(k + q) * 64] = run;
            run += k + q < k1 ? v[q] : 0u;
        }
    }
    if (g != 0) return;
    const int tx = (int(blockIdx.x) % sx) * 8 + (t & 7), ty = (int(blockIdx.x) / sx) * 8 + (t >> 3);
    if (tx < grid.gx && ty < grid.gy) {
        ranges[2 * (uint64_t(ty) * grid.gx + tx) + 1] = total;
    } else {
        total = 0;                                             // (no rectangle reaches it)
    }
    for (int o = 4; o > 0; o >>= 1) total += uint32_t(__shfl_xor(int(total), o));
    if ((t & 7) == 0 && ty < grid.gy && total) atomicAdd(&row_total[ty], total);
}

// One block per tile row: the tiles' totals to [start, end) (0, 0 for an
// empty tile; all empty when the pairs overflow the capacity).
__global__ void __launch_bounds__(256)
super_ranges(const uint32_t* __restrict__ row_total, const unsigned long long* __restrict__ pairs,
             uint32_t capacity, Grid grid, uint32_t* __restrict__ ranges) {
    __shared__ uint32_t s_w[4];
    const bool fits = *pairs <= capacity;
    uint32_t sum = 0, start;
    for (uint32_t r = threadIdx.x; r < blockIdx.x; r += 256u) sum += row_total[r];
    (void)block_scan<256>(sum, s_w, start);
    for (int x0 = 0; x0 < grid.gx; x0 += 256) {
        const int x = x0 + int(threadIdx.x);
        const uint64_t tile = uint64_t(blockIdx.x) * grid.gx + x;
        const uint32_t c = fits && x < grid.gx ? ranges[2 * tile + 1] : 0u;
        uint32_t all;
        const uint32_t at = start + block_scan<256>(c, s_w, all);
        if (x < grid.gx) {
            ranges[2 * tile] = c ? at : 0u;
            ranges[2 * tile + 1] = c ? at + c : 0u;
        }
        start += all;
    }
}

constexpr int kExpandStage = 1024;                         // entries staged at once

// One block per chunk, one wavefront per tile row of its supertile: the chunk
// is staged in LDS (a wavefront that loaded from memory between its stores
// would wait for the stores too); of each 64 entries, those of the row are
// kept in a second list in LDS; each 64 of these are appended to the row's
// eight tiles, a ballot per tile giving every lane its place.  Each tile's
// open line of 64 places is a register, a lane per place: the ids are moved
// to their places' lanes (a lane permutation), and a line is written when it
// is complete, by one store.  Consecutive chunks (which share the lines at
// the ends of their runs) go to one XCD.
//
// Bound by the stores and, close behind, by the instructions per tile and 64
// entries (9 vector, 9 scalar).  In this order 256-byte lines written whole
// reach 5.5 TB/s, the same bytes in stores that split lines 3.5 (a plain fill:
// 6.9).  Storing each tile's ids where they come took 264 us at 3M Gaussians
// on a 3840 x 2160 view at stride 2 (237 M pairs) and 1160 us at stride 1
// (886 M); whole lines take 240 and 920 us.  Measured and set aside: rings of
// ids in LDS instead of the permutation (249-271, 906-925 us), a lane per tile
// walking the entries (282, 985), every wavefront loading its own entries (289, 921).
__global__ void __launch_bounds__(512)
super_expand(const uint2* __restrict__ list, const uint4* __restrict__ desc,
             const uint32_t* __restrict__ nchunks, const uint32_t* __restrict__ tcnt,
             const uint32_t* __restrict__ ranges, int sx, Grid grid, uint32_t* __restrict__ out) {
    __shared__ uint2 s_in[kExpandStage];
    __shared__ uint2 s_kept[8][128];
    const uint32_t nc = *nchunks;
    const uint32_t per = (nc + 7u) / 8u;
    const uint32_t c = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per || c >= nc) return;           // block-uniform
    const int r = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const uint32_t lane = uint32_t(__lane_id());
    const uint4 d = desc[c];
    const int ty = (int(d.x) / sx) * 8 + r, tx = (int(d.x) % sx) * 8;
    // the eight tiles' next places
    uint32_t place = 0;
    if (lane < 8 && tx + int(lane) < grid.gx && ty < grid.gy)
        place = ranges[2 * (uint64_t(ty) * grid.gx + tx + lane)] + tcnt[uint64_t(c) * 64 + r * 8 + lane];
    // per tile: the line of 64 places that is open and the next place in it
    // (scalars), and the line's ids, a lane per place
    uint32_t line[8], off[8], skip[8], pend[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t p = uint32_t(__builtin_amdgcn_readlane(int(place), k));
        line[k] = p & ~63u;
        off[k] = skip[k] = p & 63u;
        pend[k] = 0;
    }
    const uint32_t nl4 = ~lane << 2;
    uint2* kept = s_kept[r];
    uint32_t have = 0;                                         // entries in `kept` (< 64 between steps)
    auto append = [&](uint2 v) {                               // v.y: no column for no entry
        uint32_t x[8], n[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint64_t m = __ballot((v.y & (0x80000000u >> k)) != 0);
            // lanes with an entry to the places' lanes, the others downwards from there
            const uint32_t to = (prefix_bits(m) << 2) + (__builtin_amdgcn_inverse_ballot_w64(m) ? 0u : nl4) + (off[k] << 2);
            x[k] = uint32_t(__builtin_amdgcn_ds_permute(int(to), int(v.x)));
            n[k] = uint32_t(__builtin_popcountll(m));
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t y = __builtin_amdgcn_inverse_ballot_w64(~uint64_t(0) << off[k]) ? x[k] : pend[k];
            pend[k] = y;
            off[k] += n[k];
            if (off[k] >= 64u) {                               // the line is complete
                // (the places before this chunk's first are another's)
                if (lane >= skip[k]) (out + line[k])[lane] = y;
                skip[k] = 0u;
                line[k] += 64u;
                off[k] -= 64u;
                pend[k] = x[k];
            }
        }
    };
    const uint32_t bit = 1u << r;
    for (uint32_t e0 = d.y; e0 < d.z; e0 += uint32_t(kExpandStage)) {
        const uint32_t cnt = min(uint32_t(kExpandStage), d.z - e0);
        if (e0 != d.y) __syncthreads();
#pragma unroll
        for (int u = 0; u < kExpandStage / 512; ++u) {
            const uint32_t i = threadIdx.x + 512u * uint32_t(u);
            s_in[i] = i < cnt ? list[e0 + i] : make_uint2(0u, 0u);
        }
        __syncthreads();
        // (a row outside the grid has no entries)
        for (uint32_t e = 0; e < cnt; e += 64u) {
            const uint2 v = s_in[e + lane];
            const bool on = (v.y & bit) != 0;
            const uint64_t m = __ballot(on);
            if (on) kept[have + prefix_bits(m)] = v;
            have += uint32_t(__builtin_popcountll(m));
            wave_sync();
            if (have >= 64u) {
                const uint2 now = kept[lane], rest = kept[64 + lane];
                wave_sync();
                have -= 64u;
                kept[lane] = rest;                             // (of which `have` are entries)
                append(now);
            }
        }
    }
    wave_sync();
    if (have) append(lane < have ? kept[lane] : make_uint2(0u, 0u));
#pragma unroll
    for (int k = 0; k < 8; ++k)                                // the open lines
        if (lane >= skip[k] && lane < off[k]) (out + line[k])[lane] = pend[k];
}

size_t mask_lds_bytes(int sx, int sy) { return size_t(sx + sy) * kSuperWaves * 8; }

// (of which the block that cuts the chunks takes two words per supertile)
size_t emit_lds_bytes(int sx, int sy) {
    return std::max(kSuperGauss * 12 + mask_lds_bytes(sx, sy), size_t(sx * sy + 1) * 8);
}

// The direct binning of small views: a wavefront per tile and part of the depth
// order looks at the part's rectangles, staged in LDS for the block's 16 tiles,
// and a ballot per 64 of them gives the tile's, in order.  Once to count (a word
// per tile and part), then, after a scan of these words by one block, once
// more to write the ids to their places and the ranges.  Small views are bound
// by their launches: three here where the two levels take seven.
template <bool EMIT>
__global__ void __launch_bounds__(1024)
direct_kernel(const uint2* __restrict__ rects, const uint32_t* __restrict__ order, int64_t n,
              const uint32_t* __restrict__ dcount, Grid grid, uint32_t capacity, uint32_t* table,
              uint32_t* __restrict__ ranges, uint32_t* __restrict__ out) {
    __shared__ uint2 s_rect[1024];
    __shared__ uint32_t s_id[EMIT ? 1024 : 1];
    const int64_t m = min(n, int64_t(*dcount));
    const uint32_t tiles = uint32_t(grid.num_tiles()), parts = gridDim.y, part = blockIdx.y;
    const int64_t per = ((m + parts - 1) / parts + 63) / 64 * 64;
    const int64_t first = min(m, per * part), last = min(m, first + per);
    const int tid = int(threadIdx.x), lane = __lane_id();
    const uint32_t tile = blockIdx.x * uint32_t(kDirectTiles) +
                          uint32_t(__builtin_amdgcn_readfirstlane(tid >> 6));
    const bool mine = tile < tiles;                            // (wavefront-uniform)
    uint32_t at = 0;
    if constexpr (EMIT) {
        const uint32_t total = table[tiles * parts];
        const bool fits = total <= capacity;
        if (mine && part == 0 && lane == 0) {
            const uint32_t b = table[tile * parts], e = table[(tile + 1) * parts];
            ranges[2 * tile] = fits && e > b ? b : 0u;
            ranges[2 * tile + 1] = fits && e > b ? e : 0u;
        }
        if (!fits) return;                                     // block-uniform
        at = mine ? table[tile * parts + part] : 0u;
    }
    const int tx = int(tile % uint32_t(grid.gx)), ty = int(tile / uint32_t(grid.gx));
    for (int64_t s0 = first; s0 < last; s0 += 1024) {
        const int cnt = int(min(int64_t(1024), last - s0));
        if (s0 != first) __syncthreads();
        if (tid < cnt) {
            const uint32_t id = order[s0 + tid];
            s_rect[tid] = rects[id];
            if constexpr (EMIT) s_id[tid] = id;
        }
        __syncthreads();
        if (!mine) continue;
        for (int k = 0; k < cnt; k += 64) {
            const Rect r = unpack_rect(s_rect[k + lane]);
            const bool in = k + lane < cnt && tx >= r.xlo && tx < r.xhi && ty >= r.ylo && ty < r.yhi;
            const uint64_t b = __ballot(in);
            if constexpr (EMIT)
                if (in) out[at + prefix_bits(b)] = s_id[k + lane];
            at += uint32_t(__builtin_popcountll(b));
        }
    }
    if constexpr (!EMIT)
        if (mine && lane == 0) table[tile * parts + part] = at;
}

__global__ void __launch_bounds__(1024)
direct_scan_kernel(uint32_t* __restrict__ table, uint32_t words, unsigned long long* __restrict__ pairs,
                   uint32_t* __restrict__ pair_count) {
    constexpr int kPer = 16;
    __shared__ uint32_t s_w[16];
    const uint32_t base = threadIdx.x * uint32_t(kPer);
    uint32_t v[kPer], sum = 0, total;
    if (base + kPer <= words) {                                // (16-byte aligned)
#pragma unroll
        for (int k = 0; k < kPer; k += 4) {
            const uint4 w = *reinterpret_cast<const uint4*>(table + base + k);
            v[k] = w.x; v[k + 1] = w.y; v[k + 2] = w.z; v[k + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k) v[k] = base + uint32_t(k) < words ? table[base + k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) sum += v[k];
    uint32_t run = block_scan<1024>(sum, s_w, total);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t x = v[k];
        v[k] = run;
        run += x;
    }
    if (base + kPer <= words) {
#pragma unroll
        for (int k = 0; k < kPer; k += 4)
            *reinterpret_cast<uint4*>(table + base + k) = make_uint4(v[k], v[k + 1], v[k + 2], v[k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (base + uint32_t(k) < words) table[base + k] = v[k];
    }
    if (threadIdx.x == 0) {
        table[words] = total;
        *pairs = total;
        *pair_count = total;
    }
}

uint64_t super_blocks(int64_t n) { return (uint64_t(n) + kSuperGauss - 1) / kSuperGauss; }

}  // namespace

hipError_t prepare_supertile_kernels() {
    // (the most for kSuperMax supertiles in a row)
    auto allow = [](const void* f, size_t bytes) {
        return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
    };
    hipError_t e = allow(reinterpret_cast<const void*>(&super_count_kernel), mask_lds_bytes(kSuperMax, 1));
    if (e != hipSuccess) return e;
    return allow(reinterpret_cast<const void*>(&super_emit_kernel), emit_lds_bytes(kSuperMax, 1));
}

uint64_t super_max_chunks(uint64_t capacity, int supers) {
    return std::min<uint64_t>(kChunkTarget, capacity / kChunkMin + 1) + uint64_t(supers);
}

// Few enough Gaussians and tiles for every tile to look at every Gaussian that
// has tiles.  The whole bin/sort (us, in two levels / directly) by tests, with
// 57 % of the Gaussians in view and with all of them:
//   tiles        16 M                      32 M                       64 M
//      64   78 / 67    93 / 79     99 / 87   119 / 111     135 / 132   177 / 188
//     169   66 / 61    74 / 72     73 / 74    87 / 94       88 / 102   107 / 138
//    1024   62 / 55    66 / 64     64 / 64    68 / 81       67 / 84     73 / 114
//    4096   41 / 32    44 / 38     55 / 51    56 / 67       66 / 79     68 / 108
//   15876   44 / 34    47 / 39     47 / 43    51 / 53       53 / 58     53 / 81
// (1.9 M on 16 tiles, 31 M tests: 207 / 146 and 295 / 197).  How many are in view
// is not known when the launches are chosen: at 32 M both cost the same for 57 %
// (and the direct binning up to 13 us more where all are).
constexpr uint64_t kDirectTests = 32'000'000;
constexpr int64_t kDirectWords = 16 * 1024;                // words the one-block scan takes

int direct_parts(int64_t n, const Grid& grid) {
    const int64_t tiles = grid.num_tiles();
    if (n <= 0 || tiles <= 0 || tiles > kDirectWords || uint64_t(n) > kDirectTests / uint64_t(tiles)) return 0;
    // parts of the depth order: about 512 blocks in all, at least 1024 Gaussians each
    const int64_t groups = (tiles + kDirectTiles - 1) / kDirectTiles;
    return int(std::max<int64_t>(1, std::min({512 / groups, kDirectWords / tiles, (n + 1023) / 1024})));
}

uint64_t super_layout(SuperLayout& L, uint64_t at, int64_t n, uint64_t cap, const Grid& grid) {
    L = SuperLayout{};
    L.sx = (grid.gx + 7) / 8;
    const int64_t S = int64_t(L.sx) * ((grid.gy + 7) / 8);
    if (S > kSuperMax) return 0;
    L.supers = int(S);
    L.max_chunks = super_max_chunks(cap, L.supers);
    const uint64_t words = super_blocks(n) * uint64_t(S);
    if (words >= 0xFFFF0000ull) return 0;                      // (the table scan is 32-bit)
    uint64_t o = at;
    auto take = [&](uint64_t bytes) {
        const uint64_t a = o;
        o = align_up(o + bytes, 256);
        return a;
    };
    L.list = take(cap * 8);
    L.table = take((words + 1) * 4);
    L.sums = take((words / kScanBlock + 1) * 4);
    L.first = take((uint64_t(S) + 1) * 4);
    L.desc = take(L.max_chunks * 16);
    L.nchunks = take(4);
    L.row_total = take(uint64_t(grid.gy) * 4);
    L.tcnt = take(L.max_chunks * 256);
    // (its table begins where the lists do)
    L.direct = direct_parts(n, grid);
    if ((uint64_t(L.direct) * uint64_t(grid.num_tiles()) + 1) * 4 > o - at) L.direct = 0;
    return o - at;
}

hipError_t launch_super_counts(uint8_t* ws, const Layout& L, const uint32_t* order, int64_t n,
                               const uint32_t* dcount, unsigned long long* pairs, const Grid& grid,
                               hipStream_t s) {
    const SuperLayout& q = L.super;
    uint32_t* pair_count = reinterpret_cast<uint32_t*>(ws + L.row_start) + grid.gy;
    if (q.direct) {
        const uint32_t tiles = uint32_t(grid.num_tiles()), parts = uint32_t(q.direct);
        auto* table = reinterpret_cast<uint32_t*>(ws + q.list);
        direct_kernel<false><<<dim3((tiles + kDirectTiles - 1) / kDirectTiles, parts), dim3(1024), 0, s>>>(
            reinterpret_cast<const uint2*>(ws + L.rects), order, n, dcount, grid, 0u, table, nullptr,
            nullptr);
        direct_scan_kernel<<<1, 1024, 0, s>>>(table, tiles * parts, pairs, pair_count);
        return hipGetLastError();
    }
    const unsigned nb = unsigned(super_blocks(n));
    if (nb == 0) return fill_u32(pair_count, 0u, 1, s);
    auto u32 = [&](uint64_t off) { return reinterpret_cast<uint32_t*>(ws + off); };
    uint32_t* block_pairs = u32(L.depth_key[1]);               // (the sort is done with it)
    super_count_kernel<<<dim3(nb), dim3(kSuperGauss), mask_lds_bytes(q.sx, q.supers / q.sx), s>>>(
        reinterpret_cast<const uint2*>(ws + L.rects), order, n, dcount, q.sx, q.supers / q.sx,
        u32(q.table), reinterpret_cast<uint2*>(ws + L.srect), block_pairs);
    const unsigned scan_blocks = unsigned(uint64_t(nb) * uint64_t(q.supers) / kScanBlock + 1);
    if (scan_blocks > 1)                                       // (else no tile is before another)
        super_scan_reduce<<<dim3(scan_blocks), dim3(kScanNT), 0, s>>>(u32(q.table), n, dcount,
                                                                     q.supers, u32(q.sums));
    super_scan_down<<<dim3(scan_blocks + 1), dim3(kScanNT), 0, s>>>(
        u32(q.table), n, dcount, q.supers, u32(q.sums), block_pairs, pairs, pair_count);
    return hipGetLastError();
}

hipError_t launch_super_lists(uint8_t* ws, const Layout& L, const uint32_t* order, int64_t n,
                              const uint32_t* dcount, const unsigned long long* pairs,
                              const Grid& grid, uint32_t capacity, hipStream_t s) {
    const SuperLayout& q = L.super;
    auto u32 = [&](uint64_t off) { return reinterpret_cast<uint32_t*>(ws + off); };
    auto* list = reinterpret_cast<uint2*>(ws + q.list);
    auto* desc = reinterpret_cast<uint4*>(ws + q.desc);
    if (q.direct) {
        const uint32_t tiles = uint32_t(grid.num_tiles()), parts = uint32_t(q.direct);
        direct_kernel<true><<<dim3((tiles + kDirectTiles - 1) / kDirectTiles, parts), dim3(1024), 0, s>>>(
            reinterpret_cast<const uint2*>(ws + L.rects), order, n, dcount, grid, capacity,
            u32(q.list), u32(L.ranges), u32(L.pair_vals));
        return hipGetLastError();
    }
    const uint64_t nb = super_blocks(n);
    super_emit_kernel<<<dim3(unsigned(nb + 1)), dim3(kSuperGauss), emit_lds_bytes(q.sx, q.supers / q.sx), s>>>(
        reinterpret_cast<const uint2*>(ws + L.srect), order, n, dcount, q.sx, q.supers, grid.gy,
        capacity, pairs, u32(q.table), list, u32(q.first), desc, u32(q.nchunks), u32(q.row_total));
    const unsigned chunks = unsigned(q.max_chunks);
    super_tile_count<<<dim3((chunks + 3) / 4), dim3(256), 0, s>>>(list, desc, u32(q.nchunks),
                                                                 u32(q.tcnt));
    super_chunk_scan<<<dim3(unsigned(q.supers)), dim3(1024), 0, s>>>(
        u32(q.tcnt), u32(q.first), q.sx, grid, u32(q.row_total), u32(L.ranges));
    super_ranges<<<dim3(unsigned(grid.gy)), dim3(256), 0, s>>>(u32(q.row_total), pairs, capacity,
                                                              grid, u32(L.ranges));
    super_expand<<<dim3((chunks + 7) / 8 * 8), dim3(512), 0, s>>>(
        list, desc, u32(q.nchunks), u32(q.tcnt), u32(L.ranges), q.sx, grid, u32(L.pair_vals));
    return hipGetLastError();
}

}  // namespace tgs
