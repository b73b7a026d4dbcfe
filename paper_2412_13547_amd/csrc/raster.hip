// Dilated compositing, forward and backward (stages (c) and (d1)), and the
// L1 loss gradient.
//
// One workgroup per tile of a DOWNSAMPLED image (Sec. 4.1: pairs live in the
// downsampled grid; each downsampled pixel is blended at its full-resolution
// position d i + o, so no thread is spent on an unrendered pixel).  One launch
// covers the tiles of up to kMaxViews views (a view table passed by value):
// workgroups are laid out view after view, so a batch of views of uneven size
// is balanced by the hardware dispatcher like one big image, and within a
// view they take the tiles heaviest first (the schedule below).  A thread has
// 1, 2 or 4 pixels (Shape), fewer where a launch has few tiles.  The tile's list
// is staged through LDS B splat records at a time (the forward at one pixel per
// thread: by each wavefront for itself); every pixel walks it front to back (Sec. 3 Eq. 2), and the backward from its last
// blended entry back to the first, with the forward's arithmetic and decisions
// (one shared inline routine).
//
// Both kernels are bound by vector instructions per visited (entry,
// wavefront): on a 3840 x 2160 view of 3M Gaussians at stride 1 the backward
// issued one per four cycles and SIMD.  What keeps their number down:
//  - decisions are lane masks in scalar registers, so that combining them is
//    scalar work (kept as bools they were moved through vector registers at
//    every branch);
//  - tests that cannot matter are left out under uniform branches
//    (splat_plain; in the backward also entries before every pixel's last);
//  - the backward sums a lane's pixels by columns and rows, applies the
//    splat's constants to those sums, and takes dL/do as the sum of dL/dpower
//    over o; a stopped pixel of the forward needs no test of its own.
// Forward 172 -> 156 us and backward 344 -> 273 us at stride 2 of that view,
// 456 -> 415 and 1070 -> 870 us at stride 1 (145 vector instructions and 8
// transcendental ones to an entry and wavefront of 4 pixels a lane in the
// backward, 176 before).
#include "common.hpp"
#include "wave.hpp"

#include <type_traits>

namespace tgs {
namespace {

constexpr float kAlphaMax = 0.99f;
constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kTMin = 1e-4f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Splat constants as staged in LDS.  The conic is pre-scaled so that the
// exponent comes out in base 2 with no extra multiply:
//   qa = -A log2(e) / 2,  qb = -B log2(e),  qc = -C log2(e) / 2,
//   log2(e) * power = dx (qa dx + qb dy) + qc dy dy,   dx = u - X, dy = v - Y.
// ga = (u, v, qa, qb), gb = (qc, o, r, g).
__device__ __forceinline__ void stage_conic(const float4 r0, const float4 r1, float4& ga,
                                            float4& gb) {
    constexpr float kHalf = -0.5f * kLog2e, kFull = -kLog2e;
    ga = make_float4(r0.x, r0.y, r0.z * kHalf, r0.w * kFull);
    gb = make_float4(r1.x * kHalf, r1.y, r1.z, r1.w);
}

// alpha = min(0.99, o 2^(log2e power)); false if the entry is skipped
// (power > 0 or alpha < 1/255; o G >= 1/255 is the same test since
// 0.99 > 1/255).  G, alpha and the partial t = qb dy are
// computed either way (branch-free callers select on the result).  Forward
// and backward evaluate exactly these operations (explicit FMAs, no
// contraction elsewhere), so they take bit-identical decisions.
// The two halves: the exponent, then the test on it.
__device__ __forceinline__ float splat_exponent(const float4 ga, const float4 gb, float X,
                                                float Y, float& dx, float& dy, float& t) {
    dx = ga.x - X;
    dy = ga.y - Y;
    t = ga.w * dy;
    return fmaf(dx, fmaf(ga.z, dx, t), (gb.x * dy) * dy);
}

// Decisions are kept as masks over the wavefront's lanes, in scalar registers:
// combining them costs no vector instruction, and one that differs between
// the two sides of a uniform branch stays a mask.
__device__ __forceinline__ bool lane_of(uint64_t mask) {
    return __builtin_amdgcn_inverse_ballot_w64(mask);
}

// The tests of the lanes' pixels k (every lane of the wavefront takes part);
// `plain` (uniform): the splat is splat_plain.  clamped: o G > 0.99.
template <int NP>
__device__ __forceinline__ void splat_test(float o, bool plain, const float* p2, float* alpha,
                                           uint64_t* hit, uint64_t* clamped) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        alpha[k] = o * __builtin_amdgcn_exp2f(p2[k]);
        hit[k] = __ballot(alpha[k] >= kAlphaMin);
        clamped[k] = 0;
    }
    if (!plain) {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            hit[k] &= __ballot(p2[k] <= 0.0f);
            clamped[k] = __ballot(alpha[k] > kAlphaMax);
            alpha[k] = __builtin_amdgcn_fmed3f(alpha[k], 0.0f, kAlphaMax);   // min(0.99, o G) for o G >= 0
        }
    }
}

// A uniform LDS byte offset in a vector register, shared by all the reads of
// an entry (their arrays lie at constant distances).
__device__ __forceinline__ uint32_t entry_offset(int e) {
    uint32_t at = uint32_t(e) * 16u;
    asm("" : "+v"(at));
    return at;
}

__device__ __forceinline__ float4 entry_part(const float4* base, uint32_t at) {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(base) + at);
}

// The number of lanes below this one in the mask.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u));
}

// LDS written by lanes of this wavefront is read by others of it.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One pixel a lane (views of few tiles): a wavefront's time is a chain of
// entries, so what an entry waits for counts, and there are registers to
// spare.  The entries it visits stand in LDS, and it takes them in pairs,
// without a branch: the constants of one pair are read while the other is
// blended, and the two entries of a pair fill each other's latencies.  A visited
// entry takes ~230 cycles in the forward and ~480 in the backward; scanning its
// bits entry by entry, with the reads waited for and the tests under branches,
// they took 390 and 750.  The forward's wavefronts also work by themselves
// (raster_fwd_px1_kernel); the backward's share their sums in LDS, so they
// list their entries of what the block has staged (a backward by wavefronts,
// adding to grad2d entry by entry: 103 -> 80 us at 468 tiles, but 158 -> 194 at
// 2040).  412 x 274 pixels of 200K Gaussians (468 tiles): forward 94 -> 55 us,
// backward 140 -> 103; 128 x 128 of 2K (64): 24.6 -> 17 and 39 -> 28; 960 x 540 of
// 3M (2040): 100 -> 80 and 158 -> 159.  With two pixels a lane there are more
// wavefronts than that and the longer code gains nothing (102 -> 102 and
// 170 -> 187 at 3600 tiles).
constexpr int kListStep = 4;                           // entries from one look at the pixels to the next
constexpr int kListPad = 8;                            // entries past the end that a step may read
struct EntryPair {
    float4 a[2], b[2], c[2];
    uint32_t at[2];                                    // LDS offsets
    // entries i and i + 1 of the list the lanes hold
    template <class E>
    __device__ __forceinline__ void load(const E& s_e, uint32_t list, uint32_t i) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            at[u] = uint32_t(__builtin_amdgcn_readlane(int(list), int(i) + u));
            uint32_t v = at[u];
            asm("" : "+v"(v));
            a[u] = entry_part(s_e[0], v);
            b[u] = entry_part(s_e[1], v);
            c[u] = entry_part(s_e[2], v);
        }
    }
};

// A splat whose exponent is never positive and whose alpha never reaches the
// clamp at any pixel, rounding included: the tests for both can be left out.
// The form's smaller eigenvalue is at least (4 qa qc - qb^2) / (4 (|qa| +
// |qc|)) and the exponent's rounding error at most 3.6e-7 (|qa| + |qc|) (dx^2
// + dy^2), a sixth of what the comparison asks for; o 2^p2 stays below 0.99.
__device__ __forceinline__ bool splat_plain(const float4 ga, const float4 gb) {
    const float qa = ga.z, qb = ga.w, qc = gb.x, tr = qa + qc;
    return qa < 0.0f && qc < 0.0f && 4.0f * qa * qc - qb * qb > 1e-5f * (tr * tr) && gb.y < 0.9899f;
}

// Exponent below which o 2^p2 < 1/255 for certain: log2(1/255 / o) less a
// margin (1/64 in log2, i.e. 1.1 % of alpha) far above the rounding of the
// exponential, the product and this logarithm.  An entry whose exponent is
// below it at every live pixel of a wavefront is skipped by the whole
// wavefront: it would be skipped by each pixel anyway (o <= 0 gives NaN or
// +inf here, and no exponent passes).
constexpr float kSkipMargin = 1.0f / 64.0f;
constexpr float kLog2AlphaMin = -7.99435343685885793f;          // log2(1/255)
__device__ __forceinline__ float skip_threshold(float o) {
    return kLog2AlphaMin - __builtin_amdgcn_logf(o) - kSkipMargin;
}

// Launch shape (the work split): a T x T tile is covered by (T/PX) x (T/PY)
// threads owning PX x PY pixels each (PPT = PX PY = 1, 2 or 4); each LDS
// read of a splat then serves PPT pixels.
// Each wavefront covers an 8 x 8 block of threads, so its pixels form a
// compact square whose walks end at similar depths (a wavefront iterates
// until its last pixel saturates).
template <int T, int PPT>
struct Shape {
    static constexpr int PX = PPT >= 2 ? 2 : 1, PY = PPT == 4 ? 2 : 1, NP = PX * PY;
    static constexpr int TX = T / PX, TY = T / PY, NT = TX * TY;   // threads
    static_assert(TX % 8 == 0 && TY % 8 == 0, "threads must tile into 8 x 8 wavefronts");
    // thread -> (column, row) of its first pixel within the tile
    __device__ static int px(int tid) { return ((tid >> 6) % (TX / 8) * 8 + (tid & 7)) * PX; }
    __device__ static int py(int tid) { return ((tid >> 6) / (TX / 8) * 8 + ((tid >> 3) & 7)) * PY; }
};

// The pixel rectangles of a tile's wavefronts, in full-resolution coordinates
// of their pixel centres (pixels past the image edge included): wavefront w
// covers x in [x0 + w_x step, x0 + w_x step + span], w_x = w mod (TX / 8),
// and likewise in y.
template <class S>
struct WaveRects {
    static constexpr int NW = S::NT / 64, WX = S::TX / 8;
    float x0, y0, stepx, stepy, spanx, spany;
    __device__ void init(const Grid& g, int tx, int ty, int T) {
        auto u = [](float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); };
        x0 = u(float(g.stride * tx * T + g.off_x));
        y0 = u(float(g.stride * ty * T + g.off_y));
        stepx = float(g.stride * 8 * S::PX);
        stepy = float(g.stride * 8 * S::PY);
        spanx = float(g.stride * (8 * S::PX - 1));
        spany = float(g.stride * (8 * S::PY - 1));
    }
};

// Whether the splat's exponent may reach thr somewhere on the rectangle
// [xa, xa + spanx] x [ya, ya + spany]: the maximum of the (negative definite)
// quadratic form over it -- 0 if it holds the centre, else the largest of the
// four edge maxima -- plus a margin (1/32 in log2 and a relative bound on the
// rounding of the form's terms) against thr.  False is a promise that no pixel
// of the rectangle passes the per-pixel test, so its wavefront skips the entry
// without evaluating it; a form that is not negative definite (`shaped`) may
// reach anything.
struct Reach {
    float ka, kc;            // maximising dx on a line dy = e: ka e; dy on a line dx = d: kc d
    bool shaped;
    __device__ Reach(const float4 ga, float qc) {
        shaped = ga.z < 0.0f && qc < 0.0f && 4.0f * ga.z * qc > ga.w * ga.w;
        // (the hardware's reciprocals: a maximum is flat, so their last bit moves
        // it by far less than the margin)
        ka = -ga.w * __builtin_amdgcn_rcpf(2.0f * ga.z);
        kc = -ga.w * __builtin_amdgcn_rcpf(2.0f * qc);
    }
    __device__ bool operator()(const float4 ga, float qc, float thr, float xa, float ya, float spanx,
                               float spany) const {
        const float qa = ga.z, qb = ga.w;
        const float d0 = ga.x - (xa + spanx), d1 = ga.x - xa;    // d0 <= d1
        const float e0 = ga.y - (ya + spany), e1 = ga.y - ya;
        auto f = [&](float d, float e) { return fmaf(d, fmaf(qa, d, qb * e), (qc * e) * e); };
        float m;
        if (d0 <= 0.0f && d1 >= 0.0f && e0 <= 0.0f && e1 >= 0.0f) {
            m = 0.0f;
        } else {
            m = f(d0, fminf(fmaxf(kc * d0, e0), e1));
            m = fmaxf(m, f(d1, fminf(fmaxf(kc * d1, e0), e1)));
            m = fmaxf(m, f(fminf(fmaxf(ka * e0, d0), d1), e0));
            m = fmaxf(m, f(fminf(fmaxf(ka * e1, d0), d1), e1));
            const float dm = fmaxf(-d0, d1), em = fmaxf(-e0, e1);
            const float mag = fmaf(-qa * dm, dm, fmaf(fabsf(qb) * dm, em, (-qc * em) * em));
            m += 1.0f / 32.0f + 4e-6f * mag;
        }
        return m >= thr;
    }
};

// The wavefronts whose rectangle it may reach, a bit each.
template <class S>
__device__ __forceinline__ uint32_t wave_mask(const float4 ga, float qc, float thr,
                                              const WaveRects<S>& wr) {
    constexpr int NW = WaveRects<S>::NW;
    const Reach reach(ga, qc);
    if (!reach.shaped) return NW >= 32 ? 0xFFFFFFFFu : (1u << NW) - 1u;
    uint32_t mask = 0;
#pragma unroll 1
    for (int w = 0; w < NW; ++w) {
        const float xa = wr.x0 + float(w % WaveRects<S>::WX) * wr.stepx;
        const float ya = wr.y0 + float(w / WaveRects<S>::WX) * wr.stepy;
        if (reach(ga, qc, thr, xa, ya, wr.spanx, wr.spany)) mask |= 1u << w;
    }
    return mask;
}

// Which view workgroup b works on, and its index within the view: the
// views' workgroups are laid out one view after the other (the index is the
// tile itself unless the view carries a tile order).  A table of one view needs
// no search: its fields are read at once where the others wait for the index
// (arguments are read from host memory, ~1 us a dependent read).
template <class Table>
__device__ __forceinline__ bool locate(const Table& vt, uint32_t b, int& v, int64_t& tile) {
    v = 0;
    if constexpr (Table::kViews == 1) {
        if (b >= vt.first_block[1]) return false;
    } else {
        if (b >= vt.first_block[vt.count]) return false;
        while (b >= vt.first_block[v + 1]) ++v;
    }
    tile = int64_t(b - vt.first_block[v]);
    return true;
}

// Clamp a tile's range to the pairs that exist: a view whose binning
// overflowed its capacity reports a pair count above it and renders nothing.
// The bounds are made wave-uniform (scalar registers).
__device__ __forceinline__ void tile_range(const RasterView& rv, int64_t tile, uint32_t& start,
                                           uint32_t& end) {
    const uint32_t pc = *rv.pair_count;
    const uint32_t lim = pc <= rv.capacity ? pc : 0u;
    const uint32_t e = min(rv.ranges[2 * tile + 1], lim);
    const uint32_t s = min(rv.ranges[2 * tile], e);
    start = uint32_t(__builtin_amdgcn_readfirstlane(int(s)));
    end = uint32_t(__builtin_amdgcn_readfirstlane(int(e)));
}

// a + b after exchanging the upper 32 lanes of a with the lower 32 of b:
// lanes 0-31 get a[i] + a[i+32], lanes 32-63 get b[i-32] + b[i].
__device__ __forceinline__ float swap32_add(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same between rows of 16 lanes: rows 0 and 2 get a[row] + a[row + 1],
// rows 1 and 3 get b[row - 1] + b[row].
__device__ __forceinline__ float swap16_add(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sums of 9 per-lane values over the wavefront.  Eight of them go through a
// transposing butterfly -- each exchange halves the values a lane keeps: the
// upper half-wave keeps values 4-7, the odd rows keep the upper two of the
// remaining four, the upper 8 lanes of a row the second one -- and end with
// a sum over the 8 lanes of each octet (row mirror, half mirror, quad swaps),
// so lane 8c (c = 0..7) returns the total of value c.  Value 8 is summed
// within each row of 16 and then across the rows, and lane 63 returns its
// total.
__device__ __forceinline__ float wave_sum9(const float* v) {
    const int lane = __lane_id();
    float w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = swap32_add(v[k], v[k + 4]);
    const float x0 = swap16_add(w[0], w[2]);
    const float x1 = swap16_add(w[1], w[3]);
    const bool h8 = lane & 8;
    const float send = h8 ? x0 : x1;
    float y = (h8 ? x1 : x0) + dpp_f<kDppRowMirror>(send);
    float z = v[8] + dpp_f<kDppQuadXor1>(v[8]);
    y += dpp_f<kDppRowHalfMirror>(y);
    z += dpp_f<kDppQuadXor2>(z);
    y += dpp_f<kDppQuadXor2>(y);
    z += dpp_f<kDppRowHalfMirror>(z);
    y += dpp_f<kDppQuadXor1>(y);
    z += dpp_f<kDppRowMirror>(z);
    // rows 1 and 3 add the last lane of the row before, then rows 2 and 3 that
    // of row 1 (the other rows keep z; the nops cover the DPP hazard)
    asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf"
        : "+v"(z));
    return lane == 63 ? z : y;
}

// The sums over a lane's pixels of dp, dp dx, dp dy, dp dx^2, dp dx dy and
// dp dy^2 (in gv[5], gv[0], gv[1], gv[2], gv[3], gv[4]).  The pixels are PX x
// PY, so dx takes one value per column and dy one per row: summing dp over
// the columns and rows first takes 21 operations for 2 x 2 pixels where
// pixel by pixel takes 34.
template <class S>
__device__ __forceinline__ void lane_moments(const float* dp, const float* dx, const float* dy,
                                             float* gv) {
    if constexpr (S::NP == 1) {
        const float x = dp[0] * dx[0], y = dp[0] * dy[0];
        gv[0] = x;
        gv[1] = y;
        gv[2] = x * dx[0];
        gv[3] = x * dy[0];
        gv[4] = y * dy[0];
        gv[5] = dp[0];
    } else if constexpr (S::NP == 2) {                 // one row of two pixels
        const float x0 = dp[0] * dx[0], x1 = dp[1] * dx[1], s = dp[0] + dp[1];
        const float y = s * dy[0];
        gv[0] = x0 + x1;
        gv[1] = y;
        gv[2] = fmaf(x1, dx[1], x0 * dx[0]);
        gv[3] = gv[0] * dy[0];
        gv[4] = y * dy[0];
        gv[5] = s;
    } else {                                           // pixels 0, 1 above 2, 3
        const float cA = dp[0] + dp[2], cB = dp[1] + dp[3];
        const float rA = dp[0] + dp[1], rB = dp[2] + dp[3];
        const float xA = cA * dx[0], xB = cB * dx[1], yA = rA * dy[0], yB = rB * dy[2];
        gv[0] = xA + xB;
        gv[1] = yA + yB;
        gv[2] = fmaf(xB, dx[1], xA * dx[0]);
        gv[4] = fmaf(yB, dy[2], yA * dy[0]);
        const float mA = fmaf(dp[2], dy[2], dp[0] * dy[0]), mB = fmaf(dp[3], dy[2], dp[1] * dy[0]);
        gv[3] = fmaf(mB, dx[1], mA * dx[0]);
        gv[5] = rA + rB;
    }
}

// Every pixel's final transmittance and the 1-based index of its last
// blended entry go to the workspace for the backward.  COUNTS adds the
// per-pixel counters n_eval, n_blend and n_tested.
//
// A pixel's state is its transmittance with a sign: positive while it
// still takes entries, negated (the magnitude kept) once it has stopped or
// when it lies outside the image.  Live transmittance never drops below
// the floor kTMin > 0, so the sign is never ambiguous, and no per-pixel
// flag has to be carried from entry to entry.
template <int T, int PPT, int BATCH, bool COUNTS>
__global__ void __launch_bounds__((Shape<T, PPT>::NT)) __attribute__((amdgpu_waves_per_eu(8)))
raster_fwd_kernel(RasterViews vt) {
    using S = Shape<T, PPT>;
    // splat constants ga, gb and blue, at one stride so one address serves all
    __shared__ float4 s_e[3][BATCH];
    // wavefronts that look at it; bit 31: splat_plain
    __shared__ uint32_t s_m[BATCH];
    int v;
    int64_t tile;
    if (!locate(vt, blockIdx.x, v, tile)) return;                // block-uniform
    const RasterView& rv = vt.v[v];
    const Grid& grid = rv.grid;
    if (rv.order)                                                // heaviest tiles first
        tile = __builtin_amdgcn_readfirstlane(
            int(min(rv.order[tile], uint32_t(grid.num_tiles() - 1))));
    const int tid = threadIdx.x;
    const int tx = int(tile % grid.gx), ty = int(tile / grid.gx);
    const int i0 = tx * T + S::px(tid), j0 = ty * T + S::py(tid);
    const uint32_t inf_colour = *rv.inf_colour;                  // (on its way with the range)
    uint32_t start, end;
    tile_range(rv, tile, start, end);
    const uint32_t every = __builtin_amdgcn_readfirstlane(int(inf_colour)) == 0 ? 3u : 0u;
    WaveRects<S> wr;
    wr.init(grid, tx, ty, T);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float X[S::NP], Y[S::NP], Ts[S::NP], c0[S::NP], c1[S::NP], c2[S::NP];
    uint32_t last[S::NP], neval[S::NP], nblend[S::NP], ntest[S::NP];
#pragma unroll
    for (int k = 0; k < S::NP; ++k) {
        const int i = i0 + k % S::PX, j = j0 + k / S::PX;
        X[k] = float(grid.stride * i + grid.off_x);
        Y[k] = float(grid.stride * j + grid.off_y);
        Ts[k] = i < grid.w_ds && j < grid.h_ds ? 1.0f : -1.0f;
        c0[k] = c1[k] = c2[k] = 0.0f;
        last[k] = 0;
        nblend[k] = 0;
        ntest[k] = 0;
        neval[k] = end - start;
    }
    auto live = [&]() {
        bool l = false;
#pragma unroll
        for (int k = 0; k < S::NP; ++k) l = l || Ts[k] > 0.0f;
        return l;
    };
    uint32_t base = start;
    for (; base < end; base += BATCH) {
        if (__syncthreads_count(live()) == 0) break;
        const int cnt = min(BATCH, int(end - base));
        for (int q = tid; q < cnt; q += S::NT) {
            const uint32_t id = rv.vals[base + q];
            const float4* r = rv.rec + 3 * uint64_t(id);
            const float4 r1 = r[1];
            float4 ga, gb;
            stage_conic(r[0], r1, ga, gb);
            const float thr = skip_threshold(r1.y);
            s_e[0][q] = ga;
            s_e[1][q] = gb;
            s_e[2][q] = make_float4(r[2].x, 0.0f, 0.0f, 0.0f);
            s_m[q] = wave_mask<S>(ga, gb.x, thr, wr) | (splat_plain(ga, gb) ? 1u << 31 : 0u);
        }
        __syncthreads();
        // branch-free per entry: a skipped entry adds exactly 0 and leaves T
        // (entries no pixel of the wavefront can reach are not visited).  A
        // stopped pixel's negative T makes every hit stop it again.
        auto entry = [&](int e, bool plain) {
            if constexpr (COUNTS) {
#pragma unroll
                for (int k = 0; k < S::NP; ++k) ntest[k] += Ts[k] > 0.0f ? 1u : 0u;
            }
            const uint32_t at = entry_offset(e);
            const float4 a = entry_part(s_e[0], at), b = entry_part(s_e[1], at);
            const float bb = entry_part(s_e[2], at).x;
            float dx[S::NP], dy[S::NP], t[S::NP], p2[S::NP], alpha[S::NP];
            uint64_t hit[S::NP], clamped[S::NP], any = 0;
#pragma unroll
            for (int k = 0; k < S::NP; ++k) p2[k] = splat_exponent(a, b, X[k], Y[k], dx[k], dy[k], t[k]);
            splat_test<S::NP>(b.y, plain, p2, alpha, hit, clamped);
            const uint32_t pos = base - start + uint32_t(e) + 1;
#pragma unroll
            for (int k = 0; k < S::NP; ++k) {
                const float w0 = alpha[k] * Ts[k];
                // T after this entry below the floor: the pixel stops here;
                // otherwise it blends (one comparison: stop implies hit)
                const uint64_t stop = hit[k] & __ballot(Ts[k] - w0 < kTMin);
                const uint64_t blend = hit[k] ^ stop;
                const float w = lane_of(blend) ? w0 : 0.0f;
                c0[k] = fmaf(b.z, w, c0[k]);
                c1[k] = fmaf(b.w, w, c1[k]);
                c2[k] = fmaf(bb, w, c2[k]);
                const float tn = Ts[k] - w;           // Ts itself when not blending
                if constexpr (COUNTS) {
                    nblend[k] += lane_of(blend) ? 1u : 0u;
                    neval[k] = lane_of(stop) && Ts[k] > 0.0f ? pos : neval[k];
                }
                Ts[k] = lane_of(stop) ? -fabsf(tn) : tn;
                last[k] = lane_of(blend) ? pos : last[k];
                any |= blend;
            }
            return any != 0;
        };
        // the entries of the batch whose wavefront mask has this wavefront's
        // bit, in order, while some pixel takes entries (looked at every four:
        // entries after every pixel has stopped change nothing, as long as the
        // colours are finite): each 64 entries' bits become one ballot, and the
        // wavefront visits the set bits only, so an entry its rectangle cannot
        // reach costs nothing.
        // Per 64 entries it also collects the bits of those some pixel of
        // this wavefront blended: they are all the backward has to visit.
        for (int c = 0; c < cnt; c += 64) {
            const int q = c + __lane_id();
            const uint32_t mq = q < cnt ? s_m[q] : 0u;
            uint64_t m = __ballot((mq >> wave) & 1u);
            const uint64_t other = m & ~__ballot(mq >> 31);
            uint64_t bm = 0;
            bool go = __ballot(live()) != 0;
            for (uint32_t u = 1; m != 0 && go; ++u) {
                const int j = int(__builtin_ctzll(m));
                m &= m - 1;
                if (entry(c + j, ((other >> j) & 1u) == 0)) bm |= uint64_t(1) << j;
                if ((u & every) == 0u) go = __ballot(live()) != 0;
            }
            if (__lane_id() == 0)                    // entry base + c is chunk (base - start + c) / 64
                rv.bits[uint64_t(wave) * rv.bits_stride + (start >> 6) + uint64_t(tile) +
                        (base - start + uint32_t(c)) / 64u] = bm;
        }
    }
    // the tile's weight for the backward's schedule; the work split the
    // blend bits were written with (one workgroup of the view records it)
    if (rv.work && tid == 0) rv.work[tile] = min(base, end) - start;
    if (tid == 0 && blockIdx.x == vt.first_block[v]) *rv.fwd_split = uint32_t(PPT);
    const uint64_t pix = uint64_t(grid.w_ds) * grid.h_ds;
#pragma unroll
    for (int k = 0; k < S::NP; ++k) {
        const int i = i0 + k % S::PX, j = j0 + k / S::PX;
        if (!(i < grid.w_ds && j < grid.h_ds)) continue;
        const uint64_t p = uint64_t(j) * grid.w_ds + i;
        const float Tr = fabsf(Ts[k]);
        if (rv.image) {
            rv.image[p] = fmaf(Tr, rv.bg[0], c0[k]);
            rv.image[pix + p] = fmaf(Tr, rv.bg[1], c1[k]);
            rv.image[2 * pix + p] = fmaf(Tr, rv.bg[2], c2[k]);
        }
        // what the backward starts from
        rv.ws_tfinal[p] = Tr;
        rv.ws_last[p] = last[k];
        if (rv.t_final) rv.t_final[p] = Tr;
        if (rv.last_contrib) rv.last_contrib[p] = last[k];
        if constexpr (COUNTS) {
            if (rv.n_eval) rv.n_eval[p] = neval[k];
            if (rv.n_blend) rv.n_blend[p] = nblend[k];
            if (rv.n_tested) rv.n_tested[p] = ntest[k];
        }
    }
}

// The forward with one pixel a lane.  A wavefront works by itself: it looks at
// 64 entries of the list at a time, a lane each, keeps those that may reach its
// 8 x 8 pixels in its own part of LDS, and blends what it has kept once that
// is kFlush entries, in pairs, with the next entries' records on their way.
// (Wavefronts that stage entries together wait for the slowest of them at
// every round: 70 us at 468 tiles, 55 without.  6 wavefronts to a SIMD: with 8
// its registers spill, 63 and 99 us at 468 and 2040 tiles against 56 and 82.)
constexpr int kFlush = 48, kKept = kFlush + 64 + kListPad, kPending = 8;

template <int T, bool COUNTS, class Table>
__global__ void __launch_bounds__(T * T) __attribute__((amdgpu_waves_per_eu(6)))
raster_fwd_px1_kernel(Table vt) {
    using S = Shape<T, 1>;
    constexpr int NW = S::NT / 64;
    // per kept entry ga, gb and (blue, 1-based place in the list)
    __shared__ float4 s_a[NW][kKept], s_b[NW][kKept];
    __shared__ float2 s_c[NW][kKept];
    __shared__ uint32_t s_walked[NW];
    int v;
    int64_t tile;
    if (!locate(vt, blockIdx.x, v, tile)) return;                // block-uniform
    const RasterView& rv = vt.v[v];
    const Grid& grid = rv.grid;
    if (rv.order)                                                // heaviest tiles first
        tile = __builtin_amdgcn_readfirstlane(
            int(min(rv.order[tile], uint32_t(grid.num_tiles() - 1))));
    const int tid = threadIdx.x, lane = __lane_id();
    const int tx = int(tile % grid.gx), ty = int(tile / grid.gx);
    const int i = tx * T + S::px(tid), j = ty * T + S::py(tid);
    const uint32_t inf_colour = *rv.inf_colour;                  // (on its way with the range)
    uint32_t start, end;
    tile_range(rv, tile, start, end);
    const uint32_t len = end - start;
    WaveRects<S> wr;
    wr.init(grid, tx, ty, T);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float xa = wr.x0 + float(wave % WaveRects<S>::WX) * wr.stepx;
    const float ya = wr.y0 + float(wave / WaveRects<S>::WX) * wr.stepy;
    const float X = float(grid.stride * i + grid.off_x), Y = float(grid.stride * j + grid.off_y);
    const bool in = i < grid.w_ds && j < grid.h_ds;
    float Ts = in ? 1.0f : -1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    uint32_t last = 0, neval = len, nblend = 0, ntest = 0;
    float4* const ka = s_a[wave];
    float4* const kb = s_b[wave];
    float2* const kc = s_c[wave];

    struct Pair {
        float4 a[2], b[2];
        float2 c[2];
    };
    auto load = [&](Pair& g, uint32_t e) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            g.a[u] = ka[e + u];
            g.b[u] = kb[e + u];
            g.c[u] = kc[e + u];
        }
    };
    // two entries (or one), with the arithmetic of the kernel above: alpha is 0
    // where an entry is skipped, so that one comparison with the floor decides (a
    // live T is at least the floor, a stopped one negative: a skipped entry keeps
    // either).  `bit` in the result: the first is blended by some pixel; the
    // bit above it, the second.
    auto blend = [&](auto count, const Pair& g, uint64_t bit) {
        constexpr int U = decltype(count)::value;
        float alpha[2];
        uint64_t hit[2], clamped;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float dx, dy, t;
            const float p2 = splat_exponent(g.a[u], g.b[u], X, Y, dx, dy, t);
            splat_test<1>(g.b[u].y, false, &p2, alpha + u, hit + u, &clamped);
            alpha[u] = lane_of(hit[u]) ? alpha[u] : 0.0f;
        }
        uint64_t blended = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t pos = __float_as_uint(g.c[u].y);      // 0: an entry of zeros
            if constexpr (COUNTS) ntest += pos != 0u && Ts > 0.0f ? 1u : 0u;
            const float w0 = alpha[u] * Ts;
            const float tn = Ts - w0;
            const bool stops = tn < kTMin;
            const uint64_t blend = hit[u] & ~__ballot(stops);
            if constexpr (COUNTS) {
                nblend += lane_of(blend) ? 1u : 0u;
                neval = stops && Ts > 0.0f ? pos : neval;
            }
            const float w = stops ? 0.0f : w0;
            Ts = stops ? -fabsf(Ts) : tn;
            c0 = fmaf(g.b[u].z, w, c0);
            c1 = fmaf(g.b[u].w, w, c1);
            c2 = fmaf(g.c[u].x, w, c2);
            last = lane_of(blend) ? pos : last;
            blended |= blend != 0 ? bit << u : 0;
        }
        return blended;
    };

    // records a look ahead, their indices two
    float4 n0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), n1 = n0;
    float n2 = 0.0f;
    uint32_t nid = 0;
    auto fetch = [&](uint32_t q) {                               // entry q, whose index is nid
        if (q < len) {
            const float4* r = rv.rec + 3 * uint64_t(nid);
            n0 = r[0];
            n1 = r[1];
            n2 = r[2].x;
        }
        if (q + 64u < len) nid = rv.vals[start + q + 64u];
    };
    if (uint32_t(lane) < len) nid = rv.vals[start + uint32_t(lane)];
    fetch(uint32_t(lane));
    const bool finite = __builtin_amdgcn_readfirstlane(int(inf_colour)) == 0;
    uint32_t have = 0, pending = 0, at = 0;                      // (uniform)
    uint64_t picked = 0;                                         // lane p: who kept in the p-th look pending
    bool go = __ballot(Ts > 0.0f) != 0;
    while (at < len && go) {
        const uint32_t q = at + uint32_t(lane);
        bool keep = false;
        float4 ga, gb;
        stage_conic(n0, n1, ga, gb);
        if (q < len) {
            const Reach reach(ga, gb.x);
            keep = !reach.shaped || reach(ga, gb.x, skip_threshold(n1.y), xa, ya, wr.spanx, wr.spany);
        }
        const uint64_t m = __ballot(keep);
        if (keep) {
            const uint32_t e = have + lanes_below(m);
            ka[e] = ga;
            kb[e] = gb;
            kc[e] = make_float2(n2, __uint_as_float(q + 1u));
        }
        fetch(q + 64u);
        have += uint32_t(__builtin_popcountll(m));
        picked = uint32_t(lane) == pending ? m : picked;
        ++pending;
        at += 64u;
        if (have < uint32_t(kFlush) && pending < uint32_t(kPending) && at < len) continue;
        // blend what is kept, looking at every fourth entry whether some pixel
        // still takes any
        if (lane < kListPad) {
            ka[have + lane] = kb[have + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            kc[have + lane] = make_float2(0.0f, 0.0f);
        }
        wave_lds_sync();
        uint64_t bm[2] = {0, 0};
        constexpr std::integral_constant<int, 1> one{};
        constexpr std::integral_constant<int, 2> two{};
#pragma unroll 1
        for (uint32_t b0 = 0; b0 < have && go; b0 += 64u) {
            const uint32_t top = min(have, b0 + 64u);
            uint64_t word = 0, bit = 1;
            Pair g0, g1;
            if (__builtin_expect(finite, 1)) {
                load(g0, b0);
                for (uint32_t e = b0; e < top && go; e += uint32_t(kListStep)) {
                    load(g1, e + 2u);
                    word |= blend(two, g0, bit);
                    load(g0, e + uint32_t(kListStep));
                    word |= blend(two, g1, bit << 2);
                    bit <<= kListStep;
                    go = __ballot(Ts > 0.0f) != 0;
                }
            } else {                                             // (every entry looked after)
                for (uint32_t e = b0; e < top && go; ++e, bit <<= 1) {
                    load(g0, e);
                    word |= blend(one, g0, bit);
                    go = __ballot(Ts > 0.0f) != 0;
                }
            }
            if (b0 == 0) bm[0] = word;
            else bm[1] = word;
        }
        wave_lds_sync();
        // the looks' blend bits, one word each
        uint64_t out = 0;
        uint32_t before = 0;
        for (uint32_t p = 0; p < pending; ++p) {
            const uint64_t pm = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(picked), int(p)))) |
                                uint64_t(uint32_t(__builtin_amdgcn_readlane(int(picked >> 32), int(p)))) << 32;
            const uint32_t e = before + lanes_below(pm);
            const uint64_t word = e < 64u ? bm[0] >> e : bm[1] >> (e - 64u);
            const uint64_t b = __ballot(lane_of(pm) && (word & 1u) != 0);
            out = uint32_t(lane) == p ? b : out;
            before += uint32_t(__builtin_popcountll(pm));
        }
        if (uint32_t(lane) < pending)
            rv.bits[uint64_t(wave) * rv.bits_stride + (start >> 6) + uint64_t(tile) + (at / 64u - pending) + lane] = out;
        have = pending = 0;
    }
    // the tile's weight for the schedule: the most any wavefront walked
    if (lane == 0) s_walked[wave] = min(at, len);
    __syncthreads();
    if (tid == 0) {
        uint32_t walked = 0;
        for (int w = 0; w < NW; ++w) walked = max(walked, s_walked[w]);
        if (rv.work) rv.work[tile] = walked;
        if (blockIdx.x == vt.first_block[v]) *rv.fwd_split = 1u;
    }
    if (!in) return;
    const uint64_t pix = uint64_t(grid.w_ds) * grid.h_ds;
    const uint64_t p = uint64_t(j) * grid.w_ds + i;
    const float Tr = fabsf(Ts);
    if (rv.image) {
        rv.image[p] = fmaf(Tr, rv.bg[0], c0);
        rv.image[pix + p] = fmaf(Tr, rv.bg[1], c1);
        rv.image[2 * pix + p] = fmaf(Tr, rv.bg[2], c2);
    }
    rv.ws_tfinal[p] = Tr;
    rv.ws_last[p] = last;
    if (rv.t_final) rv.t_final[p] = Tr;
    if (rv.last_contrib) rv.last_contrib[p] = last;
    if constexpr (COUNTS) {
        if (rv.n_eval) rv.n_eval[p] = neval;
        if (rv.n_blend) rv.n_blend[p] = nblend;
        if (rv.n_tested) rv.n_tested[p] = ntest;
    }
}

// The blend backward: each pixel walks its list back to front, from the
// last entry it blended (ws_last) down to the first, starting from its
// final transmittance (ws_tfinal); both were left by the forward, and so
// were the blend bits, by which a wavefront visits only the entries some
// of its pixels blended.  With
// T_k the transmittance in front of entry k and B_k the colour behind it
// seen through it (the blended colours of the later entries and the
// background, composited from the back):
//   T_k = T_{k+1} / (1 - alpha_k),
//   dC/dalpha_k = T_k (c_k - B_k),   B_{k-1} = alpha_k c_k + (1 - alpha_k) B_k,
// B starting at the background.  Only the gradient-weighted S_k = sum_c
// dL/dC_c B_k,c is needed, updated by the same convex combination, so every
// quantity keeps its relative precision however small T gets (the colour
// behind is never formed as a difference of the whole pixel colour and a
// prefix).  The skip decisions (alpha < 1/255, exponent > 0) are the
// forward's inline routine; an entry is blended iff it passes them and lies
// before the pixel's last blended entry.
//
// Per blended entry the lane's contribution to the nine sums, as moments:
//   dL/du = ln2 (qa2 Sx + qb Sy),  dL/dv = ln2 (qc2 Sy + qb Sx),
//   Sx = sum dp dx,  Sy = sum dp dy,  dL/do = sum dp / o,
//   dL/dA = -1/2 sum dp dx^2,  dL/dB = -sum dp dx dy,  dL/dC = -1/2 sum dp dy^2,
// with dp = dL/dpower, qa2 = 2 qa, qc2 = 2 qc; the constant factors are applied
// once per wave to the reduced sums.
template <int T, int PPT, int BATCH, class Table>
__global__ void __launch_bounds__((Shape<T, PPT>::NT)) __attribute__((amdgpu_waves_per_eu(7)))
raster_bwd_kernel(Table vt) {
    using S = Shape<T, PPT>;
    constexpr bool kListed = PPT == 1;
    // splat constants ga, gb and (blue, 2 qa, 2 qc, 1 / o), at one stride so one
    // address serves all (kListed: and an entry of zeros, which blends nothing)
    __shared__ float4 s_e[3][BATCH + kListed];
    __shared__ uint64_t s_row[BATCH];                            // its row of grad2d, in bytes
    __shared__ uint16_t s_list[kListed ? S::NT / 64 : 1][kListed ? BATCH + 64 : 1];
    __shared__ uint32_t s_plain[kListed ? 1 : BATCH];            // splat_plain
    __shared__ uint32_t s_end;                                   // entries the tile walks
    // multi-wavefront tiles add their wavefronts' sums in LDS and flush each
    // batch with one set of global atomics per entry
    constexpr bool kBlockSum = S::NT > 64;
    __shared__ float s_g[kBlockSum ? (BATCH + kListed) * kGrad2d : 1];
    int v;
    int64_t tile;
    if (!locate(vt, blockIdx.x, v, tile)) return;                // block-uniform
    const RasterView& rv = vt.v[v];
    const Grid& grid = rv.grid;
    if (rv.order)                                                // heaviest tiles first
        tile = __builtin_amdgcn_readfirstlane(
            int(min(rv.order[tile], uint32_t(grid.num_tiles() - 1))));
    const int tid = threadIdx.x;
    const int tx = int(tile % grid.gx), ty = int(tile / grid.gx);
    const int i0 = tx * T + S::px(tid), j0 = ty * T + S::py(tid);
    uint32_t start, end;
    tile_range(rv, tile, start, end);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long* wbits = rv.bits + uint64_t(wave) * rv.bits_stride;
    // the bits describe this launch's wavefronts only if the forward used the
    // same work split
    const bool use_bits = __builtin_amdgcn_readfirstlane(int(*rv.fwd_split)) == PPT;
    const uint64_t pix = uint64_t(grid.w_ds) * grid.h_ds;
    // per pixel: the transmittance behind the current entry (T_final at the
    // start), the gradient-weighted colour behind it (the background at the
    // start), dL/dC and the 1-based index of the last blended entry
    float X[S::NP], Y[S::NP], Ts[S::NP], Sb[S::NP];
    float g0[S::NP], g1[S::NP], g2[S::NP];
    uint32_t last[S::NP];
    uint32_t lmax = 0, lmin = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < S::NP; ++k) {
        const int i = i0 + k % S::PX, j = j0 + k / S::PX;
        const bool in = i < grid.w_ds && j < grid.h_ds;
        X[k] = float(grid.stride * i + grid.off_x);
        Y[k] = float(grid.stride * j + grid.off_y);
        // (a pixel that blends nothing: T = 0, so that w and dp are 0 whatever
        // it is tested on)
        Ts[k] = 0.0f;
        g0[k] = g1[k] = g2[k] = 0.0f;
        last[k] = 0;
        if (in) {
            const uint64_t p = uint64_t(j) * grid.w_ds + i;
            g0[k] = rv.dL[p];
            g1[k] = rv.dL[pix + p];
            g2[k] = rv.dL[2 * pix + p];
            last[k] = min(rv.ws_last[p], end - start);
            if (last[k] != 0u) {
                Ts[k] = rv.ws_tfinal[p];
                lmin = min(lmin, last[k]);
            }
        }
        Sb[k] = fmaf(g2[k], rv.bg[2], fmaf(g1[k], rv.bg[1], g0[k] * rv.bg[0]));
        lmax = max(lmax, last[k]);
    }
    // entries [0, wend) hold every blend of this wavefront's pixels, [0, s_end)
    // those of the tile
    // [0, wall) lies before the last blend of every pixel that blends at all
    for (int o = 32; o > 0; o >>= 1) {
        lmax = max(lmax, uint32_t(__shfl_xor(int(lmax), o)));
        lmin = min(lmin, uint32_t(__shfl_xor(int(lmin), o)));
    }
    const uint32_t wend = uint32_t(__builtin_amdgcn_readfirstlane(int(lmax)));
    const uint32_t wall = uint32_t(__builtin_amdgcn_readfirstlane(int(lmin)));
    if (S::NT > 64) {
        if (tid == 0) s_end = 0;
        __syncthreads();
        if (__lane_id() == 0) atomicMax(&s_end, wend);
        __syncthreads();
    }
    const uint32_t tend = S::NT > 64 ? uint32_t(__builtin_amdgcn_readfirstlane(int(s_end))) : wend;
    // factor of the component this lane owns after wave_sum9
    const int lane = __lane_id();
    const int own = (lane & 7) == 0 ? (lane >> 3) : (lane == 63 ? 8 : -1);
    const float scale = own == 0 || own == 1 ? kLn2
                        : own == 2 || own == 4 ? -0.5f
                        : own == 3 ? -1.0f : 1.0f;
    char* const mine = reinterpret_cast<char*>(rv.g2d + max(own, 0));   // its component of row 0
    if (kListed && tid < 3) s_e[tid][BATCH] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    // batches of the list from the back, starting at multiples of BATCH
    const int top = int(tend) == 0 ? -1 : (int(tend) - 1) / BATCH * BATCH;
    for (int lo = top; lo >= 0; lo -= BATCH) {
        const int cnt = min(BATCH, int(tend) - lo);
        if (lo != top) __syncthreads();                          // the previous batch is done
        for (int q = tid; q < cnt; q += S::NT) {
            const uint32_t id = rv.vals[start + uint32_t(lo + q)];
            const float4* r = rv.rec + 3 * uint64_t(id);
            float4 ga, gb;
            stage_conic(r[0], r[1], ga, gb);
            s_e[0][q] = ga;
            s_e[1][q] = gb;
            s_e[2][q] = make_float4(r[2].x, ga.z + ga.z, gb.x + gb.x, 1.0f / gb.y);
            s_row[q] = uint64_t(id) * (kGrad2d * 4);
            if constexpr (!kListed) s_plain[q] = splat_plain(ga, gb) ? 1u : 0u;
        }
        if constexpr (kBlockSum)
            for (int q = tid; q < cnt * kGrad2d; q += S::NT) s_g[q] = 0.0f;
        __syncthreads();
        auto entry = [&](int e, bool plain) {
            const uint32_t at = entry_offset(e);
            const float4 a = entry_part(s_e[0], at), b = entry_part(s_e[1], at);
            const uint32_t pos = uint32_t(lo + e);    // 0-based position in the list
            // the forward's skip decisions; blended iff also before the last blend
            float dx[S::NP], dy[S::NP], t[S::NP], p2[S::NP], alpha[S::NP];
            uint64_t blend[S::NP], clamped[S::NP];
#pragma unroll
            for (int k = 0; k < S::NP; ++k) p2[k] = splat_exponent(a, b, X[k], Y[k], dx[k], dy[k], t[k]);
            splat_test<S::NP>(b.y, plain, p2, alpha, blend, clamped);
            if (pos >= wall) {                        // (uniform)
#pragma unroll
                for (int k = 0; k < S::NP; ++k) blend[k] &= __ballot(pos < last[k]);
            }
            if (!use_bits) {                          // (with the bits some pixel blends it)
                uint64_t any = 0;
#pragma unroll
                for (int k = 0; k < S::NP; ++k) any |= blend[k];
                if (any == 0) return;
            }
            const float4 c = entry_part(s_e[2], at);  // (b, qa2, qc2, 1 / o)
            // ab = alpha where the pixel blends the entry, 0 elsewhere: then
            // w, the S update and dp vanish by themselves, and T is divided by
            // exactly 1 (v_rcp_f32(1) is 1).  dp = dL/dpower.
            float dp[S::NP], gr = 0.0f, gg = 0.0f, gb = 0.0f;
#pragma unroll
            for (int k = 0; k < S::NP; ++k) {
                const float ab = lane_of(blend[k]) ? alpha[k] : 0.0f;
                const float T0 = Ts[k] * __builtin_amdgcn_rcpf(1.0f - ab);    // in front of the entry
                const float w = ab * T0;
                // dL/dalpha = T0 (sum_c dL/dC_c rgb_c - S)
                const float diff = fmaf(g2[k], c.x, fmaf(g1[k], b.w, fmaf(g0[k], b.z, -Sb[k])));
                dp[k] = w * diff;
                Sb[k] = fmaf(ab, diff, Sb[k]);
                gr = k == 0 ? w * g0[k] : fmaf(w, g0[k], gr);
                gg = k == 0 ? w * g1[k] : fmaf(w, g1[k], gg);
                gb = k == 0 ? w * g2[k] : fmaf(w, g2[k], gb);
                Ts[k] = T0;
            }
            if (!plain) {                             // no gradient through the 0.99 clamp
#pragma unroll
                for (int k = 0; k < S::NP; ++k) dp[k] = lane_of(clamped[k]) ? 0.0f : dp[k];
            }
            // the lane's moments of dp, over its columns and rows of pixels, and
            // with the splat's constants dL/du, dL/dv and dL/do = sum dp / o.
            float gv[kGrad2d];
            lane_moments<S>(dp, dx, dy, gv);
            const float mx = gv[0], my = gv[1];
            gv[0] = fmaf(c.y, mx, a.w * my);
            gv[1] = fmaf(c.z, my, a.w * mx);
            gv[5] *= c.w;
            gv[6] = gr;
            gv[7] = gg;
            gv[8] = gb;
            float sum = wave_sum9(gv);
            sum *= scale;
            asm volatile("" : "+v"(sum));             // (summed by all lanes, not below)
            if (own >= 0) {
                if constexpr (kBlockSum) {
                    atomicAdd(&s_g[e * kGrad2d + own], sum);
                } else {
                    atomicAdd(reinterpret_cast<float*>(mine + s_row[e]), sum);
                }
            }
        };
        // two entries (kListed).  The splat's constants go to the sums, which
        // costs nothing here (the kernel waits for its chain of entries, not for
        // instructions) and is as exact as per lane: dL/du of 4000 random splats
        // over 8 x 8 pixels, in float32 against 64 bits, median relative error
        // 9.6e-8 against 8.6e-8, nine tenths below 6.1e-7 against 5.1e-7.
        auto pair = [&](const EntryPair& g) {
            float ab[2], dx[2], dy[2];
            uint64_t clamped[2];
            uint32_t row[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float t, alpha;
                uint64_t hit;
                const float p2 = splat_exponent(g.a[u], g.b[u], X[0], Y[0], dx[u], dy[u], t);
                splat_test<1>(g.b[u].y, false, &p2, &alpha, &hit, clamped + u);
                const uint32_t pos = uint32_t(lo) + (g.at[u] >> 4);
                hit &= __ballot(pos < last[0]);
                ab[u] = lane_of(hit) ? alpha : 0.0f;
                row[u] = g.at[u] >> 4;
            }
            float sum[2], gv[2][kGrad2d];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 b = g.b[u], c = g.c[u];
                const float T0 = Ts[0] * __builtin_amdgcn_rcpf(1.0f - ab[u]);
                const float w = ab[u] * T0;
                const float diff = fmaf(g2[0], c.x, fmaf(g1[0], b.w, g0[0] * b.z)) - Sb[0];
                float dp = ab[u] * (T0 * diff);
                Sb[0] = fmaf(ab[u], diff, Sb[0]);
                Ts[0] = T0;
                dp = lane_of(clamped[u]) ? 0.0f : dp;
                lane_moments<S>(&dp, dx + u, dy + u, gv[u]);
                gv[u][5] *= c.w;
                gv[u][6] = w * g0[0];
                gv[u][7] = w * g1[0];
                gv[u][8] = w * g2[0];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) sum[u] = wave_sum9(gv[u]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // lanes 0 and 8 hold Sx and Sy: exchange them (rotation by 8
                // within a row of 16 lanes)
                const float cross = g.a[u].w * dpp_f<kDppRowRor8>(sum[u]);
                sum[u] = own == 0 ? fmaf(g.c[u].y, sum[u], cross) : sum[u];
                sum[u] = own == 1 ? fmaf(g.c[u].z, sum[u], cross) : sum[u];
                sum[u] *= scale;
                asm volatile("" : "+v"(sum[u]));      // (summed by all lanes, not below)
            }
            if (own >= 0) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if constexpr (kBlockSum) {
                        atomicAdd(&s_g[row[u] * kGrad2d + uint32_t(own)], sum[u]);
                    } else if (row[u] != uint32_t(BATCH)) {
                        atomicAdd(reinterpret_cast<float*>(mine + s_row[row[u]]), sum[u]);
                    }
                }
            }
        };
        if constexpr (kListed) {
            // the entries the blend bits name (below), from the last to the
            // first: their LDS offsets, then the entry of zeros
            const int wcnt = min(cnt, max(0, int(wend) - lo));
            uint64_t word = ~uint64_t(0);             // lane l: the bits of entries [64 l, 64 l + 64)
            if (use_bits && lane * 64 < wcnt)
                word = wbits[(start >> 6) + uint64_t(tile) + uint64_t(lo / 64 + lane)];
            uint32_t n = 0;
#pragma unroll
            for (int c = BATCH - 64; c >= 0; c -= 64) {
                uint64_t m = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(word), c / 64))) |
                             uint64_t(uint32_t(__builtin_amdgcn_readlane(int(word >> 32), c / 64))) << 32;
                if (!use_bits) {                      // as the forward would have left them
                    m = 0;
                    for (int e = c; e < min(c + 64, wcnt); ++e) {
                        float dx, dy, t, alpha;
                        uint64_t hit, clamped;
                        const float p2 = splat_exponent(s_e[0][e], s_e[1][e], X[0], Y[0], dx, dy, t);
                        splat_test<1>(s_e[1][e].y, false, &p2, &alpha, &hit, &clamped);
                        hit &= __ballot(uint32_t(lo + e) < last[0]);
                        m |= hit != 0 ? uint64_t(1) << (e - c) : 0;
                    }
                }
                if (wcnt - c < 64) m = wcnt > c ? m & ((uint64_t(1) << (wcnt - c)) - 1) : 0;
                const uint32_t all = uint32_t(__builtin_popcountll(m));
                if ((m >> lane) & 1u)
                    s_list[wave][n + all - 1u - lanes_below(m)] = uint16_t((c + lane) * 16);
                n += all;
            }
            if (lane < kListPad) s_list[wave][n + uint32_t(lane)] = uint16_t(BATCH * 16);
            wave_lds_sync();
            for (uint32_t b0 = 0; b0 < n; b0 += 64) {
                const uint32_t nb = min(64u, n - b0);
                const uint32_t at = s_list[wave][b0 + uint32_t(lane)];
                EntryPair g0, g1;
                g0.load(s_e, at, 0);
                for (uint32_t i = 0; i < nb; i += kListStep) {
                    g1.load(s_e, at, i + 2);
                    pair(g0);
                    g0.load(s_e, at, (i + kListStep) & 63u);
                    pair(g1);
                }
            }
        } else {
            // from the last to the first, the entries that some pixel of this
            // wavefront blended in the forward: the blend bits, one word per 64
            // entries (the batch starts at a multiple of 64 entries of the tile's
            // list).  Without usable bits (a forward with another work split has
            // another wavefront partition) every entry is visited; each pixel
            // still decides its own.  Entries at or past this wavefront's last
            // blend change nothing.
            const int wcnt = min(cnt, max(0, int(wend) - lo));
            const uint64_t chunk = (start >> 6) + uint64_t(tile) + uint64_t(lo / 64);
            for (int c = ((wcnt - 1) >> 6) << 6; c >= 0; c -= 64) {
                uint64_t m = use_bits ? uint64_t(wbits[chunk + uint64_t(c >> 6)]) : ~uint64_t(0);
                if (wcnt - c < 64) m &= (uint64_t(1) << (wcnt - c)) - 1;
                const int q = c + lane;
                const uint64_t other = m & ~__ballot(q < cnt && s_plain[q] != 0u);
                while (m != 0) {
                    const int hb = 63 - __builtin_clzll(m);
                    m ^= uint64_t(1) << hb;
                    entry(c + hb, ((other >> hb) & 1u) == 0);
                }
            }
        }
        if constexpr (kBlockSum) {
            __syncthreads();
            for (int q = tid; q < cnt * kGrad2d; q += S::NT) {
                const float g = s_g[q];
                if (g != 0.0f)
                    atomicAdd(reinterpret_cast<float*>(reinterpret_cast<char*>(rv.g2d) +
                                                       s_row[q / kGrad2d]) +
                                  q % kGrad2d, g);
            }
        }
    }
}

// L1 photometric loss of the rendered pixels against the full-resolution
// pixels they are rendered at (Sec. 4.1, Fig. 2: supervision from the
// corresponding high-resolution pixels; Sec. 4.2 names the L1 loss) and its
// gradient, for a table of views in one launch.  A view's blocks walk rows of its strided image
// (the rows of a pixel phase), so the image and dL accesses are contiguous;
// one double atomic per block adds the block's share of the view's loss (a
// bounded number of atomics on one address).
constexpr uint32_t kL1MaxBlocks = 2048;

template <class Table>
__global__ void __launch_bounds__(256) l1_grad_kernel(Table vt) {
    __shared__ double wsum[4];
    int v = 0;
    if constexpr (Table::kViews > 1)
        while (v + 1 < vt.count && blockIdx.x >= vt.first_block[v + 1]) ++v;   // block-uniform
    const L1View& lv = vt.v[v];
    const Grid& grid = lv.grid;
    const uint32_t lb = blockIdx.x - vt.first_block[v];
    const uint32_t nb = vt.first_block[v + 1] - vt.first_block[v];
    const uint32_t w = uint32_t(grid.w_ds), h = uint32_t(grid.h_ds);
    const uint64_t pix = uint64_t(w) * h;
    const uint64_t full = uint64_t(grid.width) * grid.height;
    const float inv = 1.0f / float(3 * pix);
    double s = 0.0;
    for (uint32_t j = lb; j < h; j += nb) {
        const uint64_t Y = uint64_t(grid.stride) * j + grid.off_y;
        const float* trow = lv.target + Y * grid.width + grid.off_x;
        // four pixels per thread and pass, every load issued before the
        // first use
        constexpr int kU = 4;
        for (uint32_t i0 = threadIdx.x; i0 < w; i0 += kU * blockDim.x) {
            float im[kU][3], tg[kU][3];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint32_t i = i0 + uint32_t(u) * blockDim.x;
                const uint64_t p = uint64_t(j) * w + i;
                const uint64_t X = uint64_t(grid.stride) * i;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    im[u][c] = i < w ? lv.image[c * pix + p] : 0.0f;
                    tg[u][c] = i < w ? trow[c * full + X] : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint32_t i = i0 + uint32_t(u) * blockDim.x;
                if (i >= w) continue;
                const uint64_t p = uint64_t(j) * w + i;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float diff = im[u][c] - tg[u][c];
                    const float sg = diff > 0.0f ? 1.0f : (diff < 0.0f ? -1.0f : 0.0f);
                    lv.dL[c * pix + p] = sg * inv;
                    s += fabs(double(diff));
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0 && lv.loss) {
        atomicAdd(lv.loss, (wsum[0] + wsum[1] + wsum[2] + wsum[3]) / double(3 * pix));
    }
}

// The views' losses to zero before the atomics (a fill kernel, so the step
// stays capturable without memset nodes).
struct LossPointers {
    int count;
    double* loss[kMaxViews];
};

__global__ void l1_zero_kernel(LossPointers p) {
    const int v = int(threadIdx.x);
    if (v < p.count && p.loss[v]) *p.loss[v] = 0.0;
}

// The table of the one view of a larger one.
template <template <int> class Table, int N>
Table<1> first_view(const Table<N>& vt) {
    return Table<1>{1, {vt.first_block[0], vt.first_block[1]}, {vt.v[0]}};
}

bool wants_counts(const RasterViews& vt) {
    for (int k = 0; k < vt.count; ++k)
        if (vt.v[k].n_eval || vt.v[k].n_blend || vt.v[k].n_tested)
            return true;
    return false;
}

// The rasterizers' schedule.  A view's tiles carry very different work
// (the entries walked before every pixel stops: up to 3x the mean at the
// 4K scene), and in row-major order the heavy tiles of the image centre
// end up unevenly on the SIMDs: the last ones finish 40-50 % after the
// mean.  The dispatcher starts workgroups in index order as slots free up,
// so the tiles of each view are handed out heaviest first by the entries a
// forward walked in them (longest-processing-time-first list scheduling):
// the backward by those of its own forward, the forward by those the
// previous forward on the same workspace left (the same view at another
// phase, or the same camera at its previous visit).  A counting sort over
// 256 weight buckets (exact below 32, then eight per power of two), one
// block per view.  Any weights give a permutation of the tiles: they
// decide the order only, never what is rendered.
constexpr int kOrderBuckets = 256;

__device__ __forceinline__ uint32_t weight_bucket(uint32_t w) {
    if (w < 32u) return w;
    const uint32_t e = 31u - uint32_t(__builtin_clz(w));         // 5 .. 31
    return 32u + (e - 5u) * 8u + ((w >> (e - 3u)) & 7u);         // < 248
}

// A block takes every `shares`-th tile, from its share-th, sorts these and
// hands them every `shares`-th place of the order.  The shares are alike, so
// the whole is heaviest first but for the differences between them.  (The time
// is that of the LDS atomics, one a clock where neighbouring tiles share a
// bucket: in one block 33 us at 32400 tiles and 9 at 8160, with kOrderShare
// tiles to a block 5 and 5.)
__device__ __forceinline__ void order_share(const RasterView& rv, uint32_t share, uint32_t shares) {
    __shared__ uint32_t s_cur[kOrderBuckets];
    const uint32_t nt = uint32_t(rv.grid.num_tiles());
    const uint32_t tid = threadIdx.x;
    if (!rv.order || !rv.work || share >= nt) return;            // block-uniform
    const uint32_t mine = (nt - share - 1) / shares + 1;
    const uint32_t* work = rv.work + share;
    uint32_t* order = rv.order + share;
    for (uint32_t k = tid; k < kOrderBuckets; k += blockDim.x) s_cur[k] = 0;
    __syncthreads();
    for (uint32_t t = tid; t < mine; t += blockDim.x)
        atomicAdd(&s_cur[weight_bucket(work[uint64_t(t) * shares])], 1u);
    __syncthreads();
    // first slot of every bucket, heaviest bucket first: lane l holds
    // buckets 255 - 4l .. 252 - 4l
    if (tid < 64) {
        uint32_t c[4], sum = 0, total;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = s_cur[kOrderBuckets - 1 - 4 * int(tid) - q];
            sum += c[q];
        }
        uint32_t run = wave_exclusive_sum(sum, total);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s_cur[kOrderBuckets - 1 - 4 * int(tid) - q] = run;
            run += c[q];
        }
    }
    __syncthreads();
    for (uint32_t t = tid; t < mine; t += blockDim.x) {
        const uint32_t pos = atomicAdd(&s_cur[weight_bucket(work[uint64_t(t) * shares])], 1u);
        if (pos < mine) order[uint64_t(pos) * shares] = share + t * shares;   // (weights changed under us)
    }
}

__global__ void __launch_bounds__(1024) tile_order_kernel(RasterViews vt) {
    order_share(vt.v[blockIdx.y], blockIdx.x, gridDim.x);
}

// What the backward needs first, in one launch: the tile order (the first
// `shares` blocks of a view) and grad2d of n Gaussians to zero (the others).
constexpr uint32_t kZeroLoop = 4;                                // 16-byte stores per thread

__global__ void __launch_bounds__(1024) bwd_prepare_kernel(RasterViews vt, uint32_t shares, uint64_t words) {
    const RasterView& rv = vt.v[blockIdx.y];
    if (blockIdx.x < shares) {
        order_share(rv, blockIdx.x, shares);
        return;
    }
    const uint64_t n4 = words / 4;
    uint64_t i = (uint64_t(blockIdx.x - shares) * kZeroLoop) * 1024u + threadIdx.x;
#pragma unroll
    for (uint32_t q = 0; q < kZeroLoop; ++q, i += 1024u)
        if (i < n4) reinterpret_cast<uint4*>(rv.g2d)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == shares && threadIdx.x < words % 4) rv.g2d[4 * n4 + threadIdx.x] = 0.0f;
}

constexpr int64_t kOrderShare = 512;                             // tiles per block

// Up to two workgroups to a CU start at once whatever their order, and the two
// launches cost more than it gives: 468 tiles 171 + 7 us with it and 175 without,
// 64 tiles 47 + 5 and 48; 920 tiles (forward) 30 + 3 and 34, 2040 tiles 243 + 10
// and 295.
constexpr uint32_t kOrderMin = 512;

uint32_t order_shares(const RasterViews& vt) {
    if (vt.first_block[vt.count] <= kOrderMin) return 0;
    int64_t most = 1;
    for (int k = 0; k < vt.count; ++k) most = std::max(most, vt.v[k].grid.num_tiles());
    return uint32_t((most + kOrderShare - 1) / kOrderShare);
}

template <int T, int PPT, int B>
void launch_both(bool fwd, const RasterViews& vt, hipStream_t s) {
    const dim3 grid(vt.first_block[vt.count]), block(Shape<T, PPT>::NT);
    if constexpr (PPT == 1) {
        const bool counts = wants_counts(vt);
        auto launch = [&](const auto& table) {
            if (!fwd) raster_bwd_kernel<T, 1, B><<<grid, block, 0, s>>>(table);
            else if (counts) raster_fwd_px1_kernel<T, true><<<grid, block, 0, s>>>(table);
            else raster_fwd_px1_kernel<T, false><<<grid, block, 0, s>>>(table);
        };
        if (vt.count == 1) launch(first_view(vt));
        else launch(vt);
    } else if (!fwd) {
        raster_bwd_kernel<T, PPT, B><<<grid, block, 0, s>>>(vt);
    } else if (wants_counts(vt)) {
        raster_fwd_kernel<T, PPT, B, true><<<grid, block, 0, s>>>(vt);
    } else {
        raster_fwd_kernel<T, PPT, B, false><<<grid, block, 0, s>>>(vt);
    }
}

template <int T, int PPT>
void launch_batch(bool fwd, int batch, const RasterViews& vt, hipStream_t s) {
    if (batch == 64) launch_both<T, PPT, 64>(fwd, vt, s);
    else if (batch == 128) launch_both<T, PPT, 128>(fwd, vt, s);
    else launch_both<T, PPT, 256>(fwd, vt, s);
}

// Work splits compiled per tile size: T = 8 one pixel per thread (a single
// wavefront); T = 16 one, two or four; T = 32 two or four.
hipError_t launch_raster(bool fwd, int tile, int ppt, int batch, RasterViews vt, hipStream_t s) {
    if (vt.first_block[vt.count] == 0) return hipGetLastError();
    if (vt.first_block[vt.count] <= kOrderMin)
        for (int k = 0; k < vt.count; ++k) vt.v[k].order = nullptr;
    if (tile == 8) {
        launch_batch<8, 1>(fwd, batch, vt, s);
    } else if (tile == 32) {
        if (ppt == 2) launch_batch<32, 2>(fwd, batch, vt, s);
        else launch_batch<32, 4>(fwd, batch, vt, s);
    } else {
        if (ppt == 2) launch_batch<16, 2>(fwd, batch, vt, s);
        else if (ppt == 4) launch_batch<16, 4>(fwd, batch, vt, s);
        else launch_batch<16, 1>(fwd, batch, vt, s);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_raster_fwd(int tile, int ppt, int batch, const RasterViews& vt, hipStream_t s) {
    if (vt.count == 0) return hipSuccess;
    if (const uint32_t shares = order_shares(vt))
        tile_order_kernel<<<dim3(shares, unsigned(vt.count)), dim3(1024), 0, s>>>(vt);
    return launch_raster(true, tile, ppt, batch, vt, s);
}

hipError_t launch_raster_bwd(int tile, int ppt, int batch, const RasterViews& vt, int64_t n,
                             hipStream_t s) {
    if (vt.count == 0) return hipSuccess;
    const uint32_t shares = order_shares(vt);
    const uint64_t words = uint64_t(n) * kGrad2d, per = 1024u * kZeroLoop;
    const uint64_t zero = n > 0 ? std::max<uint64_t>(1, (words / 4 + per - 1) / per) : 0;
    if (shares + zero > 0)
        bwd_prepare_kernel<<<dim3(unsigned(shares + zero), unsigned(vt.count)), dim3(1024), 0, s>>>(vt, shares, words);
    return launch_raster(false, tile, ppt, batch, vt, s);
}

hipError_t launch_l1_grad(L1Views& vt, hipStream_t s) {
    uint32_t blocks = 0;
    for (int k = 0; k < vt.count; ++k) {
        vt.first_block[k] = blocks;
        const Grid& g = vt.v[k].grid;
        const uint64_t pix = uint64_t(g.w_ds) * g.h_ds;
        blocks += pix == 0 ? 0u : uint32_t(std::min<uint64_t>(uint64_t(g.h_ds), kL1MaxBlocks));
    }
    vt.first_block[vt.count] = blocks;
    if (vt.count == 0) return hipSuccess;
    LossPointers p{vt.count, {}};
    for (int k = 0; k < vt.count; ++k) p.loss[k] = vt.v[k].loss;
    l1_zero_kernel<<<1, 64, 0, s>>>(p);
    if (blocks > 0 && vt.count == 1) l1_grad_kernel<<<dim3(blocks), dim3(256), 0, s>>>(first_view(vt));
    else if (blocks > 0) l1_grad_kernel<<<dim3(blocks), dim3(256), 0, s>>>(vt);
    return hipGetLastError();
}

}  // namespace tgs
