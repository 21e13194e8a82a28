// Per-tile front-to-back alpha compositing (Eq. 2) and its hand-written
// backward.
//
// One wavefront owns one screen tile made of QX x QY quadrants of 8x8 pixels
// (or, split per tile from the frame's plan, a run of its quadrants); lane l
// holds pixel (l % 8, l / 8) of every quadrant, so PPL = QX * QY pixels per
// lane.  The wave walks the tile's record list in (depth, record) order,
// staging a batch of records at a time in a wave-private LDS slice (one record
// per lane, read back as broadcasts): no workgroup barrier in the walk, and
// each wave stops as soon as all its pixels have terminated.  While staging,
// each lane also computes which quadrants its record can reach (pixel box and
// an exact, conservative bound of alpha over the quadrant); only records that
// reach one are staged (compacted with a ballot prefix), and the compositing
// loop skips (uniformly, per quadrant) every Gaussian that cannot reach
// alpha_min there.  The forward hands these quadrant masks to the backward,
// one byte per list entry.  Past that test the per-pixel work is predicated
// (selects, not branches): a pixel that does not keep a Gaussian adds an
// exact zero and keeps its transmittance, and the forward keeps its per-pixel
// stop flags as wave-wide lane masks, so their bookkeeping runs on the scalar
// unit.  Workgroups are remapped so that each XCD renders one contiguous run
// of tiles (neighbouring tiles share records in that XCD's L2).
//
// The backward runs front to back as well: it recomputes alpha, T and the
// accumulated colour with the forward's operations, keeps a Gaussian at a
// pixel exactly when alpha >= alpha_min and its list position is below the
// forward's contributor count there, and gets the colour behind a Gaussian
// as C_final - C_accumulated, so no per-pair transmittance is ever stored.
// Per (tile, record) pair it forms nine partials per lane and reduces those
// of two records at once with the gfx950 lane-swap instructions and a row
// sum; a row's last lane stores them at the pair's emission index, where the
// projection backward adds each record's pairs in a fixed order
// (deterministic, no float atomics).  The nine values are, with
// ge = dL/dalpha * alpha summed over the pair's pixels and (e1, e2) the
// offset pixel - mean in the footprint's axes (e1 along the conic's narrow
// axis (c, s) that the record carries, e2 = (-s, c) across):
//   sum ge, sum ge e1, sum ge e2, sum ge e1^2, sum ge e1 e2, sum ge e2^2,
//   and dL/dcolour (r, g, b).
// The geometric gradients follow from these moments in closed form.
#include "gs_device.hpp"
#include "gs_internal.hpp"

namespace gs {

constexpr int kRenderWaves = 4;
constexpr int kBwdBatch = 48;   // records staged per backward batch (of the 64 lanes)

// record words as produced by the projection
enum { R_MX = 0, R_MY, R_QA, R_QB, R_QC, R_LO, R_CR, R_CG, R_CB, R_AXIS, R_HX, R_HY };
// LDS slots of a staged backward record past the first nine: the moment frame
enum { S_AXC = 9, S_AXS = 10 };

template <typename T>
struct Rec {
    T mx, my, qa, qb, qc, lo, c[3];
};

// log2 of the Gaussian's alpha at offset (dx, dy) from its mean:
// log2 o - (a dx^2 + 2 b dx dy + c dy^2) log2(e) / 2 with the scale folded
// into qa, qb, qc
template <typename T>
__device__ inline T log2_alpha(const Rec<T>& g, T dx, T dy) {
    using N = Num<T>;
    const T t = N::fma(g.qa, dx, g.qb * dy);
    return N::fma(t, dx, N::fma(g.qc * dy, dy, g.lo));
}

// min(alpha, alpha_max) for alpha >= +0 or NaN: non-negative floats order
// like their bit patterns, and a NaN's pattern lies above every finite one,
// so the unsigned minimum equals fminf (NaN gives alpha_max) in one integer
// instruction, without the NaN quieting fminf costs
template <typename T> __device__ inline T clamp_alpha(T al, T amax);
template <> __device__ inline float clamp_alpha<float>(float al, float amax) {
    return __uint_as_float(min(__float_as_uint(al), __float_as_uint(amax)));
}
template <> __device__ inline double clamp_alpha<double>(double al, double amax) { return Num<double>::min(al, amax); }

template <typename T> __device__ inline T recip(T x);
template <> __device__ inline float recip<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <> __device__ inline double recip<double>(double x) { return 1.0 / x; }

template <typename T>
__device__ inline Rec<T> lds_rec(const T* s) {
    Rec<T> g;
    g.mx = s[R_MX]; g.my = s[R_MY]; g.qa = s[R_QA]; g.qb = s[R_QB]; g.qc = s[R_QC]; g.lo = s[R_LO];
    g.c[0] = s[R_CR]; g.c[1] = s[R_CG]; g.c[2] = s[R_CB];
    return g;
}

// Load record r into registers (one record per lane while staging).
template <typename T>
__device__ inline void load_rec(const T* __restrict__ rec, uint32_t r, T (&w)[GS_REC_WORDS]) {
    const T* src = rec + int64_t(r) * GS_REC_WORDS;
#pragma unroll
    for (int i = 0; i < GS_REC_WORDS; i++) w[i] = src[i];
}

template <typename T>
__device__ inline T clamp_to(T v, T lo, T hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Quadrant mask of a record for the tile whose top-left pixel is (px0, py0):
// bit k is set unless no pixel centre of quadrant k can reach alpha_min.
// Two conservative tests must both pass.  (1) The record's pixel box
// [mean -+ half-extent] meets the quadrant.  (2) The largest log2 alpha over
// the quadrant's rectangle of pixel centres is at least log2 alpha_min, less a
// margin that covers the rounding of this bound and of the per-pixel
// evaluation.  The exponent is a concave quadratic in (dx, dy): over a
// rectangle that holds the mean its maximum is at the mean, otherwise on an
// edge, at the edge's stationary point clamped to the edge.  Test (2) drops
// what the box keeps only because it is axis-aligned (elongated, rotated
// Gaussians); a skipped pixel would have had alpha < alpha_min, so images and
// gradients are unchanged.
template <typename T>
__device__ inline uint32_t quad_mask_n(const T (&w)[GS_REC_WORDS], int px0, int py0, int nqx, int nq, T lmin) {
    using N = Num<T>;
    const T mx = w[R_MX], my = w[R_MY], qa = w[R_QA], qb = w[R_QB], qc = w[R_QC], lo = w[R_LO];
    const T x0 = mx - w[R_HX], x1 = mx + w[R_HX];
    const T y0 = my - w[R_HY], y1 = my + w[R_HY];
    // on an edge dx = e the maximum over dy sits at dy = sx e; on dy = e, at dx = sy e
    const T sx = -qb * recip(T(2) * qc), sy = -qb * recip(T(2) * qa);
    const T aqb = qb < T(0) ? -qb : qb;
    const T alo = lo < T(0) ? -lo : lo;
    auto expo = [&](T dx, T dy) { return N::fma(N::fma(qa, dx, qb * dy), dx, qc * dy * dy); };
    uint32_t mask = 0;
#pragma unroll 1
    for (int k = 0; k < nq; k++) {
        const T qx = T(px0 + 8 * (k % nqx)), qy = T(py0 + 8 * (k / nqx));
        const bool box = x1 >= qx + T(0.5) && x0 <= qx + T(7.5) && y1 >= qy + T(0.5) && y0 <= qy + T(7.5);
        const T ax = qx + T(0.5) - mx, bx = qx + T(7.5) - mx;
        const T ay = qy + T(0.5) - my, by = qy + T(7.5) - my;
        const bool inside = ax <= T(0) && bx >= T(0) && ay <= T(0) && by >= T(0);
        T best = expo(ax, clamp_to(sx * ax, ay, by));
        best = N::max(best, expo(bx, clamp_to(sx * bx, ay, by)));
        best = N::max(best, expo(clamp_to(sy * ay, ax, bx), ay));
        best = N::max(best, expo(clamp_to(sy * by, ax, bx), by));
        // magnitude of the exponent's terms over the rectangle: scale of the rounding
        const T X = N::max(-ax, bx), Y = N::max(-ay, by);
        const T mag = N::fma(-qa * X, X, N::fma(aqb * X, Y, -qc * Y * Y)) + alo;
        const bool ell = inside || best + lo >= lmin - (T(1e-3) + mag * T(4e-6));
        mask |= box && ell ? (1u << k) : 0u;
    }
    return mask;
}

// the same over the QX x QY quadrants from pixel (px0, py0)
template <typename T, int QX, int QY>
__device__ inline uint32_t quad_mask(const T (&w)[GS_REC_WORDS], int px0, int py0, T lmin) {
    return quad_mask_n(w, px0, py0, QX, QX * QY, lmin);
}

__device__ inline uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// centre coordinate of a lane's pixel in quadrant column/row q: the lane's
// quadrant-0 centre plus 8 q (exact in floating point), so that every tile
// shape computes the same pixel - mean offsets bit for bit
template <typename T>
__device__ inline T quad_centre(T base, int q) {
    return q == 0 ? base : base + T(8 * q);
}

__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Stores the nine partials of two records' pairs (a at da, b at db; db may
// be null), each summed over the wave's 64 lanes.  The two records are
// reduced together; a swap of wave halves (v_permlane32_swap) and an add
// leave record a's sums in lanes 0-31 and b's in lanes 32-63; a swap of
// odd and even rows (v_permlane16_swap) between neighbouring partials and an
// add leave in each row of 16 lanes five partials of one record (the even or
// the odd ones); a row sum finishes them in the row's last lane, which
// stores them.  A fixed sequence of operations: the sums are deterministic.
__device__ inline float swap_add32(float a, float b) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ inline float swap_add16(float a, float b) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// the same swaps of the two 32-bit halves of a double
template <bool ROWS>
__device__ inline double swap_add_f64(double a, double b) {
    const uint64_t ua = uint64_t(__double_as_longlong(a)), ub = uint64_t(__double_as_longlong(b));
    const auto swap = [](uint32_t x, uint32_t y) {
        return ROWS ? __builtin_amdgcn_permlane16_swap(x, y, false, false)
                    : __builtin_amdgcn_permlane32_swap(x, y, false, false);
    };
    const auto lo = swap(uint32_t(ua), uint32_t(ub)), hi = swap(uint32_t(ua >> 32), uint32_t(ub >> 32));
    const uint64_t p = uint64_t(lo[0]) | uint64_t(hi[0]) << 32, q = uint64_t(lo[1]) | uint64_t(hi[1]) << 32;
    return __longlong_as_double((long long)p) + __longlong_as_double((long long)q);
}
__device__ inline double swap_add32(double a, double b) { return swap_add_f64<false>(a, b); }
__device__ inline double swap_add16(double a, double b) { return swap_add_f64<true>(a, b); }

template <typename T>
__device__ inline void store_pair_partials(const T (&va)[9], const T (&vb)[9], T* da, T* db) {
    const int lane = lane_id();
    T x[9], y[5];
#pragma unroll
    for (int q = 0; q < 9; q++) x[q] = swap_add32(va[q], vb[q]);
#pragma unroll
    for (int j = 0; j < 4; j++) y[j] = swap_add16(x[2 * j], x[2 * j + 1]);
    y[4] = swap_add16(x[8], T(0));
#pragma unroll
    for (int j = 0; j < 5; j++) y[j] = row_sum_last(y[j]);
    if ((lane & 15) == 15) {
        const int r = lane >> 4;
        T* dst = r < 2 ? da : db;
        const int par = r & 1;
        if (dst)
#pragma unroll
            for (int j = 0; j < 5; j++)
                if (2 * j + par < 9) dst[2 * j + par] = y[j];
    }
}

// ---------------------------------------------------------------------------
// forward

// STATS: also add the number of (pixel, Gaussian) contributions of the
// launch to *kept (one 64-bit atomic per wave).  At least kFwdWavesPerSimd
// wavefronts per SIMD: the FP32 forward then fits in 72 registers without
// spilling, against 80 (6 per SIMD) left to itself.
constexpr int kFwdWavesPerSimd = 7;
template <typename T, int QX, int QY, int NS, bool STATS>
__global__ __launch_bounds__(kWave * kRenderWaves, kFwdWavesPerSimd) void k_render_fwd(
    gs_frame frame, gs_raster_cfg cfg, const T* __restrict__ rec, const uint32_t* __restrict__ vals,
    const uint2* __restrict__ ranges, T* __restrict__ rgb, T* __restrict__ Tout, uint32_t* __restrict__ ncontrib,
    unsigned long long* __restrict__ kept, const uint32_t* __restrict__ order, uint8_t* __restrict__ qmask) {
    constexpr int PPL = QX * QY;
    // NS wavefronts per tile, wave `sub` owning the tile's sub-tile of QX x QY
    // quadrants; NS = 0: the plan's wavefronts, heavy tiles first, each owning
    // a run of the tile's quadrants (QX x QY is then the tile)
    constexpr bool ADAPT = NS == 0;
    constexpr int NSD = ADAPT ? 1 : NS;
    __shared__ T s_rec[kRenderWaves][kWave][GS_REC_WORDS];
    __shared__ uint32_t s_mask[kRenderWaves][kWave];
    const int wave = threadIdx.x / kWave, lane = lane_id();
    int tile, sub;
    uint32_t owned = (1u << PPL) - 1u;
    if (ADAPT) {
        int waves;
        if (!plan_wave<false>(order, frame.n_tiles, blockIdx.x * kRenderWaves + wave, tile, sub, waves)) return;
        owned = owned_quadrants(PPL, waves, sub);
    } else {
        const int gw = xcd_block(blockIdx.x, gridDim.x) * kRenderWaves + wave;
        tile = gw / NSD;
        sub = gw % NSD;
        if (tile >= frame.n_tiles) return;
    }
    const int j = job_of_tile(frame.jobs, frame.n_jobs, tile);
    const gs_job job = frame.jobs[j];
    const gs_camera& cam = frame.cams[job.cam];
    const int W = cam.width, H = cam.height;
    const int lt = tile - job.tile0;
    const int sxn = cfg.tile_w / (8 * QX);   // sub-tiles per tile row
    const int tpx = (lt % job.tiles_x) * cfg.tile_w + (ADAPT ? 0 : (sub % sxn) * 8 * QX);
    const int tpy = (lt / job.tiles_x) * cfg.tile_h + (ADAPT ? 0 : (sub / sxn) * 8 * QY);
    const int lx = lane & 7, ly = lane >> 3;
    // pixel centre of quadrant k: (bx + 8 (k % QX), by + 8 (k / QX))
    const T bx = T(tpx + lx) + T(0.5), by = T(tpy + ly) + T(0.5);

    // per quadrant, the lanes whose pixel has stopped (or lies outside the
    // image or the wavefront's quadrants): a wave-uniform lane mask, so the
    // stop bookkeeping runs on the scalar unit
    T Tr[PPL], C[PPL][3];
    uint64_t stopm[PPL];
    uint32_t last[PPL];
    uint32_t n_kept = 0;
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        const int x = tpx + 8 * (k % QX) + lx, y = tpy + 8 * (k / QX) + ly;
        stopm[k] = lane_mask(!(x < W && y < H && (owned & (1u << k))));
        Tr[k] = T(1);
        C[k][0] = C[k][1] = C[k][2] = T(0);
        last[k] = 0;
    }
    const uint2 range = ranges[tile];
    const T amin = T(cfg.alpha_min), amax = T(cfg.alpha_max), tmin = T(cfg.T_min);
    const T lmin = Num<T>::log2(amin);
    for (uint32_t base = range.x; base < range.y; base += kWave) {
        uint64_t all_stopped = ~uint64_t(0);
#pragma unroll
        for (int k = 0; k < PPL; k++) all_stopped &= stopm[k];
        if (all_stopped == ~uint64_t(0)) break;
        const uint32_t cnt = min(uint32_t(kWave), range.y - base);
        // stage the batch's records that reach some quadrant, compacted, each
        // with its quadrant mask and its position in the tile list
        T w[GS_REC_WORDS];
        uint32_t m = 0, r = 0;
        if (uint32_t(lane) < cnt) {
            r = vals[base + lane];
            load_rec(rec, r, w);
            if (ADAPT || NSD == 1) {
                // this wavefront's quadrants are the tile's: its mask is the tile mask
                const uint32_t mt = quad_mask<T, QX, QY>(w, tpx, tpy, lmin);
                if (qmask) qmask[base + lane] = uint8_t(mt);
                m = mt & owned;
            } else {
                m = quad_mask<T, QX, QY>(w, tpx, tpy, lmin) & owned;
                if (qmask) {
                    const int tx0 = (lt % job.tiles_x) * cfg.tile_w, ty0 = (lt / job.tiles_x) * cfg.tile_h;
                    const int nqx = cfg.tile_w / 8;
                    qmask[base + lane] = uint8_t(quad_mask_n(w, tx0, ty0, nqx, nqx * (cfg.tile_h / 8), lmin));
                }
            }
        }
        const uint64_t staged = __ballot(m != 0);
        if (m != 0) {
            const uint32_t slot = __builtin_popcountll(staged & lanemask_lt());
            const T* src = rec + int64_t(r) * GS_REC_WORDS;
            T* dst = s_rec[wave][slot];
#pragma unroll
            for (int q = 0; q < 6; q++) dst[q] = w[q];
#pragma unroll
            for (int q = 6; q < 9; q++) dst[q] = src[q];
            s_mask[wave][slot] = m | (uint32_t(lane) << 8);
        }
        wave_lds_sync();
        const uint32_t n = __builtin_popcountll(staged);
        for (uint32_t i = 0; i < n; i++) {
            const uint32_t word = uniform(s_mask[wave][i]);
            const uint32_t qmask = word & 0xffu, pos = word >> 8;
            const Rec<T> g = lds_rec(s_rec[wave][i]);
#pragma unroll
            for (int k = 0; k < PPL; k++) {
                if (!(qmask & (1u << k))) continue;   // uniform: box misses quadrant k
                const T dx = quad_centre(bx, k % QX) - g.mx, dy = quad_centre(by, k / QX) - g.my;
                const T al = Num<T>::exp2(log2_alpha(g, dx, dy));
                const uint64_t livem = lane_mask(al >= amin) & ~stopm[k];
                if (livem == 0) continue;     // uniform: no pixel of the wave reached
                const T a = clamp_alpha(al, amax);
                const T aT = a * Tr[k];
                const T tn = Tr[k] - aT;
                const uint64_t stopb = lane_mask(tn < tmin) & livem;
                stopm[k] |= stopb;
                const uint64_t keepm = livem & ~stopb;
                const bool keep = lane_in(keepm);
                const T wgt = keep ? aT : T(0);
                C[k][0] = Num<T>::fma(wgt, g.c[0], C[k][0]);
                C[k][1] = Num<T>::fma(wgt, g.c[1], C[k][1]);
                C[k][2] = Num<T>::fma(wgt, g.c[2], C[k][2]);
                Tr[k] = keep ? tn : Tr[k];
                last[k] = keep ? base - range.x + pos + 1 : last[k];
                if (STATS) n_kept += uint32_t(__builtin_popcountll(keepm));   // uniform: the wave's count
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (STATS && lane == 0) atomicAdd(kept, static_cast<unsigned long long>(n_kept));
    const int64_t plane = int64_t(W) * H;
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        const int x = tpx + 8 * (k % QX) + lx, y = tpy + 8 * (k / QX) + ly;
        if (x < W && y < H && (owned & (1u << k))) {
            const int64_t p = job.px0 + int64_t(y) * W + x;
            T* out = rgb + 3 * job.px0 + int64_t(y) * W + x;
            out[0] = C[k][0] + Tr[k] * T(cfg.bg[0]);
            out[plane] = C[k][1] + Tr[k] * T(cfg.bg[1]);
            out[2 * plane] = C[k][2] + Tr[k] * T(cfg.bg[2]);
            Tout[p] = Tr[k];
            ncontrib[p] = last[k];
        }
    }
}

// ---------------------------------------------------------------------------
// backward

// FP32: 5 wavefronts per SIMD (96 registers without a spill, against 100 and 4
// left to itself): bound by VALU issue, 169 -> 163 us at 500k, 1600x1066
template <typename T, int QX, int QY, int NS>
__global__ __launch_bounds__(kWave * kRenderWaves, sizeof(T) == 4 ? 5 : 1) void k_render_bwd(
    gs_frame frame, gs_raster_cfg cfg, const T* __restrict__ rec, const uint4* __restrict__ meta,
    const uint32_t* __restrict__ pair_off, const uint32_t* __restrict__ vals, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ order, uint64_t capacity, const T* __restrict__ rgb,
    const uint32_t* __restrict__ ncontrib, int mode, const T* __restrict__ gin, LossSum<T> loss_to,
    T* __restrict__ pg, const uint8_t* __restrict__ qmask) {
    constexpr int PPL = QX * QY;
    // NS wavefronts per tile, wave `sub` owning the tile's sub-tile of QX x QY
    // quadrants; NS = 0: the plan's wavefronts, heavy tiles first, each owning
    // a run of the tile's quadrants (QX x QY is then the tile).  A tile's
    // wavefronts share a workgroup; each stores its own nine partials per
    // pair (slot `sub`), which they fold into slot 0 at the end
    constexpr bool ADAPT = NS == 0;
    constexpr int NSD = ADAPT ? 1 : NS;
    __shared__ T s_rec[kRenderWaves][kBwdBatch][GS_REC_WORDS];
    __shared__ uint32_t s_mask[kRenderWaves][kBwdBatch];
    __shared__ uint32_t s_eown[kRenderWaves][kBwdBatch];   // emission index of each staged pair
    const int wave = threadIdx.x / kWave, lane = lane_id();
    int tile = 0, sub = 0, nwaves = NSD;
    uint32_t owned = (1u << PPL) - 1u;
    bool valid = true;   // no early return: the workgroup may meet at a barrier below
    __shared__ uint32_t s_wend[kRenderWaves];   // per wavefront: list entries its pixels need (the fold reads as many)
    if (ADAPT) {
        valid = plan_wave<true>(order, frame.n_tiles, blockIdx.x * kRenderWaves + wave, tile, sub, nwaves);
        owned = valid ? owned_quadrants(PPL, nwaves, sub) : 0u;
    } else {
        const int gw = xcd_block(blockIdx.x, gridDim.x) * kRenderWaves + wave;
        tile = gw / NSD;
        sub = gw % NSD;
        valid = tile < frame.n_tiles;
    }
    // where this wavefront's partials of pair e lie (partial_slot): from own on,
    // every `apart` values, both uniform; formed here, as a choice by sub for
    // every record took registers (four spilled with the plan) and held up
    // wavefronts that have a SIMD to themselves (500k at 1600x1066 with the
    // plan 154.5 -> 151 us; 200k in 320x240 with 2 per tile 433 -> 418)
    const bool further = NS != 1 && uniform(uint32_t(sub)) > 0u;
    T* const own = pg + (further ? partial_slot(capacity, 0, int(uniform(uint32_t(sub)))) : 0);
    const uint32_t apart = further ? 27u : 9u;
    auto pslot = [&](uint32_t e) { return own + uint64_t(e) * apart; };
    do {
    if (!valid) break;
    const int j = job_of_tile(frame.jobs, frame.n_jobs, tile);
    const gs_job job = frame.jobs[j];
    const gs_camera& cam = frame.cams[job.cam];
    const int W = cam.width, H = cam.height;
    const int lt = tile - job.tile0;
    const int tx = lt % job.tiles_x, ty = lt / job.tiles_x;
    const int sxn = cfg.tile_w / (8 * QX);
    const int tpx = tx * cfg.tile_w + (ADAPT ? 0 : (sub % sxn) * 8 * QX);
    const int tpy = ty * cfg.tile_h + (ADAPT ? 0 : (sub / sxn) * 8 * QY);
    const int lx = lane & 7, ly = lane >> 3;
    const T bx = T(tpx + lx) + T(0.5), by = T(tpy + ly) + T(0.5);
    const int64_t plane = int64_t(W) * H;
    const T inv = T(job.loss_weight) / T(3 * plane);

    // per pixel: transmittance, dL/dC, what the Gaussians behind contribute,
    // R = sum_c dL/dC_c (C_final_c - C_accumulated_c), and the forward's count
    // of list entries up to its last contributor (nc): a Gaussian is kept
    // at a pixel exactly when alpha >= alpha_min and its list position is
    // below nc, so the forward's stop rule needs no re-evaluation
    T Tr[PPL], gc[PPL][3], R[PPL];
    uint32_t nc[PPL];
    T loss = T(0);
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        const int x = tpx + 8 * (k % QX) + lx, y = tpy + 8 * (k / QX) + ly;
        const bool in = x < W && y < H && (owned & (1u << k));
        Tr[k] = T(1);
        R[k] = T(0);
        gc[k][0] = gc[k][1] = gc[k][2] = T(0);
        nc[k] = 0u;
        if (in) {
            nc[k] = ncontrib[job.px0 + int64_t(y) * W + x];
            const int64_t o = 3 * job.px0 + int64_t(y) * W + x;
#pragma unroll
            for (int ch = 0; ch < 3; ch++) {
                const T c = rgb[o + ch * plane];
                T g;
                if (mode == GS_LOSS_L1) {
                    const T d = c - gin[o + ch * plane];
                    g = d > T(0) ? inv : (d < T(0) ? -inv : T(0));
                    loss += (d < T(0) ? -d : d) * inv;
                } else {
                    g = gin[o + ch * plane];
                }
                gc[k][ch] = g;
                R[k] = Num<T>::fma(g, c, R[k]);
            }
        }
    }
    if (mode == GS_LOSS_L1 && loss_to.out) {
        const T l = wave_sum(loss);
        if (lane == 0) {
            if (loss_to.room(frame.n_tiles)) {
                T* slot = loss_to.slots + 4 * int64_t(tile);
                slot[sub] = l;
                if (sub == 0)
                    for (int q = nwaves; q < 4; q++) slot[q] = T(0);
            } else {
                atomicAdd(loss_to.out + j, l);
            }
        }
    }

    const uint2 range = ranges[tile];
    const T amin = T(cfg.alpha_min), amax = T(cfg.alpha_max);
    const T lmin = Num<T>::log2(amin);
    // per quadrant, the list entries any of its pixels still needs
    uint32_t qend[PPL];
    uint32_t wend = 0u;
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        qend[k] = uniform(wave_max_u32(nc[k]));
        wend = qend[k] > wend ? qend[k] : wend;
    }
    if (NS != 1 && lane == 0) s_wend[wave] = wend;
    for (uint32_t base = range.x; base < range.y; base += kBwdBatch) {
        const uint32_t cnt = min(uint32_t(kBwdBatch), range.y - base);
        const uint32_t pos0 = base - range.x;   // list position of the batch's first entry
        if (NS != 1 && sub > 0 && pos0 >= wend) break;   // the fold does not read this slot past wend
        uint32_t e_own = 0;   // pair this lane stores at the end of the batch
        T w[GS_REC_WORDS];
        uint32_t m = 0, r = 0;
        if (uint32_t(lane) < cnt) {
            r = vals[base + lane];
            const uint32_t pos = pos0 + uint32_t(lane);
            if (pos < wend) {
                load_rec(rec, r, w);
                if (qmask == nullptr) {
                    m = quad_mask<T, QX, QY>(w, tpx, tpy, lmin);
                } else if (ADAPT || NSD == 1) {
                    m = qmask[base + lane];   // the forward's tile mask: this wavefront's quadrants are the tile's
                } else {
                    // the forward's tile mask, bits of this wavefront's sub-tile
                    const uint32_t mt = qmask[base + lane];
                    const int nqx = cfg.tile_w / 8, qx0 = (sub % sxn) * QX, qy0 = (sub / sxn) * QY;
                    m = 0;
#pragma unroll
                    for (int k = 0; k < PPL; k++)
                        m |= ((mt >> ((qy0 + k / QX) * nqx + qx0 + k % QX)) & 1u) << k;
                }
                m &= owned;
#pragma unroll
                for (int k = 0; k < PPL; k++) m &= pos < qend[k] ? ~0u : ~(1u << k);
            }
            // emission index of pair (this tile, r): the record's pairs run
            // row by row over its tile rectangle
            const uint4 mt = meta[r];
            const uint32_t x0 = mt.z & 0xffffu, y0 = mt.z >> 16, x1 = mt.w & 0xffffu;
            e_own = pair_off[r] + (uint32_t(ty) - y0) * (x1 - x0 + 1) + (uint32_t(tx) - x0);
        }
        if (pos0 >= wend) {
            // past every pixel's last contributor: the rest of the tile's
            // pairs carry zero gradient (slot 0 of all of them is stored)
            if (uint32_t(lane) < cnt)
#pragma unroll
                for (int q = 0; q < 9; q++) pslot(e_own)[q] = T(0);
            continue;
        }
        // records that reach some quadrant are staged compacted, with their
        // list position; the others store zero partials below
        const uint64_t staged = __ballot(m != 0);
        const uint32_t slot = __builtin_popcountll(staged & lanemask_lt());
        if (m != 0) {
            const T* src = rec + int64_t(r) * GS_REC_WORDS;
            T* dst = s_rec[wave][slot];
#pragma unroll
            for (int q = 0; q < 6; q++) dst[q] = w[q];
#pragma unroll
            for (int q = 6; q < 9; q++) dst[q] = src[q];
            narrow_axis(w[R_AXIS], dst[S_AXC], dst[S_AXS]);
            s_mask[wave][slot] = m | (uint32_t(lane) << 8);
            s_eown[wave][slot] = e_own;
        } else if (uint32_t(lane) < cnt) {
            // reaches no quadrant this wave owns: zero partials
#pragma unroll
            for (int q = 0; q < 9; q++) pslot(e_own)[q] = T(0);
        }
        wave_lds_sync();
        const uint32_t n = __builtin_popcountll(staged);
        // composites staged record i over the wave's quadrants, leaves its nine
        // partials (per lane) in v; false when no pixel kept it
        auto composite = [&](uint32_t i, T (&v)[9]) -> bool {
            const uint32_t word = uniform(s_mask[wave][i]);
            const uint32_t qmask = word & 0xffu, pos = pos0 + (word >> 8);
            const Rec<T> g = lds_rec(s_rec[wave][i]);
            const T axc = s_rec[wave][i][S_AXC], axs = s_rec[wave][i][S_AXS];
#pragma unroll
            for (int q = 0; q < 9; q++) v[q] = -T(0);   // -0: the first x + v folds to x
            T* mo = v;
            T* dcol = v + 6;
            bool hit = false;   // uniform: some lane kept the record
#pragma unroll
            for (int k = 0; k < PPL; k++) {
                if (!(qmask & (1u << k))) continue;   // uniform: box misses quadrant k
                const T dx = quad_centre(bx, k % QX) - g.mx, dy = quad_centre(by, k / QX) - g.my;
                const T al = Num<T>::exp2(log2_alpha(g, dx, dy));
                const bool keep = al >= amin && pos < nc[k];
                if (__ballot(keep) == 0) continue;     // uniform: no pixel of the wave keeps it
                hit = true;
                // the forward's operations on the kept pixels; zeros elsewhere
                const T a = clamp_alpha(al, amax);
                const T ak = keep ? a : T(0);
                const T wgt = ak * Tr[k];
                const T gcc = Num<T>::fma(gc[k][2], g.c[2], Num<T>::fma(gc[k][1], g.c[1], gc[k][0] * g.c[0]));
                R[k] = Num<T>::fma(-wgt, gcc, R[k]);
                // dL/dalpha = sum_c gc_c (c_c T - (C_final_c - C_acc_c) / (1 - alpha))
                const T ga = Num<T>::fma(Tr[k], gcc, -R[k] * recip(T(1) - a));
#pragma unroll
                for (int ch = 0; ch < 3; ch++) dcol[ch] = Num<T>::fma(gc[k][ch], wgt, dcol[ch]);
                Tr[k] -= wgt;
                // alpha clamped at alpha_max: no gradient to the Gaussian's shape
                const T ge = (al < amax ? ak : T(0)) * ga;
                const T e1 = Num<T>::fma(axc, dx, axs * dy), e2 = Num<T>::fma(axc, dy, -(axs * dx));
                const T t1 = ge * e1, t2 = ge * e2;
                mo[0] += ge;
                mo[1] += t1;
                mo[2] += t2;
                mo[3] = Num<T>::fma(t1, e1, mo[3]);
                mo[4] = Num<T>::fma(t1, e2, mo[4]);
                mo[5] = Num<T>::fma(t2, e2, mo[5]);
            }
            return hit;
        };
        // records in pairs: composited in list order, their partials summed
        // over the wave together and stored
        for (uint32_t i = 0; i < n; i += 2) {
            T va[9], vb[9];
            const bool ha = composite(i, va);
            bool hb = false;
            if (i + 1 < n) {
                hb = composite(i + 1, vb);
            } else {
#pragma unroll
                for (int q = 0; q < 9; q++) vb[q] = T(0);
            }
            T* da = pslot(uniform(s_eown[wave][i]));
            T* db = i + 1 < n ? pslot(uniform(s_eown[wave][i + 1])) : nullptr;
            if (ha || hb) {
                store_pair_partials(va, vb, da, db);
            } else if (lane < 9) {
                da[lane] = T(0);
                if (db) db[lane] = T(0);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    } while (0);

    // A split tile's wavefronts share this workgroup.  Once all of them have
    // stored their partials, fold each pair's further slots into slot 0
    // (slot 0 + 1 + 2 + 3, in that order), so the projection backward reads
    // one dense slot per pair.  Whether a workgroup holds a split tile is the
    // same for all its wavefronts (every one with NS > 1; the plan puts split
    // tiles first), and none of them has left the kernel.
    if (NS != 1) {
        PassPlan plan = {0u, 0u, 0u};
        if (ADAPT) pass_plan<true>(order, frame.n_tiles, plan);
        if (!ADAPT || 4ull * blockIdx.x < 4ull * plan.m4 + 2ull * plan.m2) {
            __syncthreads();
            if (valid && nwaves > 1) {
                const int jf = job_of_tile(frame.jobs, frame.n_jobs, tile);
                const gs_job jb = frame.jobs[jf];
                const int ltf = tile - jb.tile0;
                const uint32_t ftx = uint32_t(ltf % jb.tiles_x), fty = uint32_t(ltf / jb.tiles_x);
                const uint2 rg = ranges[tile];
                // entries past what the further wavefronts' pixels need have nothing to fold
                const int w0 = wave - sub;
                uint32_t end = 0u;
                for (int sl = 1; sl < nwaves; sl++) end = max(end, s_wend[w0 + sl]);
                end = min(end, rg.y - rg.x);
                for (uint32_t pos = uint32_t(sub * kWave + lane); pos < end; pos += uint32_t(nwaves * kWave)) {
                    const uint32_t r = vals[rg.x + pos];
                    const uint4 mt = meta[r];
                    const uint32_t x0 = mt.z & 0xffffu, y0 = mt.z >> 16, x1 = mt.w & 0xffffu;
                    const uint32_t e = pair_off[r] + (fty - y0) * (x1 - x0 + 1) + (ftx - x0);
                    T* d0 = pg + partial_slot(capacity, e, 0);
                    T acc[9];
#pragma unroll
                    for (int q = 0; q < 9; q++) acc[q] = d0[q];
                    for (int sl = 1; sl < nwaves; sl++) {
                        if (pos >= s_wend[w0 + sl]) continue;
                        const T* src = pg + partial_slot(capacity, e, sl);
#pragma unroll
                        for (int q = 0; q < 9; q++) acc[q] += src[q];
                    }
#pragma unroll
                    for (int q = 0; q < 9; q++) d0[q] = acc[q];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------

// Wavefronts per tile of a launch (0: the plan's): what the configuration
// asks for, except that a frame of few tiles, which one wavefront per tile
// would leave most of the chip's 1,024 SIMDs idle with, takes 4 (at most the
// tile's quadrants) up to fill4 tiles, and 2 up to fill2 tiles; a pass that
// splits by the plan takes 4 up to fill_plan tiles.  The lines lie where the
// split stops paying on scenes of long uneven lists (the scale scene's 500k
// Gaussians), of even ones (30k of the parity scene's) and of lists that end
// early (200k of them), 16x16 tiles, us with 1 / 2 / 4 / the plan:
//   forward,  1,617 tiles: 227 / 141 / 122 / 142, 91 / 62 / 61 / 83, 97 / 69 / 67 / 99;
//             2,072 tiles: 192 / 127 / 128 / 120, 81 / 64 / 67 / 79, 95 / 75 / 77 / 102;
//             4,056 tiles: 132 / 126 / 134 / 85, 85 / 85 / 93 / 75, 103 / 96 / 108 / 109;
//   backward,   988 tiles: 601 / 383 / 300 / 398, 157 / 129 / 128 / 168, 168 / 150 / 150 / 181;
//             1,350 tiles: 543 / 368 / 313 / 333, 162 / 130 / 140 / 152, 182 / 164 / 179 / 185;
//             1,617 tiles: 453 / 314 / 299 / 289, 153 / 138 / 152 / 146, 170 / 193 / 198 / 183.
// (The backward pays for each split with another reduction per record.)
struct FillRule {
    int fill4, fill2, fill_plan;
};
constexpr FillRule kFwdFill = {1800, 3600, 1800};
constexpr FillRule kBwdFill = {1000, 1400, 1400};
static int launch_waves(const gs_raster_cfg& cfg, int waves, int n_tiles, const FillRule& f) {
    if (waves > 1) return waves;
    const int quads = (cfg.tile_w / 8) * (cfg.tile_h / 8);
    if (n_tiles <= (waves == 0 ? f.fill_plan : f.fill4)) return quads < 4 ? quads : 4;
    if (waves == 1 && n_tiles <= f.fill2) return quads < 2 ? quads : 2;
    return waves;
}

// grid of a compositing launch: NS (or 4, adaptive) wavefronts per tile, in
// workgroups of kRenderWaves wavefronts (1, adaptive)
template <int NS>
static void compositing_grid(const gs_frame& f, dim3& grid, dim3& block) {
    const int wpt = NS == 0 ? 4 : NS;   // adaptive: at most 4 per tile, the plan's count
    grid = dim3(unsigned((int64_t(f.n_tiles) * wpt + kRenderWaves - 1) / kRenderWaves));
    block = dim3(unsigned(kWave * kRenderWaves));
}

template <typename T, int QX, int QY, int NS>
static void fwd_launch(const gs_frame& f, const gs_raster_cfg& cfg, const T* rec, const gs_bins& b, T* rgb,
                       T* Tfin, uint32_t* nc, unsigned long long* kept, hipStream_t s) {
    dim3 grid, block;
    compositing_grid<NS>(f, grid, block);
    if (kept)
        GS_LAUNCH("k_render_fwd", (k_render_fwd<T, QX, QY, NS, true>), grid, block, 0, s, f, cfg, rec, b.vals,
                  reinterpret_cast<const uint2*>(b.ranges), rgb, Tfin, nc, kept, b.tile_order, b.qmask);
    else
        GS_LAUNCH("k_render_fwd", (k_render_fwd<T, QX, QY, NS, false>), grid, block, 0, s, f, cfg, rec, b.vals,
                  reinterpret_cast<const uint2*>(b.ranges), rgb, Tfin, nc, kept, b.tile_order, b.qmask);
}

template <typename T, int QX, int QY, int NS>
static void bwd_launch(const gs_frame& f, const gs_raster_cfg& cfg, const T* rec, const uint32_t* meta,
                       const gs_bins& b, const T* rgb, const uint32_t* nc, int mode, const T* gin,
                       const LossSum<T>& loss, T* pg, hipStream_t s) {
    dim3 grid, block;
    compositing_grid<NS>(f, grid, block);
    GS_LAUNCH("k_render_bwd", (k_render_bwd<T, QX, QY, NS>), grid, block, 0, s, f, cfg, rec,
              reinterpret_cast<const uint4*>(meta), b.pair_off, b.vals, reinterpret_cast<const uint2*>(b.ranges),
              b.tile_order, b.capacity, rgb, nc, mode, gin, loss, pg, b.qmask);
}

// (binning tile, wavefronts per tile) -> quadrants per wavefront QX x QY:
// 8x8/1 = 1x1; 16x8/1 = 2x1, /2 = 1x1; 16x16/1 = 2x2, /2 = 2x1 (halves stacked),
// /4 = 1x1; 32x8/1 = 4x1, /2 = 2x1 (halves side by side), /4 = 1x1.  Adaptive
// (WAVES = 0): the whole tile's quadrants, split per tile at run time.
#define GS_TILE_DISPATCH(WAVES, FN, ...)                                                  \
    do {                                                                                  \
        const int S_ = WAVES;                                                             \
        if (cfg.tile_w == 8 && cfg.tile_h == 8) {                                         \
            if (S_ == 0) FN<T, 1, 1, 0>(__VA_ARGS__);                                     \
            else FN<T, 1, 1, 1>(__VA_ARGS__);                                             \
        } else if (cfg.tile_w == 16 && cfg.tile_h == 8) {                                 \
            if (S_ == 0) FN<T, 2, 1, 0>(__VA_ARGS__);                                     \
            else if (S_ == 2) FN<T, 1, 1, 2>(__VA_ARGS__);                                \
            else FN<T, 2, 1, 1>(__VA_ARGS__);                                             \
        } else if (cfg.tile_w == 32 && cfg.tile_h == 8) {                                 \
            if (S_ == 0) FN<T, 4, 1, 0>(__VA_ARGS__);                                     \
            else if (S_ == 4) FN<T, 1, 1, 4>(__VA_ARGS__);                                \
            else if (S_ == 2) FN<T, 2, 1, 2>(__VA_ARGS__);                                \
            else FN<T, 4, 1, 1>(__VA_ARGS__);                                             \
        } else {                                                                          \
            if (S_ == 0) FN<T, 2, 2, 0>(__VA_ARGS__);                                     \
            else if (S_ == 4) FN<T, 1, 1, 4>(__VA_ARGS__);                                \
            else if (S_ == 2) FN<T, 2, 1, 2>(__VA_ARGS__);                                \
            else FN<T, 2, 2, 1>(__VA_ARGS__);                                             \
        }                                                                                 \
    } while (0)

template <typename T>
hipError_t launch_render_fwd(const gs_frame& f, const gs_raster_cfg& cfg, const T* rec, const gs_bins& bins,
                             T* rgb, T* Tfin, uint32_t* ncontrib, unsigned long long* kept, hipStream_t s) {
    if (f.n_tiles == 0) return hipSuccess;
    GS_TILE_DISPATCH(launch_waves(cfg, fwd_waves(cfg), f.n_tiles, kFwdFill), fwd_launch, f, cfg, rec, bins, rgb, Tfin, ncontrib, kept, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_render_bwd(const gs_frame& f, const gs_raster_cfg& cfg, const T* rec, const uint32_t* meta,
                             const gs_bins& bins, const T* rgb, const uint32_t* nc, gs_loss_mode mode, const T* gin,
                             const LossSum<T>& loss, T* pg, hipStream_t s) {
    if (f.n_tiles == 0) return hipSuccess;
    GS_TILE_DISPATCH(launch_waves(cfg, bwd_waves(cfg), f.n_tiles, kBwdFill), bwd_launch, f, cfg, rec, meta, bins, rgb, nc, int(mode), gin, loss, pg, s);
    return hipGetLastError();
}

template hipError_t launch_render_fwd<float>(const gs_frame&, const gs_raster_cfg&, const float*, const gs_bins&, float*, float*, uint32_t*, unsigned long long*, hipStream_t);
template hipError_t launch_render_fwd<double>(const gs_frame&, const gs_raster_cfg&, const double*, const gs_bins&, double*, double*, uint32_t*, unsigned long long*, hipStream_t);
template hipError_t launch_render_bwd<float>(const gs_frame&, const gs_raster_cfg&, const float*, const uint32_t*, const gs_bins&, const float*, const uint32_t*, gs_loss_mode, const float*, const LossSum<float>&, float*, hipStream_t);
template hipError_t launch_render_bwd<double>(const gs_frame&, const gs_raster_cfg&, const double*, const uint32_t*, const gs_bins&, const double*, const uint32_t*, gs_loss_mode, const double*, const LossSum<double>&, double*, hipStream_t);

}  // namespace gs
