// Device-side helpers shared by the libgs kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gs.h"

namespace gs {

constexpr int kWave = 64;

// 16-byte accesses with the non-temporal hint, for state that one step
// touches once (the optimiser's moments and the consensus target): they
// keep it from evicting the lines that the same kernel reads again.  Any
// element may be the first (4-byte alignment: planes of an odd stride)
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ inline float4 load4(const float* p) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline void store4(float* p, float4 v) {
    const f32x4 w = {v.x, v.y, v.z, v.w};
    *reinterpret_cast<f32x4*>(p) = w;
}
__device__ inline float4 load_stream4(const float* p) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline void store_stream4(float* p, float4 v) {
    const f32x4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<f32x4*>(p));
}

// ---------------------------------------------------------------------------
// scalar-type traits: FP32 product path, FP64 instantiation for adjoint checks

template <typename T> struct Num;
template <> struct Num<float> {
    __device__ static inline float exp2(float x) { return __builtin_amdgcn_exp2f(x); }
    __device__ static inline float log2(float x) { return __log2f(x); }
    __device__ static inline float exp(float x) { return __expf(x); }
    __device__ static inline float log(float x) { return __logf(x); }
    __device__ static inline float sqrt(float x) { return __builtin_sqrtf(x); }
    __device__ static inline float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }   // hardware, ~1 ulp
    __device__ static inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }    // hardware, ~1 ulp
    __device__ static inline float fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
    __device__ static inline float max(float a, float b) { return __builtin_fmaxf(a, b); }
    __device__ static inline float min(float a, float b) { return __builtin_fminf(a, b); }
};
template <> struct Num<double> {
    __device__ static inline double exp2(double x) { return ::exp2(x); }
    __device__ static inline double log2(double x) { return ::log2(x); }
    __device__ static inline double exp(double x) { return ::exp(x); }
    __device__ static inline double log(double x) { return ::log(x); }
    __device__ static inline double sqrt(double x) { return ::sqrt(x); }
    __device__ static inline double rsqrt(double x) { return 1.0 / ::sqrt(x); }
    __device__ static inline double rcp(double x) { return 1.0 / x; }
    __device__ static inline double fma(double a, double b, double c) { return ::fma(a, b, c); }
    __device__ static inline double max(double a, double b) { return ::fmax(a, b); }
    __device__ static inline double min(double a, double b) { return ::fmin(a, b); }
};

// ln 2 and log2 e as the scalar type
template <typename T> __device__ constexpr T kLn2() { return T(0.69314718055994530942); }
template <typename T> __device__ constexpr T kLog2e() { return T(1.44269504088896340736); }

// ---------------------------------------------------------------------------
// Frame of the compositing backward's second moments.  A footprint much
// longer than it is wide puts almost all of sum ge (p - m)(p - m)^T along its
// long axis, while the gradient of the screen covariance is dominated by the
// part across it; taken from pixel-frame sums, that part would come out of a
// near-cancellation.  So the backward accumulates the moments in the
// footprint's axes: e1 along the axis of the conic's largest eigenvalue (the
// narrow one) and e2 across it.  The projection stores that axis as one word,
// t = tan(theta / 2) of its direction (cos theta, sin theta) with
// cos theta >= 0, and every user decodes the same word with the same
// operations, so all of them rotate by the same matrix.

// code of the narrow axis of the conic [[a, b], [b, c]] (any axis when a = c
// and b = 0)
template <typename T>
__device__ inline T narrow_axis_code(T a, T b, T c) {
    const T h = T(0.5) * (a - c);
    const T r = Num<T>::sqrt(Num<T>::fma(h, h, b * b));
    // eigenvector of the eigenvalue (a + c) / 2 + r, from the better-conditioned row
    T vx = h >= T(0) ? h + r : b;
    T vy = h >= T(0) ? b : r - h;
    const T n2 = Num<T>::fma(vx, vx, vy * vy);
    if (!(n2 > T(0))) return T(0);
    const T inv = Num<T>::rsqrt(n2);
    vx *= inv;
    vy *= inv;
    if (vx < T(0)) {
        vx = -vx;
        vy = -vy;
    }
    return vy / (T(1) + vx);
}

// (cos theta, sin theta) of a narrow-axis code
template <typename T>
__device__ inline void narrow_axis(T t, T& c, T& s) {
    const T w = T(1) / Num<T>::fma(t, t, T(1));
    c = Num<T>::fma(-t, t, T(1)) * w;
    s = (t + t) * w;
}

// ---------------------------------------------------------------------------
// per-record metadata word 1: covered tiles in the low 24 bits, the colour
// clamp of each channel (SH sum + 0.5 <= 0) in bits 24..26

// compositing wavefronts per tile of the forward and the backward (0 reads
// as 1; GS_WAVES_ADAPTIVE in the backward: per tile, see adaptive_waves)
__host__ __device__ inline int fwd_waves(const gs_raster_cfg& c) {
    return c.fwd_waves == GS_WAVES_ADAPTIVE ? 0 : (c.fwd_waves <= 1 ? 1 : c.fwd_waves);
}
__host__ __device__ inline bool bwd_adaptive(const gs_raster_cfg& c) { return c.bwd_waves == GS_WAVES_ADAPTIVE; }
__host__ __device__ inline int bwd_waves(const gs_raster_cfg& c) {
    return bwd_adaptive(c) ? 0 : (c.bwd_waves <= 1 ? 1 : c.bwd_waves);
}

// Most wavefronts of one tile in an adaptive compositing pass (its group in
// the plan), from its list length against the frame's mean list length: 4
// above 4 x the mean, 2 above 1.25 x, else 1; never more than the tile's
// quadrants.  Exact integer arithmetic, so every kernel that needs it agrees.
__device__ inline int adaptive_waves(uint32_t count, uint32_t pairs, int n_tiles, int quads) {
    const uint64_t a = 4ull * count * uint64_t(n_tiles);
    const int s = a > 16ull * pairs ? 4 : (a > 5ull * pairs ? 2 : 1);
    return s < quads ? s : quads;
}

// How much of a frame's plan a compositing pass splits.  The plan lists the
// tiles longest first (its wavefront groups, then buckets of half the mean
// list length); a pass splits a leading run of it, over 4 wavefronts in the
// plan's first group and 2 beyond.  A tile is worth splitting when its list
// alone would outlast the launch: when it is longer than the entries per
// resident wavefront by some factor, so the line moves with n_tiles / resident
// wavefronts, in units of the mean list length; below some 5,000 tiles the
// plan's 1.25 (forward) and 2 (backward; below 2,400 tiles 1.5) times the mean
// take over.  Splitting below the line repeats staging and, in the backward,
// each record's reduction and store for nothing.  Measured, us with every tile
// above 1.25x the mean split / with the line here / with no split (1600x1066
// unless noted; Gaussians of the scale scene; three views: 1280x720, 800x600
// and 1920x1080):
//   backward: 500k 201-217 / 164 / 184; 3M 775 / 467 / 443; three views of
//             800k 692 / 542 / 542; four views of 1.5M 2073 / 1551 / 1551;
//             500k at 979x651 227 / 218 / 334;
//             the whole backward above 1.5x / 2x the mean: 500k 304 / 304 at
//             1,520 tiles, 278 / 277 at 1,900, 236 / 232 at 2,542, and the
//             parity scene's 200k 264 / 315, 229 / 275, 226 / 238;
//   forward:  500k 68-74 / 68 / 99; 3M 201 / 200 / 204; three views of 800k
//             213 / 183 / 202; four of 1.5M 602 / 530 / 530.
// Line in half means, rounded: the bucket from which tiles are split.
__host__ __device__ inline int fwd_split_bucket(int n_tiles) {
    const int b = (n_tiles + 1080) / 2160;     // 1.66 x entries per wavefront at 7 per SIMD
    return b < 3 ? 2 : b;                      // 2: every tile of the plan's groups
}
__host__ __device__ inline int bwd_split_bucket(int n_tiles) {
    const int b = (n_tiles + 560) / 1120;      // 1.83 x entries per wavefront at 4 per SIMD
    const int least = n_tiles < 2400 ? 3 : 4;
    return b < least ? least : b;
}

// The plan a pass runs (word 3 of the plan array holds the share of the list
// it splits, in 1/65536: the forward's in the low half, the backward's in the
// high half): tiles taking 4, 2 and 1 wavefronts, in list order; false for an
// array that does not describe n_tiles tiles.
struct PassPlan {
    uint32_t m4, m2, m1;
};
template <bool BWD>
__device__ inline bool pass_plan(const uint32_t* __restrict__ order, int n_tiles, PassPlan& p) {
    const uint32_t nt = uint32_t(n_tiles), n4 = order[0], n2 = order[1], n1 = order[2];
    p = {0u, 0u, 0u};
    if (n4 > nt || n2 > nt || n1 > nt || n4 + n2 + n1 != nt) return false;
    const uint32_t share = BWD ? order[3] >> 16 : order[3] & 0xffffu;
    const uint32_t split = min(uint32_t((uint64_t(share) * nt) >> 16), n4 + n2);
    p.m4 = min(n4, split);
    p.m2 = split - p.m4;
    p.m1 = nt - split;
    return true;
}

// Wavefront gw of an adaptive compositing launch -> (tile, sub, waves) from
// the plan; false when the wavefront has no work.
template <bool BWD>
__device__ inline bool plan_wave(const uint32_t* __restrict__ order, int n_tiles, uint32_t gw, int& tile, int& sub,
                                 int& waves) {
    PassPlan p;
    if (!pass_plan<BWD>(order, n_tiles, p)) return false;
    const uint32_t* list = order + 4;
    uint32_t g = gw, t;
    if (g < 4u * p.m4) {
        t = list[g / 4u];
        sub = int(g % 4u);
        waves = 4;
    } else if ((g -= 4u * p.m4) < 2u * p.m2) {
        t = list[p.m4 + g / 2u];
        sub = int(g % 2u);
        waves = 2;
    } else if ((g -= 2u * p.m2) < p.m1) {
        t = list[p.m4 + p.m2 + g];
        sub = 0;
        waves = 1;
    } else {
        return false;
    }
    tile = int(t);
    return t < uint32_t(n_tiles);
}

// Partials of wavefront `sub` for pair e: slot 0 of every pair dense at e,
// the slots of the further wavefronts of split tiles after all of them (3
// per pair), so a one-wavefront tile's pairs stay contiguous.  The split
// tiles' wavefronts fold theirs into slot 0, the only one the projection
// backward reads.  Capacity counts pairs; 9 values per slot.
__host__ __device__ inline int64_t partial_slot(uint64_t capacity, uint64_t e, int sub) {
    return sub == 0 ? int64_t(e) * 9 : (int64_t(capacity) + int64_t(e) * 3 + (sub - 1)) * 9;
}

// Where the compositing backward leaves the L1 loss of wavefront `sub` of a
// tile: the last 4 n_tiles values of the partials' workspace (4 per tile),
// free when the frame's pairs leave that much of the further slots unused;
// the projection backward's launch then adds them up, a workgroup per job, in
// a fixed order.  Without the room every wavefront adds its own sum to the
// job's loss: some thousand same-address FP32 atomics in no fixed order,
// whose rounding reached 1e-6 of the loss.
template <typename T>
struct LossSum {
    T* slots;                   // 4 per tile
    T* out;                     // per job; null: no loss wanted
    const uint32_t* counters;
    uint64_t capacity;
    __device__ bool room(int n_tiles) const {
        const uint64_t pairs = counters[GS_CTR_PAIRS];   // 0: none, or the caller has cleared the counters since
        return pairs > 0 && pairs < capacity && (capacity - pairs) * 27u >= 4ull * uint64_t(n_tiles);
    }
};
template <typename T>
inline LossSum<T> loss_sum(T* ws, T* out, const uint32_t* counters, uint64_t capacity, int n_tiles) {
    const int64_t at = int64_t(capacity) * 36 - 4 * int64_t(n_tiles);
    return {out && at > 0 ? ws + at : ws, out, counters, capacity};
}

// quadrants (bit k = quadrant k of the tile) owned by wavefront `sub` of `waves`
__device__ inline uint32_t owned_quadrants(int quads, int waves, int sub) {
    const int per = quads / waves;
    return ((1u << per) - 1u) << (sub * per);
}

constexpr uint32_t kTilesMask = 0xffffffu;
__host__ __device__ inline uint32_t meta_tiles(uint32_t y) { return y & kTilesMask; }
__host__ __device__ inline uint32_t meta_clamp(uint32_t y) { return (y >> 24) & 7u; }

// ---------------------------------------------------------------------------
// job lookup: jobs are laid out in ascending rec0 / tile0 / px0 order

__device__ inline int job_of_record(const gs_job* __restrict__ jobs, int n_jobs, int64_t r) {
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].rec0 <= r) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ inline int job_of_tile(const gs_job* __restrict__ jobs, int n_jobs, int tile) {
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].tile0 <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// wave64 primitives

__device__ inline int lane_id() { return __lane_id(); }

__device__ inline uint64_t lanemask_lt() { return (uint64_t(1) << lane_id()) - 1; }

// lanes where b holds, as a wave-uniform 64-bit mask (every lane active)
__device__ inline uint64_t lane_mask(bool b) { return __builtin_amdgcn_ballot_w64(b); }
// this lane's bit of a wave-uniform lane mask, read as a per-lane condition
// without moving the mask into vector registers
__device__ inline bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Sum over the 64 lanes of a wave, returned to every lane.  FP32 uses DPP
// (quad permutes, row rotations, then row broadcasts into lane 63); FP64
// uses a butterfly of cross-lane shuffles.
template <int CTRL, int ROW_MASK>
__device__ inline float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

// DPP move over all rows and banks in which a lane without a source reads 0
template <int CTRL>
__device__ inline float dpp_move_bc(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

__device__ inline float wave_sum(float v) {
    v += dpp_move<0xb1, 0xf>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4e, 0xf>(v);   // quad_perm [2,3,0,1]
    v += dpp_move<0x124, 0xf>(v);  // row_ror:4
    v += dpp_move<0x128, 0xf>(v);  // row_ror:8
    v += dpp_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Sum over each row of 16 lanes, complete in the row's last lane (15):
// quad sums, then shifts right by 4 and 8 lanes within the row (lanes with
// no source add zero), so every step is one fused DPP add.
__device__ inline float row_sum_last(float v) {
    v += dpp_move_bc<0xb1>(v);    // quad_perm [1,0,3,2]
    v += dpp_move_bc<0x4e>(v);    // quad_perm [2,3,0,1]
    v += dpp_move_bc<0x114>(v);   // row_shr:4
    v += dpp_move_bc<0x118>(v);   // row_shr:8
    return v;
}

// (the two halves of a double moved by the same DPP steps)
template <int CTRL>
__device__ inline double dpp_move_bc_f64(double v) {
    const uint64_t u = uint64_t(__double_as_longlong(v));
    const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(u)), CTRL, 0xf, 0xf, true));
    const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(u >> 32)), CTRL, 0xf, 0xf, true));
    return __longlong_as_double((long long)(uint64_t(lo) | uint64_t(hi) << 32));
}
__device__ inline double row_sum_last(double v) {
    v += dpp_move_bc_f64<0xb1>(v);
    v += dpp_move_bc_f64<0x4e>(v);
    v += dpp_move_bc_f64<0x114>(v);
    v += dpp_move_bc_f64<0x118>(v);
    return v;
}

__device__ inline double wave_sum(double v) {
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// DPP move of a 32-bit word; lanes without a source (or outside the row mask)
// read `old`
template <int CTRL, int ROW_MASK>
__device__ inline uint32_t dpp_u32(uint32_t old, uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(old), int(v), CTRL, ROW_MASK, 0xf, false));
}

// smallest / largest value over the wave (wave-uniform)
__device__ inline uint32_t wave_min_u32_dpp(uint32_t v) {
    v = min(v, dpp_u32<0xb1, 0xf>(v, v));     // quad_perm [1,0,3,2]
    v = min(v, dpp_u32<0x4e, 0xf>(v, v));     // quad_perm [2,3,0,1]
    v = min(v, dpp_u32<0x124, 0xf>(v, v));    // row_ror:4
    v = min(v, dpp_u32<0x128, 0xf>(v, v));    // row_ror:8
    v = min(v, dpp_u32<0x142, 0xa>(v, v));    // row_bcast:15 into rows 1 and 3
    v = min(v, dpp_u32<0x143, 0xc>(v, v));    // row_bcast:31 into rows 2 and 3
    return uint32_t(__builtin_amdgcn_readlane(int(v), 63));
}
__device__ inline uint32_t wave_max_u32_dpp(uint32_t v) { return ~wave_min_u32_dpp(~v); }

// inclusive prefix sum over the lanes of a wave
__device__ inline uint32_t wave_incl_scan_dpp(uint32_t v) {
    v += dpp_u32<0x111, 0xf>(0u, v);          // row_shr:1
    v += dpp_u32<0x112, 0xf>(0u, v);          // row_shr:2
    v += dpp_u32<0x114, 0xf>(0u, v);          // row_shr:4
    v += dpp_u32<0x118, 0xf>(0u, v);          // row_shr:8
    v += dpp_u32<0x142, 0xa>(0u, v);          // row_bcast:15 into rows 1 and 3
    v += dpp_u32<0x143, 0xc>(0u, v);          // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ inline uint32_t wave_sum_u32(uint32_t v) {
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ inline uint32_t wave_max_u32(uint32_t v) {
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t o = __shfl_xor(v, off, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// One workgroup (of up to 1024 threads): adds job j's loss, left per tile and
// wavefront by the compositing backward, to out[j].
template <typename T>
__device__ inline void add_job_loss(const gs_frame& frame, const LossSum<T>& L, int j) {
    __shared__ T s_sum[16];
    if (!L.room(frame.n_tiles)) return;     // uniform: the wavefronts added theirs themselves
    const gs_job& job = frame.jobs[j];
    const T* src = L.slots + 4 * int64_t(job.tile0);
    const int64_t n = 4 * int64_t(job.tiles_x) * job.tiles_y;
    T acc = T(0);
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) acc += src[i];
    acc = wave_sum(acc);
    if (lane_id() == 0) s_sum[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T t = T(0);
        for (int w = 0; w < int(blockDim.x) / kWave; w++) t += s_sum[w];
        atomicAdd(L.out + j, t);
    }
}

// ---------------------------------------------------------------------------
// XCD-aware block order: the dispatcher hands consecutive workgroups to the
// 8 XCDs round robin.  Remapping so that each XCD receives one contiguous run
// of work items keeps neighbouring tiles (which share Gaussians) in the same
// L2.
__device__ inline int xcd_block(int b, int nb) {
    const int xcd = b & 7, idx = b >> 3;
    const int per = nb >> 3, rem = nb & 7;
    const int base = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
    return base + idx;
}

}  // namespace gs
