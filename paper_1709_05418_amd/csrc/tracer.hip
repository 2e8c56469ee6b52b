// Monte Carlo transport in the cloud (Sec. 3.2 Eq. (1), Sec. 4, Sec. 4.4, Sec. 5.1):
// delta tracking against a global majorant, ratio-tracked transmittance toward the
// light, Henyey-Greenstein scattering, absorption by Russian roulette.  A path is walked
// by a team of lanes (k_paths), a short one by one thread; per-record sums of the path estimates are accumulated in
// FP64 and reduced in a fixed order, so results are reproducible bit for bit.
#include <math.h>

#include "internal.h"
#include "stream.h"

namespace ds {
namespace {

constexpr int kPaths = 64;                  // paths per partial sum of a record
constexpr int64_t kMaxSteps = 1ll << 26;    // hard bound on tentative collisions per path

// ------------------------------------------------------------------ random words
struct Rng {
    uint32_t k0, k1;        // key = seed
    uint32_t c0, c1, c2, c3; // counter = (stream id lo, hi, block, 0)
    uint32_t buf[4];
    int used;

    __device__ void init(uint64_t seed, uint64_t id)
    {
        k0 = (uint32_t)seed;
        k1 = (uint32_t)(seed >> 32);
        c0 = (uint32_t)id;
        c1 = (uint32_t)(id >> 32);
        c2 = 0;
        c3 = 0;
        used = 4;
    }
    __device__ void refill()
    {
        philox(k0, k1, c0, c1, c2, c3, buf);
        if (++c2 == 0)
            ++c3;
        used = 0;
    }
    // the top 24 bits of the next word
    __device__ uint32_t bits24()
    {
        if (used == 4)
            refill();
        return buf[used++] >> 8;
    }
    // uniform in [0, 1) on the 2^-24 grid
    __device__ float u() { return (float)bits24() * (1.f / 16777216.f); }
};

__device__ __forceinline__ float unit24(uint32_t k) { return (float)k * (1.f / 16777216.f); }

// Member of a light set drawn by one uniform's top 24 bits k: the first j with
// k < thr[j] (thresholds strictly increasing, the last 2^24), by binary search.
__device__ __forceinline__ int set_pick(const TracerParams &tp, uint32_t k)
{
    int lo = 0, hi = tp.set_m - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (k < tp.set_thr[mid])
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// ------------------------------------------------------------------ geometry helpers
struct V3 {
    float x, y, z;
};
__host__ __device__ __forceinline__ V3 v3(float x, float y, float z) { return V3{x, y, z}; }
// Products are fused in a fixed order, the same wherever the function is inlined.
__device__ __forceinline__ float dot(V3 a, V3 b)
{
    return fmaf(a.z, b.z, fmaf(a.x, b.x, a.y * b.y));
}
__device__ __forceinline__ float dot_direct(V3 a, V3 b)  // of the direct terms
{
    return fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x));
}
__device__ __forceinline__ V3 neg(V3 a) { return v3(-a.x, -a.y, -a.z); }
__device__ __forceinline__ V3 madd(V3 a, float t, V3 d) { return v3(a.x + t * d.x, a.y + t * d.y, a.z + t * d.z); }

__device__ __forceinline__ bool unit(const float *v, V3 &u)
{
    float a = v[0], b = v[1], c = v[2];
    if (!(isfinite(a) && isfinite(b) && isfinite(c)))
        return false;
    float m = fmaxf(fabsf(a), fmaxf(fabsf(b), fabsf(c)));
    if (m == 0.f)
        return false;
    a /= m;
    b /= m;
    c /= m;
    float l = sqrtf(a * a + b * b + c * c);
    u = v3(a / l, b / l, c / l);
    return true;
}

// Orthonormal pair around unit n (branchless construction of Duff et al. 2017).
__device__ __forceinline__ void basis(V3 n, V3 &t1, V3 &t2)
{
    const float sg = copysignf(1.f, n.z);
    const float a = -1.f / (sg + n.z);
    const float b = n.x * n.y * a;
    t1 = v3(1.f + sg * n.x * n.x * a, sg * b, -sg * n.x);
    t2 = v3(b, sg + n.y * n.y * a, -n.y);
}

// ------------------------------------------------------------------ medium
struct Medium {
    const float4 *cells;  // corner-packed extinction: cell c = entries 2c, 2c + 1
    int cx, cy;           // cell-grid dims in x and y (grid dims + 2)
    float hx, hy, hz;     // clamp bounds of the shifted cell coordinate (grid dims + 1)
    V3 amin, amax;
    float inv_h, maj;
    float inv_ff;         // mean free-flight length 1 / (maj * extinction scale); the scale
                          // thins the medium uniformly (the chop of a tabulated phase
                          // function), so collision and transmittance ratios keep maj
    unsigned long long *truncated;  // paths stopped at kMaxSteps (the context's counter)
    // Occupied bricks (2^occ_s cells per axis) as bits, brick (i, j, k) at bit
    // i + bx (j + by k); a clear bit says that every cell of the brick is zero.  Entry
    // occ_words is 1 if a transmittance factor 1 - mu / maj may not be finite.
    const uint32_t *occ;
    int occ_s, bx, by, occ_words;
};

// A path whose tentative collisions reach kMaxSteps stops there; the call that crosses
// the bound counts it once in the context's counter (s0: the path's count before the call).
__device__ __forceinline__ void note_cap(const Medium &M, int64_t s0, int64_t steps)
{
    if (steps >= kMaxSteps && s0 < kMaxSteps && M.truncated)
        atomicAdd(M.truncated, 1ull);
}

// Voxel-centred trilinear extinction, zero outside the grid.  The cell coordinate (the
// voxel-centred coordinate plus one), clamped to [0, n + 1], selects a cell whose eight
// corners are the lattice values around the point; the border cells hold zeros, so points
// outside the grid read zero without tests.
__device__ __forceinline__ float mu_lerp(float4 lo, float4 hi, float fx, float fy, float fz)
{
    // corner c = dx + 2 dy + 4 dz
    const float a00 = fmaf(fx, lo.y - lo.x, lo.x), a10 = fmaf(fx, lo.w - lo.z, lo.z);
    const float a01 = fmaf(fx, hi.y - hi.x, hi.x), a11 = fmaf(fx, hi.w - hi.z, hi.z);
    const float b0 = fmaf(fy, a10 - a00, a00), b1 = fmaf(fy, a11 - a01, a01);
    return fmaf(fz, b1 - b0, b0);
}

__device__ float mu_at(const Medium &M, V3 p)
{
    const float ux = __builtin_amdgcn_fmed3f((p.x - M.amin.x) * M.inv_h + 0.5f, 0.f, M.hx);
    const float uy = __builtin_amdgcn_fmed3f((p.y - M.amin.y) * M.inv_h + 0.5f, 0.f, M.hy);
    const float uz = __builtin_amdgcn_fmed3f((p.z - M.amin.z) * M.inv_h + 0.5f, 0.f, M.hz);
    const uint32_t i = (uint32_t)ux, j = (uint32_t)uy, k = (uint32_t)uz;
    const float fx = __builtin_amdgcn_fractf(ux), fy = __builtin_amdgcn_fractf(uy),
                fz = __builtin_amdgcn_fractf(uz);
    const int64_t cell = (int64_t)i + (int64_t)M.cx * ((int64_t)j + (int64_t)M.cy * k);
    return mu_lerp(M.cells[2 * cell], M.cells[2 * cell + 1], fx, fy, fz);
}

// Parametric interval [t0, t1] of o + t d inside the grid box, t >= 0.
__device__ bool clip(const Medium &M, V3 o, V3 d, float &t0, float &t1)
{
    float lo = 0.f, hi = INFINITY;
    t0 = t1 = 0.f;
    const float oo[3] = {o.x, o.y, o.z}, dd[3] = {d.x, d.y, d.z};
    const float mn[3] = {M.amin.x, M.amin.y, M.amin.z}, mx[3] = {M.amax.x, M.amax.y, M.amax.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (dd[a] != 0.f) {
            float ta = (mn[a] - oo[a]) / dd[a], tb = (mx[a] - oo[a]) / dd[a];
            if (ta > tb) {
                const float s = ta;
                ta = tb;
                tb = s;
            }
            lo = fmaxf(lo, ta);
            hi = fminf(hi, tb);
        } else if (oo[a] < mn[a] || oo[a] > mx[a]) {
            return false;
        }
    }
    t0 = lo;
    t1 = hi;
    return hi > lo;
}

// Exponential free-flight length in units of the mean free path, -ln(1 - u), for u on the
// 2^-24 grid in [0, 1): 1 - u is exact and at least 2^-24, so the hardware base-2 logarithm
// (v_log_f32, no denormal inputs here) times ln 2 serves.
__device__ __forceinline__ float exp_flight(float u)
{
    return -__builtin_amdgcn_logf(1.f - u) * 0.693147180559945f;
}

// Free flight from o along unit d: true and the collision point, false on escape.
__device__ bool delta_track(const Medium &M, V3 o, V3 d, Rng &r, V3 &x, int64_t &steps)
{
    float t0, t1;
    if (!clip(M, o, d, t0, t1) || !(M.maj > 0.f))
        return false;
    float t = t0;
    const float inv = M.inv_ff;
    const int64_t s0 = steps;
    while (steps < kMaxSteps) {
        ++steps;
        t += exp_flight(r.u()) * inv;
        if (t >= t1)
            return false;
        const V3 p = madd(o, t, d);
        if (r.u() * M.maj < mu_at(M, p)) {
            x = p;
            return true;
        }
    }
    note_cap(M, s0, steps);
    return false;
}

// Ratio-tracking estimate of the transmittance from o along unit d to the box exit.
__device__ float ratio_track(const Medium &M, V3 o, V3 d, Rng &r, int64_t &steps)
{
    float t0, t1;
    if (!clip(M, o, d, t0, t1) || !(M.maj > 0.f))
        return 1.f;
    float T = 1.f, t = t0;
    const float inv = 1.f / M.maj;
    const int64_t s0 = steps;
    while (steps < kMaxSteps) {
        ++steps;
        t += exp_flight(r.u()) * M.inv_ff;
        if (t >= t1)
            return T;
        T *= 1.f - mu_at(M, madd(o, t, d)) * inv;
    }
    note_cap(M, s0, steps);
    return T;
}

__device__ __forceinline__ float hg(float g, float mu)
{
    const float den = 1.f + g * g - 2.f * g * mu;
    return (1.f - g * g) / (4.f * (float)M_PI * den * sqrtf(den));
}

// Inverse-CDF sample of the Henyey-Greenstein cosine (isotropic for |g| < 1e-3).
__device__ __forceinline__ float hg_cos(float g, float u)
{
    if (fabsf(g) < 1e-3f)
        return 2.f * u - 1.f;
    const float s = (1.f - g * g) / (1.f - g + 2.f * g * u);
    return fminf(1.f, fmaxf(-1.f, (1.f + g * g - s * s) / (2.f * g)));
}

// Tabulated phase function p at theta_i = i pi / (n - 1): linear in theta between nodes.
__device__ __forceinline__ float tab_eval(const float *p, int n, float mu)
{
    const float th = acosf(fminf(1.f, fmaxf(-1.f, mu))) * ((float)(n - 1) / (float)M_PI);
    const int i = min((int)th, n - 2);
    const float f = th - (float)i;
    return fmaf(f, p[i + 1] - p[i], p[i]);
}

// cos(theta) from the table: the node interval by binary search of the CDF, then theta
// inside it from the density linear between the nodes' p sin(theta) (the root of the
// interval's quadratic CDF, in the form without cancellation).
__device__ __forceinline__ float tab_sample(const float *p, const float *cdf, int n, float u)
{
    int lo = 0, hi = n - 1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cdf[mid] <= u)
            lo = mid;
        else
            hi = mid;
    }
    const float dth = (float)M_PI / (float)(n - 1);
    const float fa = p[lo] * sinf((float)lo * dth), fb = p[lo + 1] * sinf((float)(lo + 1) * dth);
    const float den = cdf[lo + 1] - cdf[lo];
    const float q = den > 0.f ? (u - cdf[lo]) / den : 0.f;
    const float sq = sqrtf(fmaxf(0.f, fa * fa + (fb - fa) * q * (fa + fb)));
    const float t = fa + sq > 0.f ? fminf(1.f, fmaxf(0.f, q * (fa + fb) / (fa + sq))) : q;
    return cosf(((float)lo + t) * dth);
}

// Phase function of the medium: the table when one is set (first: the first-collision
// table of camera rays, else the scattering table), else Henyey-Greenstein.  TAB (any
// table set) is a compile-time choice, so the kernels without tables keep the registers
// (and the occupancy) of the plain Henyey-Greenstein code.
template <bool TAB>
__device__ __forceinline__ float phase_eval(const TracerParams &tp, bool first, float mu)
{
    if constexpr (TAB) {
        if (first && tp.pf_n)
            return tp.pf_scale * tab_eval(tp.pf_p, tp.pf_n, mu);
        if (tp.ph_n)
            return tab_eval(tp.ph_p, tp.ph_n, mu);
    }
    return hg(tp.g, mu);
}

template <bool TAB> __device__ __forceinline__ float phase_sample(const TracerParams &tp, float u)
{
    if constexpr (TAB) {
        if (tp.ph_n)
            return tab_sample(tp.ph_p, tp.ph_cdf, tp.ph_n, u);
    }
    return hg_cos(tp.g, u);
}

__device__ V3 around(V3 w, float c, float u)
{
    V3 t1, t2;
    basis(w, t1, t2);
    const float s = sqrtf(fmaxf(0.f, 1.f - c * c));
    float sp, cp;
    sincosf(2.f * (float)M_PI * u, &sp, &cp);
    V3 o = v3(s * cp * t1.x + s * sp * t2.x + c * w.x, s * cp * t1.y + s * sp * t2.y + c * w.y,
              s * cp * t1.z + s * sp * t2.z + c * w.z);
    const float l = sqrtf(dot(o, o));
    return v3(o.x / l, o.y / l, o.z / l);
}

// ------------------------------------------------------------------ team walker
// One path is walked by a team of TEAM consecutive lanes.  A path's uniforms come from one
// counter-based stream, and a flight's length does not depend on the extinction found at
// its end, so a team draws a whole window of 4 TEAM words at once (one Philox block per
// lane), sums the flights in stream order along its lanes, looks the extinction up at all
// the window's tentative collisions together, and only then decides which collision
// ends the flight (delta tracking) or multiplies the transmittance factors up in order
// (ratio tracking).  Every value and its order are those of one thread walking the stream
// word by word, so estimates are bit for bit the serial walk's.
//
// What bounds it: paths at albedo 0.999 take from tens to 2.7e5 tentative collisions, 97 %
// of them in ratio tracking toward the light.  With one thread per path (nested loops) 6
// of 64 lanes were active in a step and the longest path was one chain of memory
// latencies; here a wave walks 64 / TEAM paths, each in its own phase of one flat loop,
// takes the next path as soon as one ends, and reads no extinction where the transmittance
// is already 0 or the brick is empty (LDS bits).  Measured on a 256^3 cloud of mean optical
// depth 130 per unit, albedo 0.999: 2048 records x 256 paths 204 -> 34 ms (one thread per
// path -> teams of 8), a 128^2 view x 64 samples 138 -> 27 ms; record draws (2048) 8.6 ->
// 0.45 ms.  The vector ALUs issue in 80 % of the cycles.  Teams of 4 take 48 ms (more
// windows per path), teams of 16 39 ms (more idle words at a phase's end); below 2^14 paths
// teams of 16 win, since there a launch lasts as long as its longest path.
struct PathArgs {
    const float *a, *b, *light;  // records: position, view, light; rays: origin, direction
    V3 wl;                       // the light of camera rays
    const int32_t *list;         // active items' records (relative to rec0), NULL: all
    const int32_t *n_list;       // device count of the list
    uint32_t *head;              // heads of the queues of items; NULL: waves take fixed shares
    int64_t rec0;                // first record of the list (or of this launch)
    uint32_t slot0, n;           // first item of this launch, its items (at most)
    int spp, s0, grab;
    uint32_t queues;
    uint64_t seed, sample;
    double *val;                 // one value per path
    float *pos, *view, *light_out, *direct;
    uint8_t *hit;
    int32_t *tries;
};

// Value of the lane before (after) this one in its row of 16; lanes without one get `edge`.
__device__ __forceinline__ float lane_before(float v, float edge)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v),
                                           0x111, 0xf, 0xf, false));
}
__device__ __forceinline__ uint32_t lane_after(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x101, 0xf, 0xf, false);
}

template <int TEAM> __device__ __forceinline__ int team_min(int v)
{
    static_assert(TEAM == 4 || TEAM == 8 || TEAM == 16, "teams lie inside a row of 16 lanes");
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true));
    if constexpr (TEAM >= 8)
        v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true));
    if constexpr (TEAM >= 16)
        v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true));
    return v;
}

// The items of a launch lie in A.queues queues; a wave takes from its block's until that is empty,
// then from the others.  With one counter for all, the 4096 waves of a full launch waited for one
// another's atomics: 64000 paths of a few collisions 222 us, with 32 queues 83 us; 320000 paths
// 312 and 143 us.  Small launches keep one queue to 16 blocks, as a wave looks at every queue
// before it ends.
constexpr uint32_t kQueues = 32, kQueueStride = 32;

constexpr int kWalkThreads = 256;
constexpr int kOccWords = 2048;  // brick bits in LDS: at most 65536 bricks

enum Phase { kNew, kStart, kBounce, kHit, kAimDelta, kAimRatio, kDelta, kRatio, kDone };

// Blocks per compute unit, 128 registers to a lane.  Two samples of 518400 camera rays with
// prediction: 5.69 ms so, 5.85 ms with 5 blocks for first hits, 6.33 with 6, 5.83 with 3.
constexpr int kWalkBlocks = 4;

template <int KIND, bool TAB, bool SET, bool DIRECT, int TEAM>
__global__ void __launch_bounds__(kWalkThreads, kWalkBlocks) k_paths(Medium M, TracerParams tp, PathArgs A)
{
    constexpr int W = 4 * TEAM;  // words of a window
    constexpr int kSteps = (int)kMaxSteps;
    const uint32_t items = A.list ? (uint32_t)max(0, min((int)A.n, *A.n_list - (int)A.slot0)) : A.n;
    const uint32_t total = items * (uint32_t)A.spp;
    if (total == 0)
        return;
    __shared__ uint32_t occ[kOccWords];
    for (int e = threadIdx.x; e < M.occ_words; e += kWalkThreads)
        occ[e] = M.occ[e];
    const bool wild = M.occ[M.occ_words] != 0;  // a zero transmittance does not stay zero
    __syncthreads();

    const int lane = threadIdx.x & 63, i = lane & (TEAM - 1), lead = lane & ~(TEAM - 1);
    const uint32_t waves = gridDim.x * (kWalkThreads / 64);
    // the wave's items: q0 .. q1 - 1; the queue it takes from (kQueues: all are empty)
    constexpr bool kQueued = KIND == kRecordPaths || KIND == kPixelPaths;
    uint32_t share = (blockIdx.x * (kWalkThreads / 64) + (threadIdx.x >> 6)) * (uint32_t)A.grab;
    uint32_t q0 = 0, q1 = 0, queue = kQueued ? blockIdx.x % A.queues : 0;

    int phase = kNew, j = 0, steps = 0;
    WordPos<KIND> q = 0;
    uint32_t id0 = 0, id1 = 0, item = 0;
    int64_t rec = 0;
    V3 p = v3(0, 0, 0), d = p, wprev = p, wh = p, wl = p;
    float t = 0.f, t1 = 0.f, T = 1.f, wgt = 0.f, sum = 0.f, direct = 0.f;
    bool uncollided = false;
    int tries = 0;

    // the end of a path: its value (or outputs), then the next item
    auto finish = [&](double e) {
        if (i == 0)
            A.val[item] = e;
        phase = kNew;
    };
    auto estimate = [&]() {  // direct: the direct term's weight x transmittance
        if constexpr (KIND == kPixelPaths)
            finish((double)tp.albedo * (double)fmaf(direct, tp.irradiance, sum));
        else
            finish((double)(DIRECT ? fmaf(direct, tp.irradiance, sum) : sum));
    };
    auto first_hit = [&](bool h, float dir) {
        if (i == 0) {
            A.pos[3 * rec] = h ? p.x : 0.f;
            A.pos[3 * rec + 1] = h ? p.y : 0.f;
            A.pos[3 * rec + 2] = h ? p.z : 0.f;
            A.view[3 * rec] = h ? wprev.x : 0.f;
            A.view[3 * rec + 1] = h ? wprev.y : 0.f;
            A.view[3 * rec + 2] = h ? wprev.z : 0.f;
            A.direct[rec] = dir;
            A.hit[rec] = h ? 1 : 0;
        }
        phase = kNew;
    };
    auto escaped = [&]() {  // no collision along d
        if constexpr (KIND == kRecordDraws) {
            phase = tries < 1000000 ? kStart : kHit;
            if (phase == kHit)
                p = v3(NAN, NAN, NAN);
        } else if constexpr (KIND == kFirstHits) {
            first_hit(false, 0.f);
        } else {
            if (KIND == kPixelPaths && j == 0) {
                finish(tp.light_mode == 1 ? (double)tp.irradiance : 0.0);
            } else {
                if (tp.light_mode == 1 && (j > 1 || uncollided))
                    sum += tp.irradiance;
                estimate();
            }
        }
    };
    auto lit = [&](float Tr) {  // a ratio estimate toward the light is complete
        if constexpr (KIND == kFirstHits) {
            first_hit(true, wgt * Tr * tp.irradiance);
        } else if (j == 0) {
            direct = wgt * Tr;
            steps = 0;
            phase = kBounce;
        } else {
            sum = fmaf(wgt * Tr, tp.irradiance, sum);
            wprev = wh;
            phase = kBounce;
        }
    };
    auto start_ratio = [&](V3 l) {
        d = l;
        phase = kAimRatio;
    };

#pragma unroll 1
    for (;;) {
        // ---- idle teams take the wave's next items
        const uint64_t idle = __ballot(phase == kNew && i == 0);
        if (idle) {
            const uint32_t n = (uint32_t)__popcll(idle), have = q1 - q0;
            const uint32_t rank = (uint32_t)__popcll(idle & ((1ull << lead) - 1));
            uint32_t next = q0 + rank;
            bool got = rank < have;
            if (n > have) {
                const uint32_t take = max((uint32_t)A.grab, n - have);
                uint32_t base = 0, avail = 0;
                if constexpr (kQueued) {
                    // items of a queue, formed anew here: kept over the walk, it costs registers
                    uint32_t queues = A.queues;
                    asm volatile("" : "+s"(queues));
                    const uint32_t per = (total + queues - 1) / queues;
                    auto items_of = [&](uint32_t k) {
                        return k * per < total ? min(per, total - k * per) : 0;
                    };
                    while (queue < kQueues && avail == 0) {
                        if (lane == 0)
                            base = atomicAdd(A.head + queue * kQueueStride, take);
                        base = __builtin_amdgcn_readfirstlane(base);
                        const uint32_t len = items_of(queue);
                        avail = base < len ? min(take, len - base) : 0;
                        base += queue * per;
                        if (avail == 0) {  // on to the next queue that is not empty
                            const uint32_t l = min((uint32_t)lane, queues - 1);
                            const uint64_t open = __ballot(
                                __hip_atomic_load(A.head + l * kQueueStride, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT) < items_of(l));
                            const uint64_t after = open & (~0ull << queue);
                            queue = open ? __builtin_ctzll(after ? after : open) % queues : kQueues;
                        }
                    }
                    if (rank >= have && rank - have < avail) {
                        next = base + (rank - have);
                        got = true;
                    }
                } else {
                    base = share;
                    avail = take;
                    share += waves * (uint32_t)A.grab;
                    if (rank >= have)
                        next = base + (rank - have);
                }
                q0 = base + min(n - have, avail);
                q1 = base + avail;
            } else {
                q0 += n;
            }
            if constexpr (!kQueued)
                got = next < total;
            if (phase == kNew) {
                if (!got) {
                    if (!kQueued || queue >= kQueues)
                        phase = kDone;
                } else {
                    item = next;
                    const uint32_t slot = item / (uint32_t)A.spp, s = item - slot * (uint32_t)A.spp;
                    rec = A.rec0 + (A.list ? (int64_t)A.list[A.slot0 + slot] : (int64_t)slot);
                    uint64_t id;
                    if constexpr (KIND == kRecordDraws)
                        id = (uint64_t)rec;
                    else if constexpr (KIND == kFirstHits)
                        id = ((uint64_t)rec << 20) + A.sample;
                    else
                        id = ((uint64_t)rec << 20) + (uint64_t)(A.s0 + (int)s);
                    id0 = (uint32_t)id;
                    id1 = (uint32_t)(id >> 32);
                    q = 0;
                    j = 0;
                    steps = 0;
                    sum = 0.f;
                    direct = 0.f;
                    tries = 0;
                    if constexpr (KIND == kRecordDraws) {
                        phase = kStart;
                    } else {
                        p = v3(A.a[3 * rec], A.a[3 * rec + 1], A.a[3 * rec + 2]);
                        if constexpr (KIND == kRecordPaths) {
                            unit(A.b + 3 * rec, wprev);  // the list holds usable directions
                            unit(A.light + 3 * rec, wl);
                            uncollided = DIRECT && tp.light_mode == 1;
                            phase = kBounce;
                            if (DIRECT && tp.light_mode != 1) {
                                wgt = phase_eval<TAB>(tp, false, -dot_direct(wprev, wl));
                                start_ratio(wl);
                            }
                        } else {
                            wl = A.wl;
                            if (unit(A.b + 3 * rec, d)) {
                                wprev = neg(d);
                                uncollided = true;
                                phase = kAimDelta;
                            } else {
                                escaped();  // first hits only: an unusable ray
                            }
                        }
                    }
                }
            }
        }
        if (!__any(phase != kDone))
            break;

        // ---- the window: words [q & ~3, q & ~3 + W) of the team's stream, four per lane
        uint32_t b[4];
        stream_block(A.seed, id0, id1, (q >> 2) + (uint32_t)i, b);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            b[c] >>= 8;
        const WordPos<KIND> qa = q & ~(WordPos<KIND>)3;
        int x = (int)(q & 3u);  // cursor: first unread word of the window
        auto word = [&]() {     // a team-uniform read of the next word
            const int w = x++;
            const uint32_t lo = (w & 1) ? b[1] : b[0], hi = (w & 1) ? b[3] : b[2];
            return (uint32_t)__shfl((int)((w & 2) ? hi : lo), lead + (w >> 2), 64);
        };

        if constexpr (KIND == kRecordDraws) {
            if (phase == kHit) {  // the record's light direction; write it out
                const float u0 = unit24(word()), u1 = unit24(word());
                const float zc = 1.f - 2.f * u0, rr = sqrtf(fmaxf(0.f, 1.f - zc * zc));
                float sp, cp;
                sincosf(2.f * (float)M_PI * u1, &sp, &cp);
                if (i == 0) {
                    A.pos[3 * rec] = p.x;
                    A.pos[3 * rec + 1] = p.y;
                    A.pos[3 * rec + 2] = p.z;
                    A.view[3 * rec] = -d.x;
                    A.view[3 * rec + 1] = -d.y;
                    A.view[3 * rec + 2] = -d.z;
                    A.light_out[3 * rec] = rr * cp;
                    A.light_out[3 * rec + 1] = rr * sp;
                    A.light_out[3 * rec + 2] = zc;
                    if (A.tries)
                        A.tries[rec] = tries;
                }
                phase = kNew;
            }
        }
        if constexpr (KIND == kRecordDraws) {
            if (phase == kStart) {  // direction uniform on the sphere, origin on the disc
                const V3 c = v3(0.5f * (M.amin.x + M.amax.x), 0.5f * (M.amin.y + M.amax.y),
                                0.5f * (M.amin.z + M.amax.z));
                const V3 e = v3(0.5f * (M.amax.x - M.amin.x), 0.5f * (M.amax.y - M.amin.y),
                                0.5f * (M.amax.z - M.amin.z));
                const float R = sqrtf(dot(e, e));
                ++tries;
                const float u0 = unit24(word()), u1 = unit24(word());
                const float zc = 1.f - 2.f * u0, rr = sqrtf(fmaxf(0.f, 1.f - zc * zc));
                float sp, cp;
                sincosf(2.f * (float)M_PI * u1, &sp, &cp);
                d = v3(rr * cp, rr * sp, zc);
                V3 e1, e2;
                basis(d, e1, e2);
                const float rad = R * sqrtf(unit24(word()));
                sincosf(2.f * (float)M_PI * unit24(word()), &sp, &cp);
                p = v3(c.x - R * d.x + rad * (cp * e1.x + sp * e2.x),
                       c.y - R * d.y + rad * (cp * e1.y + sp * e2.y),
                       c.z - R * d.z + rad * (cp * e1.z + sp * e2.z));
                steps = 0;
                phase = kAimDelta;
            }
        } else {
            // ---- a collision: absorption, then next-event estimation
            if (phase == kHit) {
                if (j == 0) {  // camera ray: direct light at the first collision
                    if constexpr (KIND == kFirstHits) {
                        wgt = tp.albedo * phase_eval<TAB>(tp, true, -dot_direct(wprev, wl));
                        start_ratio(wl);
                    } else if constexpr (SET) {
                        const float4 lw = tp.set_dw[set_pick(tp, word())];
                        const V3 lj = v3(lw.x, lw.y, lw.z);
                        wgt = lw.w * phase_eval<TAB>(tp, true, -dot_direct(wprev, lj));
                        uncollided = false;
                        start_ratio(lj);
                    } else if (tp.light_mode == 0) {
                        wgt = phase_eval<TAB>(tp, true, -dot_direct(wprev, wl));
                        uncollided = false;
                        start_ratio(wl);
                    } else {
                        steps = 0;
                        phase = kBounce;
                    }
                } else if (unit24(word()) >= tp.albedo) {
                    estimate();
                } else if constexpr (SET) {
                    const float4 lw = tp.set_dw[set_pick(tp, word())];
                    const V3 lj = v3(lw.x, lw.y, lw.z);
                    wgt = lw.w * phase_eval<TAB>(tp, false, -dot(wh, lj));
                    start_ratio(lj);
                } else if (tp.light_mode == 0) {
                    wgt = phase_eval<TAB>(tp, false, -dot(wh, wl));
                    start_ratio(wl);
                } else {
                    wprev = wh;
                    phase = kBounce;
                }
            }
            // ---- the next flight's direction, for three teams or more at a time (its 300
            // instructions run for the whole wave), or when no team has steps to take
            const int waiting = __popcll(__ballot(phase == kBounce));
            const bool go = waiting >= 3 * TEAM ||
                            !__any(phase >= kAimDelta && phase <= kRatio);
            if (go && phase == kBounce) {
                ++j;
                if ((tp.max_interactions > 0 && j > tp.max_interactions) || steps >= kSteps) {
                    estimate();
                } else {
                    const float c = phase_sample<TAB>(tp, unit24(word()));
                    wh = around(wprev, c, unit24(word()));
                    d = neg(wh);
                    phase = kAimDelta;
                }
            }
        }

        // ---- the segment of the new direction inside the box
        if (phase == kAimDelta || phase == kAimRatio) {
            const bool r = phase == kAimRatio;
            float a0, a1;
            const bool in = clip(M, p, d, a0, a1) && M.maj > 0.f && !(r && steps >= kSteps);
            t = a0;
            t1 = a1;
            T = 1.f;
            if (in)
                phase = r ? kRatio : kDelta;
            else if (r)
                lit(1.f);
            else
                escaped();
        }

        // ---- the window's tentative collisions
        const bool ratio = phase == kRatio, delta = phase == kDelta;
        if (!ratio && !delta)
            q = qa + (uint32_t)x;
        if (!__any(ratio || delta))
            continue;
        const int left = kSteps - steps;
        // a bounce's free flight rarely takes more than a few steps, a camera ray's does
        const int wd = KIND == kFirstHits || KIND == kRecordDraws || j == 0 ? W : min(W, 16);
        const int lim = ratio ? min(W, x + left) : min(wd, x + 2 * min(left, W));
        const int odd = ratio ? 0 : 1;
        float tj[4], ej[4], wj[4];
        bool fl[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int w = 4 * i + c;
            // ratio: every word is a flight; delta: a flight, then the collision's uniform
            fl[c] = (w >= x) & (w + odd < lim) & (((w - x) & odd) == 0) & (ratio | delta);
            ej[c] = exp_flight(unit24(b[c]));
            wj[c] = fl[c] ? M.inv_ff : 0.f;
        }
        // flight ends in stream order: lane after lane, four words each
        float tin = t;
#pragma unroll
        for (int st = 0; st < TEAM; ++st) {
            tj[0] = fmaf(ej[0], wj[0], tin);
            tj[1] = fmaf(ej[1], wj[1], tj[0]);
            tj[2] = fmaf(ej[2], wj[2], tj[1]);
            tj[3] = fmaf(ej[3], wj[3], tj[2]);
            if (st < TEAM - 1) {
                tin = lane_before(tj[3], t);
                tin = i == 0 ? t : tin;
            }
        }
        // extinction where it can matter: inside the box, in an occupied brick, and for a
        // transmittance only while it is not zero (all other slots read cell 0, which stays in
        // the cache, and count as empty)
        const bool live = delta | (ratio & ((T != 0.f) | wild));
        float mu[4] = {0.f, 0.f, 0.f, 0.f};
        bool out[4], need[4], any = false;
        float fx[4], fy[4], fz[4];
        uint64_t cell[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            out[c] = fl[c] & (tj[c] >= t1);
            const V3 y = madd(p, tj[c], d);
            const float ux = __builtin_amdgcn_fmed3f((y.x - M.amin.x) * M.inv_h + 0.5f, 0.f, M.hx);
            const float uy = __builtin_amdgcn_fmed3f((y.y - M.amin.y) * M.inv_h + 0.5f, 0.f, M.hy);
            const float uz = __builtin_amdgcn_fmed3f((y.z - M.amin.z) * M.inv_h + 0.5f, 0.f, M.hz);
            const uint32_t ci = (uint32_t)ux, cj = (uint32_t)uy, ck = (uint32_t)uz;
            fx[c] = __builtin_amdgcn_fractf(ux);
            fy[c] = __builtin_amdgcn_fractf(uy);
            fz[c] = __builtin_amdgcn_fractf(uz);
            const uint32_t br =
                (ci >> M.occ_s) +
                __umul24((uint32_t)M.bx, (cj >> M.occ_s) + __umul24((uint32_t)M.by, ck >> M.occ_s));
            need[c] = live & fl[c] & !out[c] & (((occ[br >> 5] >> (br & 31)) & 1u) != 0);
            const uint64_t at = (uint64_t)(uint32_t)M.cx * (cj + (uint32_t)M.cy * ck) + ci;
            cell[c] = need[c] ? at : 0;
            any = any | need[c];
        }
        if (__any(any)) {
            float4 lo[4], hi[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                lo[c] = M.cells[2 * cell[c]];
                hi[c] = M.cells[2 * cell[c] + 1];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
                mu[c] = need[c] ? mu_lerp(lo[c], hi[c], fx[c], fy[c], fz[c]) : 0.f;
        }
        // the first word whose flight ends the walk (none: W)
        const uint32_t b4 = lane_after(b[0]);
        int first = W;
#pragma unroll
        for (int c = 3; c >= 0; --c) {
            const bool acc =
                delta & need[c] & (unit24(c < 3 ? b[c < 3 ? c + 1 : 0] : b4) * M.maj < mu[c]);
            first = (out[c] | acc) ? 4 * i + c : first;
        }
        first = team_min<TEAM>(first);
        // transmittance factors in stream order (slots without a lookup multiply by 1)
        if (__any(ratio && live)) {
            const float inv = 1.f / M.maj;
            float f[4], Tin = T, To;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                f[c] = 1.f - mu[c] * inv;
#pragma unroll
            for (int st = 0; st < TEAM; ++st) {
                To = Tin * f[0];
                To *= f[1];
                To *= f[2];
                To *= f[3];
                if (st < TEAM - 1) {
                    Tin = lane_before(To, T);
                    Tin = i == 0 ? T : Tin;
                }
            }
            To = __shfl(To, lead + TEAM - 1, 64);
            T = ratio ? To : T;
        }
        const bool ends = first < W;
        const int at = ends ? first : W - 1;
        const float lo_t = (at & 1) ? tj[1] : tj[0], hi_t = (at & 1) ? tj[3] : tj[2];
        const float te = __shfl((at & 2) ? hi_t : lo_t, lead + (at >> 2), 64);
        if (ratio) {
            const int n = ends ? first - x + 1 : lim - x;
            steps += n;
            q = qa + (uint32_t)(x + n);
            t = te;
            if (ends) {
                lit(T);
            } else if (steps >= kSteps) {
                note_cap(M, i == 0 ? 0 : kMaxSteps, steps);
                lit(T);
            }
        } else if (delta) {
            const int n = ends ? ((first - x) >> 1) + 1 : (lim - x) >> 1;
            steps += n;
            const bool esc = te >= t1;
            q = qa + (uint32_t)(x + 2 * n) - (ends && esc ? 1u : 0u);
            t = te;
            if (ends && !esc) {
                p = madd(p, te, d);
                phase = kHit;
            } else if (ends) {
                escaped();
            } else if (steps >= kSteps) {
                note_cap(M, i == 0 ? 0 : kMaxSteps, steps);
                escaped();
            }
        }
    }
}

// Launch geometry of the per-record sums: a wave holds kPaths / seg records, each owning
// seg consecutive lanes (seg a power of two); records with more than kPaths paths have
// nblk partial sums (then seg = kPaths), which k_finish_sums adds in order.
struct Split {
    int seg, nblk;
};

// ------------------------------------------------------------------ one path per thread
// For short paths (serial_paths, serial_first_hits, serial_draws say which): no windows drawn for a
// flight or two, no list, no stored path values, one launch and the sums' instead of four.  The
// same words in the same order, so bitwise the walker's estimates.  320000 paths in a cloud of
// two mean free paths: 62 us (teams 178), 1024^2 camera rays on a 64^3 cloud of 60: 147 us (329).
// One path estimate of the indirect in-scattered radiance at x toward w
// (directional light: next-event estimation at every collision; uniform
// environment: the radiance of escaping paths after at least one collision, or
// any escape when count_uncollided).
template <bool TAB, bool SET>
__device__ float li_path(const Medium &M, const TracerParams &tp, V3 x, V3 w, V3 wl,
                         bool count_uncollided, Rng &r)
{
    V3 wprev = w, p = x;
    float sum = 0.f;
    int64_t steps = 0;
    for (int j = 1;; ++j) {
        if ((tp.max_interactions > 0 && j > tp.max_interactions) || steps >= kMaxSteps)
            break;
        const float c = phase_sample<TAB>(tp, r.u());
        const V3 wh = around(wprev, c, r.u());
        V3 xn;
        if (!delta_track(M, p, neg(wh), r, xn, steps)) {
            if (tp.light_mode == 1 && (j > 1 || count_uncollided))
                sum += tp.irradiance;
            break;
        }
        p = xn;
        if (r.u() >= tp.albedo)
            break;
        if constexpr (SET) {
            const float4 lw = tp.set_dw[set_pick(tp, r.bits24())];
            const V3 lj = v3(lw.x, lw.y, lw.z);
            sum = fmaf(lw.w * phase_eval<TAB>(tp, false, -dot(wh, lj)) *
                           ratio_track(M, p, lj, r, steps),
                       tp.irradiance, sum);
        } else if (tp.light_mode == 0) {
            sum = fmaf(phase_eval<TAB>(tp, false, -dot(wh, wl)) * ratio_track(M, p, wl, r, steps),
                       tp.irradiance, sum);
        }
        wprev = wh;
    }
    return sum;
}

// Deterministic segmented reduction of (sum, sum of squares) in FP64: thread
// t of each segment ends holding nothing; the segment leader writes the totals.
__device__ void segment_sums(double s1, double s2, int seg, bool write, double *out)
{
    __shared__ double a[kPaths], b[kPaths];
    const int t = threadIdx.x;
    a[t] = s1;
    b[t] = s2;
    __syncthreads();
    for (int w = seg >> 1; w > 0; w >>= 1) {
        if ((t & (seg - 1)) < w) {
            a[t] += a[t + w];
            b[t] += b[t + w];
        }
        __syncthreads();
    }
    if (write && (t & (seg - 1)) == 0) {
        out[0] = a[t];
        out[1] = b[t];
    }
}

// One record estimate: L_i, or with tp.include_direct all in-scattered radiance L_s =
// L_d + L_i (directional light: the direct term by ratio tracking, drawn before the path;
// uniform environment: uncollided light counted too).
template <bool TAB, bool DIRECT>
__device__ float record_path(const Medium &M, const TracerParams &tp, V3 x, V3 w, V3 wl, Rng &r)
{
    if constexpr (!DIRECT) {
        return li_path<TAB, false>(M, tp, x, w, wl, false, r);
    } else {
        if (tp.light_mode == 1)
            return li_path<TAB, false>(M, tp, x, w, wl, true, r);
        int64_t steps = 0;
        const float d =
            phase_eval<TAB>(tp, false, -dot_direct(w, wl)) * ratio_track(M, x, wl, r, steps);
        return fmaf(d, tp.irradiance, li_path<TAB, false>(M, tp, x, w, wl, false, r));
    }
}

// Paths s0 .. s0 + spp - 1 of every record (path s on stream id rec * 2^20 + s).
template <bool TAB, bool DIRECT>
__global__ void __launch_bounds__(kPaths) k_trace_li(Medium M, TracerParams tp, const float *pos,
                                                     const float *view, const float *light,
                                                     int64_t P, int s0, int spp, Split sp,
                                                     uint64_t seed, const uint8_t *mask,
                                                     uint8_t mask_bits, double *partial)
{
    const int64_t group = blockIdx.x / sp.nblk;
    const int blk = blockIdx.x % sp.nblk;
    const int64_t rec = group * (kPaths / sp.seg) + threadIdx.x / sp.seg;
    const int s = blk * sp.seg + (threadIdx.x & (sp.seg - 1));
    double e = 0.0;
    V3 w, wl;
    const bool wanted = rec < P && (!mask || (mask[rec] & mask_bits) == mask_bits);
    if (wanted && s < spp && unit(view + 3 * rec, w) && unit(light + 3 * rec, wl)) {
        const V3 x = v3(pos[3 * rec], pos[3 * rec + 1], pos[3 * rec + 2]);
        Rng r;
        r.init(seed, ((uint64_t)rec << 20) + (uint64_t)(s0 + s));
        e = (double)record_path<TAB, DIRECT>(M, tp, x, w, wl, r);
    }
    segment_sums(e, e * e, sp.seg, rec < P, partial + 2 * ((size_t)rec * sp.nblk + blk));
}

// Record configurations (Sec. 5.1): direction d uniform on the sphere, origin
// uniform over the bounding sphere's cross-section orthogonal to d, a free flight
// along d into the cloud, retried on escape; view = -d, light uniform.
__global__ void __launch_bounds__(256) k_sample_records(Medium M, int64_t N, uint64_t seed,
                                                        float *pos, float *view, float *light,
                                                        int32_t *attempts)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    const V3 c = v3(0.5f * (M.amin.x + M.amax.x), 0.5f * (M.amin.y + M.amax.y),
                    0.5f * (M.amin.z + M.amax.z));
    const V3 e = v3(0.5f * (M.amax.x - M.amin.x), 0.5f * (M.amax.y - M.amin.y),
                    0.5f * (M.amax.z - M.amin.z));
    const float R = sqrtf(dot(e, e));
    Rng r;
    r.init(seed, (uint64_t)i);
    V3 d = v3(0, 0, 1), x = v3(NAN, NAN, NAN);
    int tries = 0;
    int64_t steps = 0;
    while (tries < 1000000) {
        ++tries;
        const float u0 = r.u(), u1 = r.u();
        const float zc = 1.f - 2.f * u0, rr = sqrtf(fmaxf(0.f, 1.f - zc * zc));
        float sp, cp;
        sincosf(2.f * (float)M_PI * u1, &sp, &cp);
        d = v3(rr * cp, rr * sp, zc);
        V3 t1, t2;
        basis(d, t1, t2);
        const float rad = R * sqrtf(r.u());
        sincosf(2.f * (float)M_PI * r.u(), &sp, &cp);
        const V3 o = v3(c.x - R * d.x + rad * (cp * t1.x + sp * t2.x),
                        c.y - R * d.y + rad * (cp * t1.y + sp * t2.y),
                        c.z - R * d.z + rad * (cp * t1.z + sp * t2.z));
        steps = 0;
        if (delta_track(M, o, d, r, x, steps))
            break;
        x = v3(NAN, NAN, NAN);
    }
    const float u0 = r.u(), u1 = r.u();
    const float zc = 1.f - 2.f * u0, rr = sqrtf(fmaxf(0.f, 1.f - zc * zc));
    float sp, cp;
    sincosf(2.f * (float)M_PI * u1, &sp, &cp);
    pos[3 * i] = x.x;
    pos[3 * i + 1] = x.y;
    pos[3 * i + 2] = x.z;
    view[3 * i] = -d.x;
    view[3 * i + 1] = -d.y;
    view[3 * i + 2] = -d.z;
    light[3 * i] = rr * cp;
    light[3 * i + 1] = rr * sp;
    light[3 * i + 2] = zc;
    if (attempts)
        attempts[i] = tries;
}

// Path-traced pixels: first collision along each camera ray, then albedo times the
// in-scattered radiance there (direct by next-event estimation plus the indirect
// path estimate for a directional light; all in-scattered environment light in mode 1).
template <bool TAB, bool SET>
__global__ void __launch_bounds__(kPaths) k_render_mc(Medium M, TracerParams tp, V3 wl,
                                                      const float *ray_o, const float *ray_d,
                                                      int64_t N, int spp, Split sp, uint64_t seed,
                                                      double *partial)
{
    const int64_t group = blockIdx.x / sp.nblk;
    const int blk = blockIdx.x % sp.nblk;
    const int64_t px = group * (kPaths / sp.seg) + threadIdx.x / sp.seg;
    const int s = blk * sp.seg + (threadIdx.x & (sp.seg - 1));
    double e = 0.0;
    V3 d;
    if (px < N && s < spp && unit(ray_d + 3 * px, d)) {
        const V3 o = v3(ray_o[3 * px], ray_o[3 * px + 1], ray_o[3 * px + 2]);
        Rng r;
        r.init(seed, ((uint64_t)px << 20) + (uint64_t)s);
        V3 x;
        int64_t steps = 0;
        if (!delta_track(M, o, d, r, x, steps)) {
            e = tp.light_mode == 1 ? tp.irradiance : 0.0;
        } else {
            const V3 w = neg(d);
            if constexpr (SET) {
                const float4 lw = tp.set_dw[set_pick(tp, r.bits24())];
                const V3 lj = v3(lw.x, lw.y, lw.z);
                const float direct = lw.w * phase_eval<TAB>(tp, true, -dot_direct(w, lj)) *
                                     ratio_track(M, x, lj, r, steps);
                e = (double)tp.albedo *
                    (double)fmaf(direct, tp.irradiance,
                                 li_path<TAB, true>(M, tp, x, w, wl, false, r));
            } else if (tp.light_mode == 0) {
                const float direct = phase_eval<TAB>(tp, true, -dot_direct(w, wl)) *
                                     ratio_track(M, x, wl, r, steps);
                e = (double)tp.albedo *
                    (double)fmaf(direct, tp.irradiance,
                                 li_path<TAB, false>(M, tp, x, w, wl, false, r));
            } else {
                e = (double)tp.albedo * (double)li_path<TAB, false>(M, tp, x, w, wl, true, r);
            }
        }
    }
    segment_sums(e, e * e, sp.seg, px < N, partial + 2 * ((size_t)px * sp.nblk + blk));
}

// One camera sample per ray for the network renderer: the delta-tracked first
// collision, the view direction there, and the direct single scattering from the
// directional light (next-event estimation, times the albedo).  Rays that escape
// get hit = 0 and zero outputs.
__global__ void __launch_bounds__(256) k_first_hits(Medium M, TracerParams tp, V3 wl,
                                                    const float *ray_o, const float *ray_d,
                                                    int64_t N, uint64_t seed, uint64_t sample,
                                                    float *pos, float *view, float *direct,
                                                    uint8_t *hit)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    V3 d;
    bool h = false;
    float dir = 0.f;
    V3 x = v3(0, 0, 0);
    if (unit(ray_d + 3 * i, d)) {
        const V3 o = v3(ray_o[3 * i], ray_o[3 * i + 1], ray_o[3 * i + 2]);
        Rng r;
        r.init(seed, ((uint64_t)i << 20) + sample);
        int64_t steps = 0;
        h = delta_track(M, o, d, r, x, steps);
        if (h)
            dir = tp.albedo * phase_eval<true>(tp, true, dot_direct(d, wl)) * ratio_track(M, x, wl, r, steps) *
                  tp.irradiance;
    }
    pos[3 * i] = x.x;
    pos[3 * i + 1] = x.y;
    pos[3 * i + 2] = x.z;
    view[3 * i] = h ? -d.x : 0.f;
    view[3 * i + 1] = h ? -d.y : 0.f;
    view[3 * i + 2] = h ? -d.z : 0.f;
    direct[i] = dir;
    hit[i] = h ? 1 : 0;
}

// Active records of a launch's range: usable directions and, with a mask, the wanted bits.
// The others get zero sums here.
__global__ void __launch_bounds__(256) k_active(const float *view, const float *light,
                                                const uint8_t *mask, uint8_t mask_bits,
                                                int64_t rec0, int n, int nblk, double *partial,
                                                int32_t *list, int32_t *n_list)
{
    const int r = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    bool on = false;
    if (r < n) {
        const int64_t rec = rec0 + r;
        V3 w;
        on = (!mask || (mask[rec] & mask_bits) == mask_bits) && unit(view + 3 * rec, w) &&
             (!light || unit(light + 3 * rec, w));
        if (!on)
            for (int64_t e = 2 * rec * nblk; e < 2 * (rec + 1) * nblk; ++e)
                partial[e] = 0.0;
    }
    const uint64_t m = __ballot(on);
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == 0 && m)
        base = atomicAdd(n_list, (int)__popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    if (on)
        list[base + (int)__popcll(m & ((1ull << lane) - 1))] = r;
}

// Sum and sum of squares in FP64 of each record's path values, in a fixed tree order, for
// the list's slots slot0 .. slot0 + n - 1; then the queues are empty for the next launch.
__global__ void __launch_bounds__(kPaths) k_path_sums(const double *val, const int32_t *list,
                                                      const int32_t *n_list, uint32_t *head,
                                                      int64_t rec0, int slot0, int n, int spp,
                                                      Split sp, double *partial)
{
    __shared__ double a[kPaths], b[kPaths];
    const int t = threadIdx.x;
    const int per = kPaths / sp.seg;
    const int items = max(0, min(n, *n_list - slot0));
    const int64_t units = ((int64_t)items + per - 1) / per * sp.nblk;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int64_t slot = u / sp.nblk * per + t / sp.seg;
        const int blk = (int)(u % sp.nblk);
        const int s = blk * sp.seg + (t & (sp.seg - 1));
        const bool in = slot < items;
        const double e = in && s < spp ? val[slot * spp + s] : 0.0;
        __syncthreads();
        a[t] = e;
        b[t] = e * e;
        __syncthreads();
        for (int w = sp.seg >> 1; w > 0; w >>= 1) {
            if ((t & (sp.seg - 1)) < w) {
                a[t] += a[t + w];
                b[t] += b[t + w];
            }
            __syncthreads();
        }
        if (in && (t & (sp.seg - 1)) == 0) {
            double *out = partial + 2 * ((rec0 + list[slot0 + slot]) * sp.nblk + blk);
            out[0] = a[t];
            out[1] = b[t];
        }
    }
    if (blockIdx.x == 0 && t < (int)kQueues)
        head[t * kQueueStride] = 0;
}

// Bits of the occupied bricks (see Medium), one wave per brick: brick (i, j, k) holds the
// cells whose corners are the voxels [i 2^s - 1, (i + 1) 2^s - 1] per axis.
// wild: an extinction that is not finite, or so large (below zero) that it or its ratio to the
// majorant overflows on the way from the corners to the factor (bound: a fourth of what FP32
// holds).
__global__ void __launch_bounds__(256) k_occupied(const float *mu, int nx, int ny, int nz, int s,
                                                  int bx, int by, int bz, int words, float maj,
                                                  uint32_t *occ)
{
    constexpr float kTame = 8e37f;
    const int64_t br = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (br >= (int64_t)bx * by * bz)
        return;
    const int lane = threadIdx.x & 63, e = (1 << s) + 1;
    const int x0 = ((int)(br % bx) << s) - 1, y0 = ((int)(br / bx % by) << s) - 1,
              z0 = ((int)(br / bx / by) << s) - 1;
    bool on = false, wild = false;
    for (int v = lane; v < e * e * e; v += 64) {
        const int x = x0 + v % e, y = y0 + v / e % e, z = z0 + v / e / e;
        if (x >= 0 && y >= 0 && z >= 0 && x < nx && y < ny && z < nz) {
            const float m = mu[((int64_t)z * ny + y) * nx + x];
            on = on || m != 0.f;
            wild = wild || !(fabsf(m) <= kTame && fabsf(m) * (1.f / maj) <= kTame);
        }
    }
    if (__any(on) && lane == 0)
        atomicOr(&occ[br >> 5], 1u << (br & 31));
    if (__any(wild) && lane == 0)
        atomicOr(&occ[words], 1u);
}

__global__ void __launch_bounds__(256) k_finish_sums(const double *partial, int64_t P, int nblk,
                                                     int spp, double *mean, double *var)
{
    const int64_t rec = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (rec >= P)
        return;
    double s1 = 0.0, s2 = 0.0;
    for (int b = 0; b < nblk; ++b) {
        s1 += partial[2 * (rec * nblk + b)];
        s2 += partial[2 * (rec * nblk + b) + 1];
    }
    const double m = s1 / spp;
    mean[rec] = m;
    if (var)
        var[rec] = spp > 1 ? fmax(0.0, (s2 - spp * m * m) / (spp - 1)) / spp : 0.0;
}

// Progressive estimates (Sec. 5.1).  k_adapt_init marks the records with usable
// directions active and zeroes their sums; after each batch of paths k_adapt_step adds
// the batch's per-block partial sums (in block order), and a record stops once
// zq * sqrt(variance of the mean) <= rel * |mean| or max_spp paths are reached, writing
// its mean, variance of the mean and path count; records still active are counted.
__global__ void __launch_bounds__(256) k_adapt_init(const float *view, const float *light,
                                                    int64_t P, uint8_t *active, double *sums,
                                                    double *mean, double *var, int32_t *n_out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P)
        return;
    V3 w, wl;
    active[i] = unit(view + 3 * i, w) && unit(light + 3 * i, wl) ? 1 : 0;
    sums[2 * i] = 0.0;
    sums[2 * i + 1] = 0.0;
    mean[i] = 0.0;
    if (var)
        var[i] = 0.0;
    if (n_out)
        n_out[i] = 0;
}

// Batches j = 0 .. kb - 1 of one round, in order: batch j's nb block partials (blocks
// j nb .. j nb + nb - 1 of the round's kb nb) join the record's running sums, and the rule
// is checked after each, so a record stops at the same batch as with one batch per round;
// later batches of a stopped record are discarded.
__global__ void __launch_bounds__(256) k_adapt_step(const double *partial, int nb, int kb,
                                                    int64_t P, int n0, int batch, int max_spp,
                                                    double rel, double zq, uint8_t *active,
                                                    double *sums, double *mean, double *var,
                                                    int32_t *n_out, unsigned long long *left)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P || !active[i])
        return;
    double s1 = sums[2 * i], s2 = sums[2 * i + 1];
    const int64_t nblk = (int64_t)nb * kb;
    for (int j = 0; j < kb; ++j) {
        for (int b = j * nb; b < (j + 1) * nb; ++b) {
            s1 += partial[2 * (i * nblk + b)];
            s2 += partial[2 * (i * nblk + b) + 1];
        }
        const int n = n0 + (j + 1) * batch;
        const double m = s1 / n;
        const double vm = fmax(0.0, (s2 - n * m * m) / (n - 1)) / n;
        if (zq * sqrt(vm) <= rel * fabs(m) || n >= max_spp) {
            active[i] = 0;
            mean[i] = m;
            if (var)
                var[i] = vm;
            if (n_out)
                n_out[i] = n;
            return;
        }
    }
    sums[2 * i] = s1;
    sums[2 * i + 1] = s2;
    atomicAdd(left, 1ull);
}

// Camera samples under a light set: the first collision as a first-hit walk finds it, then `draws`
// members of the set, each drawn by one uniform and followed by one ratio-tracking
// estimate toward it, on the same stream in draw order.  Row i * draws + q receives the
// collision, the view direction, the drawn direction and its weight; rays that escape
// get zero rows.
__global__ void __launch_bounds__(256) k_first_hits_set(Medium M, TracerParams tp, int draws,
                                                        const float *ray_o, const float *ray_d,
                                                        int64_t N, uint64_t seed, uint64_t sample,
                                                        float *pos, float *view, float *light,
                                                        float *weight, float *direct, uint8_t *hit)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    V3 d;
    bool h = false;
    V3 x = v3(0, 0, 0);
    Rng r;
    int64_t steps = 0;
    if (unit(ray_d + 3 * i, d)) {
        const V3 o = v3(ray_o[3 * i], ray_o[3 * i + 1], ray_o[3 * i + 2]);
        r.init(seed, ((uint64_t)i << 20) + sample);
        h = delta_track(M, o, d, r, x, steps);
    }
    float sum = 0.f;
    for (int q = 0; q < draws; ++q) {
        const int64_t row = i * draws + q;
        float4 lw = make_float4(0.f, 0.f, 0.f, 0.f);
        if (h) {
            lw = tp.set_dw[set_pick(tp, r.bits24())];
            const V3 lj = v3(lw.x, lw.y, lw.z);
            sum += lw.w * phase_eval<true>(tp, true, dot(d, lj)) * ratio_track(M, x, lj, r, steps);
        }
        pos[3 * row] = x.x;
        pos[3 * row + 1] = x.y;
        pos[3 * row + 2] = x.z;
        view[3 * row] = h ? -d.x : 0.f;
        view[3 * row + 1] = h ? -d.y : 0.f;
        view[3 * row + 2] = h ? -d.z : 0.f;
        light[3 * row] = lw.x;
        light[3 * row + 1] = lw.y;
        light[3 * row + 2] = lw.z;
        weight[row] = lw.w;
    }
    direct[i] = h ? tp.albedo * tp.irradiance * sum / (float)draws : 0.f;
    hit[i] = h ? 1 : 0;
}

__global__ void __launch_bounds__(256) k_philox(const uint32_t *ck, int64_t n, uint32_t *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    Rng r;
    r.c0 = ck[6 * i];
    r.c1 = ck[6 * i + 1];
    r.c2 = ck[6 * i + 2];
    r.c3 = ck[6 * i + 3];
    r.k0 = ck[6 * i + 4];
    r.k1 = ck[6 * i + 5];
    r.refill();
#pragma unroll
    for (int j = 0; j < 4; ++j)
        out[4 * i + j] = r.buf[j];
}

// Training targets: t = log(1 + L_i) in FP32 at record stride `stride`.
__global__ void __launch_bounds__(256) k_targets(const double *li, int64_t N, int64_t stride,
                                                 float *t)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N)
        t[i * stride] = log1pf((float)li[i]);
}

// One camera sample per pixel added to the pixel sums (Sec. 4.4): radiance
// direct + albedo * E * L_i at a collision, with L_i from the network or, where
// the stencil leaves the grid (fallback flag), from the path-traced estimate; 0 for
// rays that escape.  sums holds (sum, sum of squares) per pixel in FP64; dsum the
// sum of the direct term alone.
__global__ void __launch_bounds__(256) k_accumulate(int64_t N, const uint8_t *hit,
                                                    const float *direct, const float *li_net,
                                                    const uint8_t *flags, const double *li_mc,
                                                    float albedo, float E, double *sums,
                                                    double *dsum, unsigned long long *n_fb)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    double e = 0.0, d = 0.0;
    if (hit[i]) {
        const bool fb = li_mc && (flags[i] & DS_FLAG_FALLBACK);
        const double li = fb ? li_mc[i] : (double)E * (double)li_net[i];
        d = (double)direct[i];
        e = d + (double)albedo * li;
        if (fb && n_fb)
            atomicAdd(n_fb, 1ull);
    }
    sums[2 * i] += e;
    sums[2 * i + 1] += e * e;
    if (dsum)
        dsum[2 * i] += d;
}

// One camera sample per pixel under a light set: direct + albedo * E * (1 / draws) *
// sum over the draws of weight * L_i (the network's per unit irradiance, or the
// path-traced estimate where the row's fallback flag is set).
__global__ void __launch_bounds__(256) k_accumulate_set(int64_t N, int draws, const uint8_t *hit,
                                                        const float *direct, const float *li_net,
                                                        const uint8_t *flags, const double *li_mc,
                                                        const float *weight, float albedo, float E,
                                                        double *sums, double *dsum,
                                                        unsigned long long *n_fb)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    double e = 0.0, d = 0.0;
    if (hit[i]) {
        double li = 0.0;
        unsigned long long nf = 0;
        for (int q = 0; q < draws; ++q) {
            const int64_t row = i * draws + q;
            const bool fb = li_mc && (flags[row] & DS_FLAG_FALLBACK);
            li += (double)weight[row] * (fb ? li_mc[row] : (double)li_net[row]);
            nf += fb ? 1 : 0;
        }
        d = (double)direct[i];
        e = d + (double)albedo * (double)E * li / draws;
        if (nf && n_fb)
            atomicAdd(n_fb, nf);
    }
    sums[2 * i] += e;
    sums[2 * i + 1] += e * e;
    if (dsum)
        dsum[2 * i] += d;
}

__global__ void __launch_bounds__(256) k_fill3(float *v, int64_t N, float x, float y, float z)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) {
        v[3 * i] = x;
        v[3 * i + 1] = y;
        v[3 * i + 2] = z;
    }
}

__global__ void __launch_bounds__(256) k_zero64(double *v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        v[i] = 0.0;
}

#define DS_TRY_MEDIUM(s, c)                \
    do {                                   \
        ds_status st_ = medium_cells(s, c); \
        if (st_)                           \
            return st_;                    \
    } while (0)

// Brick grid of the occupancy bits: the smallest bricks (2^s cells per axis) whose bits
// fit the walker's LDS table.
struct Bricks {
    int s, bx, by, bz, words;
};

Bricks bricks(const ds_cloud *c)
{
    Bricks b;
    for (b.s = 0;; ++b.s) {
        b.bx = ((c->nx + 1) >> b.s) + 1;
        b.by = ((c->ny + 1) >> b.s) + 1;
        b.bz = ((c->nz + 1) >> b.s) + 1;
        if ((int64_t)b.bx * b.by * b.bz <= 32 * (int64_t)kOccWords)
            break;
    }
    b.words = (b.bx * b.by * b.bz + 31) / 32;
    return b;
}

// The corner-packed extinction of the cloud and the bits of its occupied bricks (after the
// cells, in the same allocation), built on the first tracer call.
ds_status medium_cells(hipStream_t s, const ds_cloud *c)
{
    if (c->mu_cells)
        return DS_OK;
    const int64_t n = (int64_t)(c->nx + 2) * (c->ny + 2) * (c->nz + 2);
    const Bricks b = bricks(c);
    const int64_t occ64 = (b.words + 2) / 2;  // 8-byte units, the flag word included
    size_t bytes = sizeof(float4) * 2 * (size_t)n + 8 * (size_t)occ64;
    float4 *cells = static_cast<float4 *>(block_take(c->ctx, &bytes));
    DS_CHECK(cells, DS_ERR_OOM,
             "out of device memory for the corner-packed extinction (%lld cells of 32 bytes)",
             (long long)n);
    Level base = {};
    base.nx = c->nx;
    base.ny = c->ny;
    base.nz = c->nz;
    uint32_t *occ = reinterpret_cast<uint32_t *>(cells + 2 * n);
    ds_status st = cloud_pack32(s, c->mu, 1, &base, cells);
    if (!st)
        st = tracer_zero(s, reinterpret_cast<double *>(occ), occ64);
    if (!st) {
        k_occupied<<<(unsigned)(((int64_t)b.bx * b.by * b.bz + 3) / 4), 256, 0, s>>>(
            c->mu, c->nx, c->ny, c->nz, b.s, b.bx, b.by, b.bz, b.words, c->majorant, occ);
        if (hipError_t e = hipGetLastError())
            st = hip_fail(e, "occupied bricks");
    }
    if (st) {
        (void)hipFree(cells);
        return st;
    }
    c->mu_cells_bytes = bytes;
    c->mu_cells = cells;
    return DS_OK;
}

Medium medium(const ds_cloud *c, float ext_scale = 1.f)
{
    Medium M;
    M.cells = c->mu_cells;
    M.cx = c->nx + 2;
    M.cy = c->ny + 2;
    M.hx = (float)(c->nx + 1);
    M.hy = (float)(c->ny + 1);
    M.hz = (float)(c->nz + 1);
    M.amin = v3(c->aabb_min[0], c->aabb_min[1], c->aabb_min[2]);
    M.amax = v3((float)((double)c->aabb_min[0] + (double)c->nx * c->h0),
                (float)((double)c->aabb_min[1] + (double)c->ny * c->h0),
                (float)((double)c->aabb_min[2] + (double)c->nz * c->h0));
    M.inv_h = (float)(1.0 / (double)c->h0);
    M.maj = c->majorant;
    M.inv_ff = (float)(1.0 / ((double)c->majorant * (double)ext_scale));
    M.truncated = c->ctx->truncated;
    const Bricks b = bricks(c);
    M.occ = reinterpret_cast<const uint32_t *>(
        c->mu_cells + 2 * (int64_t)(c->nx + 2) * (c->ny + 2) * (c->nz + 2));
    M.occ_s = b.s;
    M.bx = b.bx;
    M.by = b.by;
    M.occ_words = b.words;
    return M;
}

Split split(int spp)
{
    Split sp;
    sp.nblk = (spp + kPaths - 1) / kPaths;
    sp.seg = 1;
    while (sp.seg < spp && sp.seg < kPaths)
        sp.seg <<= 1;
    return sp;
}

ds_status reduce_records(hipStream_t s, const double *partial, int64_t P, int nblk, int spp,
                         double *mean, double *var)
{
    k_finish_sums<<<(unsigned)((P + 255) / 256), 256, 0, s>>>(partial, P, nblk, spp, mean, var);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

// ------------------------------------------------------------------ which walk
// Teams pay for a window per flight, whatever its length; one thread per path pays for every
// collision, and a wave for its longest path.  So short paths are walked one per thread, and the
// more of them there are the longer they may be, as then nothing waits for the longest.  The
// measure is the box in mean free paths of the majorant, s (64^3 and 256^3 clouds, teams' time
// over one thread's for s = 4 / 8 / 16 / 32 / 60):
//   albedo 0.999,   64 paths    1.18 0.67 0.47 0.29 0.17      64000      1.59 0.98 0.57 0.38 0.30
//                  320000       2.25 1.69 1.03 0.66 0.48      3200000    3.01 2.18 1.38 0.79 0.52
//   albedo 0.5,   1000          1.20 1.00 0.76 0.43 0.31      320000     2.57 2.07 1.33 0.89 0.62
//   environment,  1000          1.32 1.01 0.76 0.67 0.54      320000     2.60 2.19 1.76 1.25 0.98
//   one interaction, 1000       1.49 1.29 0.91 0.65 0.49      320000     4.41 4.14 3.19 2.33 1.74
//   1 / 4 / 16 paths (s = 8)    1.48 1.20 0.92: three launches more
// The lines below follow the sizes at which both take as long, in paths (6 up to 2^15, 8 at 2^16,
// 16 at 3 10^5, 24 from 2 10^6 on), in interactions that a path may have (few: less to wait
// for) and for an environment (no ratio tracking).
double box_flights(const ds_cloud *c, double ext_scale)
{
    return (double)c->majorant * ext_scale * c->h0 * ((double)c->nx + c->ny + c->nz) / 3.0;
}

bool serial_paths(const ds_cloud *c, const TracerParams &tp, int64_t paths)
{
    const double n = (double)std::max<int64_t>(1, paths);
    double depth = 1.0 / std::max(1e-6, 1.0 - (double)tp.albedo);
    if (tp.max_interactions > 0)
        depth = std::min(depth, (double)tp.max_interactions);
    const bool env = tp.light_mode == 1, many = n > 32768.0, single = n < 4.0;
    if (env && single && depth <= 32.0)  // some twenty steps: 17 us, against 27 at any s
        return true;
    const double shallow = 1.0 + 5.0 * pow(depth, -2.5);
    double line = std::max(6.0 + 30.0 / n, std::min(24.0, 8.0 + 3.3 * (log2(n) - 16.0)));
    line *= many || single ? shallow : std::min(1.5, shallow);
    if (env)
        line *= many ? 3.0 : 1.5;
    return box_flights(c, tp.ext_scale) < line;
}

// A launch of one thread per path holds fewer than 2^32 threads, up to two per path.
constexpr int64_t kMaxSerial = (int64_t)1 << 31;

// First hits: one flight and one ratio estimate per ray.  From 2^18 rays on one thread per ray
// wins where the cells are near (64^3, 9 MB: 960 x 540 camera rays 1.58 to 1.09 for s = 4 to
// 130, 1024^2 2.7 to 2.1) or the flights short; teams win where every lookup waits for HBM
// (256^3, 550 MB: 960 x 540 rays 1.49 0.90 0.65 0.56 for s = 4 16 40 80, 1920 x 1080 1.89 1.09
// 0.86 0.77; 128^3 1.59 1.15 1.04 0.91 and 2.48 1.96 1.72 1.64) or with fewer rays (384^2: 0.3 to
// 0.76 everywhere).
bool serial_first_hits(const ds_cloud *c, const TracerParams &tp, int64_t rays)
{
    if (rays < (int64_t)1 << 18 || rays >= kMaxSerial)
        return false;
    const double r = (double)rays / (1 << 18);
    const double near = (double)(1 << 27) / (32.0 * (c->nx + 2.0) * (c->ny + 2.0) * (c->nz + 2.0));
    return box_flights(c, tp.ext_scale) < 4.0 + 8.0 * r * sqrt(r) * near;
}

// Record draws: tries of one flight each, most of them a miss in thin clouds.  One thread per
// record where a try is a flight or two and there are records enough to hide the longest
// series of tries, or none to share with (s = 1 / 2 / 4: 262144 records 1.62 1.38 1.05, 40000
// 0.93 0.74 0.60, one 1.30 1.17 1.02, four at s = 4 0.92).
bool serial_draws(const ds_cloud *c, int64_t n)
{
    return box_flights(c, 1.0) < 4.0 && (n < 3 || n >= 200000) && n < kMaxSerial;
}

unsigned grid_of(int64_t n, Split sp)
{
    const int64_t rpb = kPaths / sp.seg;
    return (unsigned)(((n + rpb - 1) / rpb) * sp.nblk);
}

// Paths per launch: the per-path values of one launch take at most 8 bytes x this (or one
// record's paths).  At 2e7 paths/s a launch of 2^23 paths lasts some 0.4 s, so that the
// few milliseconds in which its longest paths run alone do not count.
constexpr int64_t kLaunchPaths = 1ll << 23;

int64_t launch_records(int64_t P, int64_t spp)
{
    return std::min<int64_t>(P, std::max<int64_t>(1, kLaunchPaths / spp));
}

// Scratch of the walker's launches: counters (active records, queue heads), the list of
// active records, the path values.
constexpr size_t kCounterBytes = 4 * kQueueStride * (1 + kQueues);

struct PathScratch {
    int32_t *counters, *list;
    double *val;
};

PathScratch path_scratch(void *ws, int64_t P)
{
    char *b = static_cast<char *>(ws);
    PathScratch r;
    r.counters = reinterpret_cast<int32_t *>(b);
    r.list = reinterpret_cast<int32_t *>(b + kCounterBytes);
    r.val = reinterpret_cast<double *>(
        b + kCounterBytes + (4 * (size_t)std::min<int64_t>(P, kLaunchPaths) + 255) / 256 * 256);
    return r;
}

// Waves of a walk: as many as the chip holds at the kernel's registers, or fewer where there
// are not enough paths; with few paths teams of 16 shorten each path's chain.  First hits
// are one flight to the first collision, so a wave is better off with more rays than with
// longer windows (two samples of 518400 camera rays with prediction: teams of 4 5.80 ms, of
// 8 5.96 ms, of 16 6.22 ms); walks with bounces are not (records of 2048 x 256 paths: 47.7,
// 36.0 and 39 to 44 ms).
constexpr int64_t kFewPaths = 1 << 14;
constexpr int kTeamFew = 16;
constexpr int team_of(int kind) { return kind == kFirstHits ? 4 : 8; }
constexpr int kComputeUnits = 256;

template <int KIND, bool TAB, bool SET, bool DIRECT>
void walk(hipStream_t s, const Medium &M, const TracerParams &tp, PathArgs &A, int64_t paths)
{
    const bool few = paths <= kFewPaths;
    const int team = few ? kTeamFew : team_of(KIND), teams = kWalkThreads / team;  // per block
    const int64_t blocks = std::min<int64_t>((paths + teams - 1) / teams,
                                             kComputeUnits * kWalkBlocks);
    const int64_t per = paths / (blocks * (kWalkThreads / 64) * 4);  // a quarter of a wave's share
    A.queues = (uint32_t)std::max<int64_t>(1, std::min<int64_t>(kQueues, blocks / 16));
    A.grab = (int)std::max<int64_t>(A.head ? 1 : 64 / team, std::min<int64_t>(per, 16));
    if (few)
        k_paths<KIND, TAB, SET, DIRECT, kTeamFew><<<(unsigned)blocks, kWalkThreads, 0, s>>>(M, tp, A);
    else
        k_paths<KIND, TAB, SET, DIRECT, team_of(KIND)>
            <<<(unsigned)blocks, kWalkThreads, 0, s>>>(M, tp, A);
}

// One walk per item without sums (first hits, record draws); waves take fixed shares, so the
// call needs no workspace.
template <int KIND, bool TAB>
ds_status walk_items(hipStream_t s, const Medium &M, const TracerParams &tp, PathArgs &A, int64_t N)
{
    for (A.rec0 = 0; A.rec0 < N; A.rec0 += kLaunchPaths) {
        A.n = (uint32_t)std::min<int64_t>(kLaunchPaths, N - A.rec0);
        walk<KIND, TAB, false, false>(s, M, tp, A, A.n);
        DS_HIP(hipGetLastError());
    }
    return DS_OK;
}

// Path values of P records (or pixels) and their partial sums: list the active records, then
// in launches of at most kLaunchPaths paths walk their paths and add each record's values
// up.  The list's length stays on the device; launches past it end at once.
template <class Launch>
ds_status walk_records(hipStream_t s, const float *dir, const float *light, const uint8_t *mask,
                       uint8_t mask_bits, PathArgs &A, int64_t P, double *partial, void *ws,
                       Launch launch)
{
    const Split sp = split(A.spp);
    const PathScratch r = path_scratch(ws, P);
    const int64_t per = launch_records(P, A.spp);  // records of a launch
    for (int64_t rec0 = 0; rec0 < P; rec0 += kLaunchPaths) {
        const int n = (int)std::min<int64_t>(kLaunchPaths, P - rec0);
        ds_status st = tracer_zero(s, reinterpret_cast<double *>(r.counters), kCounterBytes / 8);
        if (st)
            return st;
        k_active<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(dir, light, mask, mask_bits, rec0, n,
                                                             sp.nblk, partial, r.list, r.counters);
        A.list = r.list;
        A.n_list = r.counters;
        A.head = reinterpret_cast<uint32_t *>(r.counters + kQueueStride);
        A.rec0 = rec0;
        A.val = r.val;
        for (int64_t slot0 = 0; slot0 < n; slot0 += per) {
            A.slot0 = (uint32_t)slot0;
            A.n = (uint32_t)std::min<int64_t>(per, n - slot0);
            launch((int64_t)A.n * A.spp);
            const int64_t lanes = kPaths / sp.seg, units = (A.n + lanes - 1) / lanes * sp.nblk;
            k_path_sums<<<(unsigned)std::min<int64_t>(units, 4096), kPaths, 0, s>>>(
                r.val, r.list, r.counters, A.head, rec0, (int)slot0, (int)A.n, A.spp, sp, partial);
            DS_HIP(hipGetLastError());
        }
    }
    return DS_OK;
}

// The walk a call needs: one thread per path or teams, and of these the specialisation for
// tabulated phase functions and L_s records, tables and light sets (pixels).  paths: those
// expected to be walked.
ds_status launch_trace_li(hipStream_t s, const ds_cloud *c, const TracerParams &tp,
                          const float *pos, const float *view, const float *light, int64_t P,
                          int s0, int spp, uint64_t seed, const uint8_t *mask, uint8_t mask_bits,
                          int64_t paths, double *partial, void *ws)
{
    PathArgs A = {};
    A.a = pos;
    A.b = view;
    A.light = light;
    A.spp = spp;
    A.s0 = s0;
    A.seed = seed;
    const Medium M = medium(c, tp.ext_scale);
    const bool tab = tp.ph_n > 0 || tp.pf_n > 0, dir = tp.include_direct != 0;
    if (P * spp < kMaxSerial && serial_paths(c, tp, paths)) {
        const Split sp = split(spp);
        auto k = tab ? (dir ? k_trace_li<true, true> : k_trace_li<true, false>)
                     : (dir ? k_trace_li<false, true> : k_trace_li<false, false>);
        k<<<grid_of(P, sp), kPaths, 0, s>>>(M, tp, pos, view, light, P, s0, spp, sp, seed, mask,
                                            mask_bits, partial);
        DS_HIP(hipGetLastError());
        return DS_OK;
    }
    auto k = tab ? (dir ? walk<kRecordPaths, true, false, true> : walk<kRecordPaths, true, false, false>)
                 : (dir ? walk<kRecordPaths, false, false, true>
                        : walk<kRecordPaths, false, false, false>);
    return walk_records(s, view, light, mask, mask_bits, A, P, partial, ws,
                        [&](int64_t paths) { k(s, M, tp, A, paths); });
}

ds_status launch_render_mc(hipStream_t s, const ds_cloud *c, const TracerParams &tp, V3 wl,
                           const float *ray_o, const float *ray_d, int64_t N, int spp,
                           uint64_t seed, double *partial, void *ws)
{
    PathArgs A = {};
    A.a = ray_o;
    A.b = ray_d;
    A.wl = wl;
    A.spp = spp;
    A.seed = seed;
    const Medium M = medium(c, tp.ext_scale);
    const bool tab = tp.ph_n > 0 || tp.pf_n > 0, set = tp.light_mode == kLightSetMode;
    if (N * spp < kMaxSerial && serial_paths(c, tp, N * spp)) {
        const Split sp = split(spp);
        auto k = tab ? (set ? k_render_mc<true, true> : k_render_mc<true, false>)
                     : (set ? k_render_mc<false, true> : k_render_mc<false, false>);
        k<<<grid_of(N, sp), kPaths, 0, s>>>(M, tp, wl, ray_o, ray_d, N, spp, sp, seed, partial);
        DS_HIP(hipGetLastError());
        return DS_OK;
    }
    auto k = tab ? (set ? walk<kPixelPaths, true, true, false> : walk<kPixelPaths, true, false, false>)
                 : (set ? walk<kPixelPaths, false, true, false>
                        : walk<kPixelPaths, false, false, false>);
    return walk_records(s, ray_d, nullptr, nullptr, 0, A, N, partial, ws,
                        [&](int64_t paths) { k(s, M, tp, A, paths); });
}

}  // namespace

size_t tracer_ws(int64_t P, int spp)
{
    const size_t vals = (size_t)launch_records(P, spp) * (size_t)spp;
    return kCounterBytes + 256 + 4 * (size_t)std::min<int64_t>(P, kLaunchPaths) +
           8 * std::max<size_t>(vals, (size_t)std::min<int64_t>(P * (int64_t)spp, kLaunchPaths));
}

ds_status tracer_li(hipStream_t s, const ds_cloud *c, const TracerParams &tp, const float *pos,
                    const float *view, const float *light, int64_t P, int spp, uint64_t seed,
                    double *partial, double *mean, double *var, const uint8_t *mask,
                    uint8_t mask_bits)
{
    const int nblk = tracer_blocks(spp);
    DS_TRY_MEDIUM(s, c);
    // of a masked call (a frame's points whose stencils leave the grid) few records are wanted
    ds_status st = launch_trace_li(s, c, tp, pos, view, light, P, 0, spp, seed, mask, mask_bits,
                                   mask ? P * spp / 16 : P * spp, partial, partial + 2 * P * nblk);
    if (st)
        return st;
    return reduce_records(s, partial, P, nblk, spp, mean, var);
}

// Batches a round of the progressive estimate traces: one while the records still running
// fill the GPU (kAheadThreads threads), more as they thin out, up to `ahead`.  Tracing
// several batches at once keeps every block partial and its order (the batch is a whole
// number of blocks), so estimates and path counts equal those of one batch per round.
constexpr int64_t kAheadThreads = 1ll << 21;

ds_status tracer_li_adaptive(hipStream_t s, const ds_cloud *c, const TracerParams &tp,
                             const float *pos, const float *view, const float *light, int64_t P,
                             int batch, int max_spp, int ahead, double rel, double zq,
                             uint64_t seed, double *partial, uint8_t *active, double *sums,
                             unsigned long long *left, double *mean, double *var, int32_t *n_out,
                             int *rounds)
{
    const Split sp1 = split(batch);
    const bool whole = batch % kPaths == 0;
    const unsigned g256 = (unsigned)((P + 255) / 256);
    DS_TRY_MEDIUM(s, c);
    k_adapt_init<<<g256, 256, 0, s>>>(view, light, P, active, sums, mean, var, n_out);
    DS_HIP(hipGetLastError());
    int r = 0;
    int64_t live = P;
    for (int n = 0; n < max_spp;) {
        int kb = 1;
        if (whole && ahead > 1) {
            const int64_t want = (kAheadThreads + live * batch - 1) / (live * batch);
            kb = (int)std::max<int64_t>(
                1, std::min<int64_t>(want, std::min<int64_t>(ahead, (max_spp - n) / batch)));
        }
        ++r;
        ds_status st = launch_trace_li(s, c, tp, pos, view, light, P, n, kb * batch, seed, active, 1,
                                       live * kb * batch, partial,
                                       partial + 2 * P * sp1.nblk * ahead);
        if (st)
            return st;
        unsigned long long h = 0;
        DS_HIP(hipMemsetAsync(left, 0, sizeof(*left), s));
        k_adapt_step<<<g256, 256, 0, s>>>(partial, sp1.nblk, kb, P, n, batch, max_spp, rel, zq,
                                          active, sums, mean, var, n_out, left);
        DS_HIP(hipGetLastError());
        DS_HIP(hipMemcpyAsync(&h, left, sizeof(h), hipMemcpyDeviceToHost, s));
        DS_HIP(hipStreamSynchronize(s));
        n += kb * batch;
        if (h == 0)
            break;
        live = (int64_t)h;
    }
    if (rounds)
        *rounds = r;
    return DS_OK;
}

// Batches ahead a progressive estimate of P records may trace in one round: 1 unless a
// batch is a whole number of blocks; else up to 64 (and the cap), within 256 MiB of
// partial sums.
int tracer_adaptive_ahead(int64_t P, int batch, int max_spp)
{
    if (batch % kPaths != 0 || P <= 0)
        return 1;
    const int64_t per = 16 * P * (batch / kPaths);
    const int64_t k = std::min<int64_t>(std::min<int64_t>(64, max_spp / batch),
                                        (256ll << 20) / per);
    return (int)std::max<int64_t>(1, k);
}

ds_status tracer_records(hipStream_t s, const ds_cloud *c, int64_t N, uint64_t seed, float *pos,
                         float *view, float *light, int32_t *attempts)
{
    DS_TRY_MEDIUM(s, c);
    if (serial_draws(c, N)) {
        k_sample_records<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(medium(c), N, seed, pos, view,
                                                                     light, attempts);
        DS_HIP(hipGetLastError());
        return DS_OK;
    }
    PathArgs A = {};
    A.spp = 1;
    A.seed = seed;
    A.pos = pos;
    A.view = view;
    A.light_out = light;
    A.tries = attempts;
    return walk_items<kRecordDraws, false>(s, medium(c), TracerParams{}, A, N);
}

ds_status tracer_render(hipStream_t s, const ds_cloud *c, const TracerParams &tp,
                        const float *light_dir, const float *ray_o, const float *ray_d, int64_t N,
                        int spp, uint64_t seed, double *partial, double *mean, double *var)
{
    float l[3];
    DS_CHECK(light_dir && unit_host(light_dir, l), DS_ERR_INVALID_ARG,
             "the light direction is not a usable vector");
    const V3 wl = v3(l[0], l[1], l[2]);
    const int nblk = tracer_blocks(spp);
    DS_TRY_MEDIUM(s, c);
    ds_status st = launch_render_mc(s, c, tp, wl, ray_o, ray_d, N, spp, seed, partial,
                                    partial + 2 * N * nblk);
    if (st)
        return st;
    return reduce_records(s, partial, N, nblk, spp, mean, var);
}

ds_status tracer_first_hits(hipStream_t s, const ds_cloud *c, const TracerParams &tp,
                            const float *light_dir, const float *ray_o, const float *ray_d,
                            int64_t N, uint64_t seed, uint64_t sample, float *pos, float *view,
                            float *direct, uint8_t *hit)
{
    float l[3];
    DS_CHECK(light_dir && unit_host(light_dir, l), DS_ERR_INVALID_ARG,
             "the light direction is not a usable vector");
    const V3 wl = v3(l[0], l[1], l[2]);
    DS_TRY_MEDIUM(s, c);
    if (serial_first_hits(c, tp, N)) {
        k_first_hits<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(medium(c, tp.ext_scale), tp, wl,
                                                                 ray_o, ray_d, N, seed, sample, pos,
                                                                 view, direct, hit);
        DS_HIP(hipGetLastError());
        return DS_OK;
    }
    PathArgs A = {};
    A.a = ray_o;
    A.b = ray_d;
    A.wl = wl;
    A.spp = 1;
    A.seed = seed;
    A.sample = sample;
    A.pos = pos;
    A.view = view;
    A.direct = direct;
    A.hit = hit;
    return walk_items<kFirstHits, true>(s, medium(c, tp.ext_scale), tp, A, N);
}

ds_status philox_blocks(hipStream_t s, const uint32_t *ctr_key, int64_t n, uint32_t *out)
{
    k_philox<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(ctr_key, n, out);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status tracer_targets(hipStream_t s, const double *li, int64_t N, int64_t stride, float *t)
{
    k_targets<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(li, N, stride, t);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status tracer_accumulate(hipStream_t s, int64_t N, const uint8_t *hit, const float *direct,
                            const float *li_net, const uint8_t *flags, const double *li_mc,
                            float albedo, float E, double *sums, double *dsum,
                            unsigned long long *n_fb)
{
    k_accumulate<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(N, hit, direct, li_net, flags, li_mc,
                                                             albedo, E, sums, dsum, n_fb);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status tracer_fill3(hipStream_t s, float *v, int64_t N, const float *xyz)
{
    k_fill3<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(v, N, xyz[0], xyz[1], xyz[2]);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status tracer_zero(hipStream_t s, double *v, int64_t n)
{
    int64_t b = (n + 255) / 256;
    k_zero64<<<(unsigned)(b > 4096 ? 4096 : (b < 1 ? 1 : b)), 256, 0, s>>>(v, n);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status tracer_finish(hipStream_t s, const double *sums, int64_t N, int spp, double *mean,
                        double *var)
{
    return reduce_records(s, sums, N, 1, spp, mean, var);
}

ds_status tracer_first_hits_set(hipStream_t s, const ds_cloud *c, const TracerParams &tp,
                                int draws, const float *ray_o, const float *ray_d, int64_t N,
                                uint64_t seed, uint64_t sample, float *pos, float *view,
                                float *light, float *weight, float *direct, uint8_t *hit)
{
    DS_CHECK(tp.light_mode == kLightSetMode && tp.set_dw && tp.set_thr && tp.set_m >= 1,
             DS_ERR_INVALID_ARG, "internal error: no light set");
    DS_TRY_MEDIUM(s, c);
    k_first_hits_set<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(
        medium(c, tp.ext_scale), tp, draws, ray_o, ray_d, N, seed, sample, pos, view, light, weight, direct, hit);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status tracer_accumulate_set(hipStream_t s, int64_t N, int draws, const uint8_t *hit,
                                const float *direct, const float *li_net, const uint8_t *flags,
                                const double *li_mc, const float *weight, float albedo, float E,
                                double *sums, double *dsum, unsigned long long *n_fb)
{
    k_accumulate_set<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(
        N, draws, hit, direct, li_net, flags, li_mc, weight, albedo, E, sums, dsum, n_fb);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

int tracer_blocks(int spp) { return split(spp).nblk; }

}  // namespace ds
