// Per-cloud precompute: mean extinction over non-zero voxels (Sec. 4.2, 5) and the
// Gaussian density mipmap with sigma_i = 2^i base voxels (Sec. 6), plus the
// corner-packed FP16 copy of every level read by the fused prediction kernel.
#include <math.h>

#include <algorithm>
#include <vector>

#include "internal.h"

namespace ds {
namespace {

__device__ __forceinline__ float load_density(const void *d, ds_dtype dt, int64_t i)
{
    if (dt == DS_F32)
        return static_cast<const float *>(d)[i];
    uint32_t b = static_cast<uint32_t>(static_cast<const uint16_t *>(d)[i]) << 16;
    return __uint_as_float(b);
}

// Error-free sum of two floats (Knuth's two-sum), used to combine (hi, lo) pairs.
__device__ __forceinline__ void two_sum(float a, float b, float &s, float &e)
{
    s = a + b;
    float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

__device__ __forceinline__ void dd_add(float &hi, float &lo, float bhi, float blo)
{
    float s, e;
    two_sum(hi, bhi, s, e);
    e += lo + blo;
    hi = s + e;
    lo = e - (hi - s);
}

constexpr int kMeanBlocks = 1024;
constexpr int kMeanThreads = 256;

// Block-level (hi, lo, maximum, count) reduction in LDS; deterministic order.
__device__ void block_reduce(float &hi, float &lo, float &m, unsigned long long &cnt)
{
    __shared__ float shi[kMeanThreads], slo[kMeanThreads], sm[kMeanThreads];
    __shared__ unsigned long long sc[kMeanThreads];
    int t = threadIdx.x;
    shi[t] = hi;
    slo[t] = lo;
    sm[t] = m;
    sc[t] = cnt;
    __syncthreads();
    for (int w = kMeanThreads / 2; w > 0; w >>= 1) {
        if (t < w) {
            float h = shi[t], l = slo[t];
            dd_add(h, l, shi[t + w], slo[t + w]);
            shi[t] = h;
            slo[t] = l;
            sm[t] = fmaxf(sm[t], sm[t + w]);
            sc[t] += sc[t + w];
        }
        __syncthreads();
    }
    hi = shi[0];
    lo = slo[0];
    m = sm[0];
    cnt = sc[0];
}

// One pass over the density: per-block sums and counts of d over d > 0 (Kahan-compensated per
// thread) and the largest extinction sigma d.  Bound by reading the density; eight loads of
// a thread in flight.
__global__ void __launch_bounds__(kMeanThreads) k_scan_density(const void *d, ds_dtype dt, int64_t n,
                                                               float sigma, float2 *part,
                                                               float *pmax,
                                                               unsigned long long *pcnt)
{
    constexpr int U = 8;
    float sum = 0.f, c = 0.f, m = 0.f;
    unsigned long long cnt = 0;
    auto add = [&](float v) {
        if (v > 0.f) {
            float y = v - c;
            float t = sum + y;
            c = (t - sum) - y;
            sum = t;
            ++cnt;
        }
    };
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + (U - 1) * stride < n; i += U * stride) {
        float v[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            v[k] = load_density(d, dt, i + k * stride);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            m = fmaxf(m, sigma * v[k]);
            add(v[k]);
        }
    }
    for (; i < n; i += stride) {
        const float v = load_density(d, dt, i);
        m = fmaxf(m, sigma * v);
        add(v);
    }
    float hi = sum, lo = -c;
    block_reduce(hi, lo, m, cnt);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = make_float2(hi, lo);
        pmax[blockIdx.x] = m;
        pcnt[blockIdx.x] = cnt;
    }
}

__global__ void __launch_bounds__(kMeanThreads) k_scan_final(const float2 *part, const float *pmax,
                                                             const unsigned long long *pcnt,
                                                             int nb, DensityScan *out)
{
    float hi = 0.f, lo = 0.f, m = 0.f;
    unsigned long long cnt = 0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) {
        dd_add(hi, lo, part[i].x, part[i].y);
        m = fmaxf(m, pmax[i]);
        cnt += pcnt[i];
    }
    block_reduce(hi, lo, m, cnt);
    if (threadIdx.x == 0) {
        out->hi = hi;
        out->lo = lo;
        out->max = m;
        out->count = cnt;
    }
}

// sum_e w[e] v(e) over e0 <= e < e1, Kahan-compensated in order, eight loads ahead.
template <class Load>
__device__ __forceinline__ float taps_sum(const float *__restrict__ w, int e0, int e1, Load load)
{
    constexpr int U = 8;
    float sum = 0.f, c = 0.f;
    auto add = [&](float we, float v) {
        const float y2 = fmaf(we, v, -c);
        const float t = sum + y2;
        c = (t - sum) - y2;
        sum = t;
    };
    int e = e0;
    for (; e + U <= e1; e += U) {
        float v[U], u[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            v[k] = load(e + k);
            u[k] = w[e + k];
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            add(u[k], v[k]);
    }
    for (; e < e1; ++e)
        add(w[e], load(e));
    return sum;
}

// Separable Gaussian passes with decimation by s = 2^level: output sample m is
// sum_e w[e] in[m s + emin + e], zero outside the input.
//
// Along x a block takes R rows whole into LDS, read once for all levels (and for the
// extinction mu = sigma d, written on the way), and its threads the rows' outputs level by
// level.  A thread per output reading memory strides 2^level elements between neighbours
// and reads the density once per level: 126 us per level of a 256^3 cloud, 1.13 ms for nine,
// against 0.22 ms here (4 vector operations and an LDS read per tap bound it, 54 taps a
// voxel over nine levels).  The rows are skewed by one word in 32 so that those strides do
// not meet in one bank.
constexpr int kMaxRow = 4096;                           // voxels along an axis
constexpr int kRowWords = kMaxRow + kMaxRow / 32;       // LDS floats for rows
__device__ __forceinline__ int skewed(int x) { return x + (x >> 5); }

struct XLevels {
    int L;
    int nout[kMaxLevels], emin[kMaxLevels], first[kMaxLevels + 1];  // outputs per row, taps
    int64_t off[kMaxLevels];                                        // of the level's volume
};

__global__ void __launch_bounds__(256) k_blur_rows(const void *in, ds_dtype dt, float scale,
                                                   float sigma, float *mu, float *out, int n0,
                                                   int64_t rows, int R, XLevels X,
                                                   const float *__restrict__ w)
{
    __shared__ float row[kRowWords];
    constexpr int U = 4;
    const int64_t r0 = (int64_t)blockIdx.x * R, i0 = r0 * n0;
    const int nr = (int)(rows - r0 < R ? rows - r0 : R), total = nr * n0;
    int t = threadIdx.x;
    for (; t + (U - 1) * 256 < total; t += U * 256) {
        float v[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            v[k] = load_density(in, dt, i0 + t + 256 * k);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            row[skewed(t + 256 * k)] = v[k] * scale;
            mu[i0 + t + 256 * k] = sigma * v[k];
        }
    }
    for (; t < total; t += 256) {
        const float v = load_density(in, dt, i0 + t);
        row[skewed(t)] = v * scale;
        mu[i0 + t] = sigma * v;
    }
    __syncthreads();
    for (int i = 0; i < X.L; ++i) {
        const int nout = X.nout[i], emin = X.emin[i], nt = X.first[i + 1] - X.first[i];
        for (int o = threadIdx.x; o < nr * nout; o += 256) {
            const int r = o / nout, j0 = ((o - r * nout) << i) + emin, q = r * n0 + j0;
            out[X.off[i] + r0 * nout + o] =
                taps_sum(w + X.first[i], j0 < 0 ? -j0 : 0, min(nt, n0 - j0),
                         [&](int e) { return row[skewed(q + e)]; });
        }
    }
}

// Row work of all levels in one launch: level i's rows (of `width` elements, 64 a wave, four
// waves a block) own the blocks from block[i] on.  The coarse levels come first: their few
// rows are long serial sums, which then overlap the fine levels' traffic (nine levels of a
// 256^3 cloud, y and z: 600 us as 18 launches with a division per element, 245 us as two;
// the packing 175 -> 153 us).
struct LevelRows {
    int L;
    uint32_t block[kMaxLevels + 1], rows[kMaxLevels];
    // the level, blocks across a row, consecutive rows a wave takes (finding its place costs a
    // wave a microsecond of dependent scalar loads, so fine levels give it many)
    uint32_t level[kMaxLevels], wide[kMaxLevels], per[kMaxLevels];
};

struct RowPos {
    uint32_t level, row, end, col;  // the wave's level and rows row .. end - 1
};

__device__ __forceinline__ RowPos row_pos(const LevelRows &W)
{
    int n = 0;
    while (n + 1 < W.L && blockIdx.x >= W.block[n + 1])
        ++n;
    const uint32_t b = blockIdx.x - W.block[n], r = b / W.wide[n];
    RowPos p;
    p.level = W.level[n];
    p.row = (r * 4 + __builtin_amdgcn_readfirstlane(threadIdx.y)) * W.per[n];
    p.end = min(p.row + W.per[n], W.rows[n]);
    p.col = (b - r * W.wide[n]) * 64 + threadIdx.x;
    return p;
}

// Rows per level and their widths to a launch: returns its blocks.
template <class Rows, class Width>
int64_t level_rows(LevelRows &W, int L, Rows rows, Width width)
{
    W.L = L;
    int64_t at = 0;
    for (int n = 0; n < L; ++n) {
        const int i = L - 1 - n;
        W.level[n] = i;
        W.block[n] = (uint32_t)at;
        W.rows[n] = (uint32_t)rows(i);
        W.wide[n] = (uint32_t)((width(i) + 63) / 64);
        W.per[n] = std::max<uint32_t>(
            1, std::min<uint32_t>(16, (uint32_t)((uint64_t)W.rows[n] * W.wide[n] / 8192)));
        at += (int64_t)((W.rows[n] + 4 * W.per[n] - 1) / (4 * W.per[n])) * W.wide[n];
    }
    W.block[L] = (uint32_t)at;
    return at;
}

// One axis of every level: out[b][m][a] from in[b][j][a], a < na contiguous in both; a wave
// takes 64 consecutive a of one output row, so loads coalesce and no thread divides.
struct AxisLevels {
    int64_t in[kMaxLevels], out[kMaxLevels], na[kMaxLevels];  // element offsets, row length
    int nj[kMaxLevels], nout[kMaxLevels], emin[kMaxLevels], first[kMaxLevels + 1];
};

__global__ void __launch_bounds__(256) k_blur_strided(const float *in, float *out, AxisLevels X,
                                                      LevelRows W, const float *__restrict__ w)
{
    const RowPos p = row_pos(W);
    const int i = (int)p.level;
    const int64_t na = X.na[i];
    if (p.col >= na)
        return;
    const uint32_t nout = (uint32_t)X.nout[i];
    const int nj = X.nj[i], emin = X.emin[i], nt = X.first[i + 1] - X.first[i];
    const float *src = in + X.in[i] + p.col, *wl = w + X.first[i];
    float *dst = out + X.out[i] + p.col;
    for (uint32_t row = p.row; row < p.end; ++row) {
        const uint32_t b = row / nout;
        const int j0 = ((int)(row - b * nout) << i) + emin;
        const float *q = src + ((int64_t)b * nj + j0) * na;
        dst[(int64_t)row * na] = taps_sum(wl, j0 < 0 ? -j0 : 0, min(nt, nj - j0),
                                          [&](int e) { return q[(int64_t)e * na]; });
    }
}

// FP16 bits of f, round to nearest even, saturated at the largest finite magnitude.
__device__ __forceinline__ uint32_t f16_sat(float f)
{
    const _Float16 h = (_Float16)fmaxf(fminf(f, 65504.f), -65504.f);
    return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

// Corner-packed level with a zero border of bd cells: cell (i, j, k) covers the lattice
// cell whose lower corner is voxel (i - bd, j - bd, k - bd), values zero outside the level
// grid.  Its trilinear function is stored as polynomial coefficients in the fractions
// (tx, ty, tz):  v(t) = P0(ty, tz) + tx P1(ty, tz),  P = A + B ty + tz (C + D ty),
// with P0 the bilinear function of the x0 face and P1 that of the x1 face minus the x0
// face.  FP16, word 0 = (A0, A1), 1 = (B0, B1), 2 = (C0, C1), 3 = (D0, D1), the P0
// coefficient in the low half; the coefficients are formed in FP32 from the level and
// rounded once.  Evaluating this form takes three packed FMAs and one mixed FMA.
// All levels in one launch; bound by writing the cells (16 bytes each; 256^3: 290 MB).
struct PackLevels {
    int nx[kMaxLevels], ny[kMaxLevels], nz[kMaxLevels], bd[kMaxLevels];
    int64_t off[kMaxLevels], cell_off[kMaxLevels];
};

__global__ void __launch_bounds__(256) k_pack(const float *__restrict__ pyr, PackLevels X, LevelRows W,
                                              uint4 *__restrict__ cells)
{
    const RowPos p = row_pos(W);
    const int l = (int)p.level, nx = X.nx[l], ny = X.ny[l], nz = X.nz[l], bd = X.bd[l];
    const int cx = nx + 2 * bd, cy = ny + 2 * bd;
    if ((int)p.col >= cx)
        return;
    const float *lv = pyr + X.off[l];
    const int i = (int)p.col - bd;
    for (uint32_t row = p.row; row < p.end; ++row) {
        const uint32_t kk = row / (uint32_t)cy;
        const int k = (int)kk - bd, j = (int)(row - kk * cy) - bd;
        float v[8];  // corner dx + 2 dy + 4 dz
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int a = i + (c & 1), b = j + ((c >> 1) & 1), e = k + ((c >> 2) & 1);
            const bool in = a >= 0 && b >= 0 && e >= 0 && a < nx && b < ny && e < nz;
            v[c] = in ? lv[((int64_t)e * ny + b) * nx + a] : 0.f;
        }
        uint32_t w[4];
        float co[2][4];
#pragma unroll
        for (int x = 0; x < 2; ++x) {  // bilinear coefficients of the x = 0 and x = 1 faces
            const float f00 = v[x], f10 = v[x + 2], f01 = v[x + 4], f11 = v[x + 6];
            co[x][0] = f00;
            co[x][1] = f10 - f00;
            co[x][2] = f01 - f00;
            co[x][3] = (f11 - f01) - (f10 - f00);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            w[q] = f16_sat(co[0][q]) | (f16_sat(co[1][q] - co[0][q]) << 16);
        cells[X.cell_off[l] + (int64_t)row * cx + p.col] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Corner-packed float32 level (the plain gather's copy): cell (i, j, k) holds the 8
// corners of the lattice cell whose lower corner is voxel (i - 1, j - 1, k - 1), corner
// c = dx + 2 dy + 4 dz at float c of the cell's 32 bytes, zero outside the grid.
__global__ void __launch_bounds__(256) k_pack32(const float *__restrict__ lv, int nx, int ny,
                                                int nz, float4 *__restrict__ cells)
{
    const int64_t cx = nx + 2, cy = ny + 2, cz = nz + 2;
    const int64_t total = cx * cy * cz;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
        const int64_t i = idx % cx - 1, r = idx / cx;
        const int64_t j = r % cy - 1, k = r / cy - 1;
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int64_t a = i + (c & 1), b = j + ((c >> 1) & 1), e = k + ((c >> 2) & 1);
            const bool in = a >= 0 && b >= 0 && e >= 0 && a < nx && b < ny && e < nz;
            v[c] = in ? lv[(e * ny + b) * nx + a] : 0.f;
        }
        cells[2 * idx] = make_float4(v[0], v[1], v[2], v[3]);
        cells[2 * idx + 1] = make_float4(v[4], v[5], v[6], v[7]);
    }
}

int grid_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    if (b > 65536)
        b = 65536;
    return (int)(b < 1 ? 1 : b);
}

// Normalised 1-D Gaussian taps of level i: weights for base offsets e = j - m 2^i
// in [emin, emin + ntaps), where t = e + 1/2 - 2^i / 2 lies within 3 sigma.  The
// normaliser runs over all such offsets, so grid borders are darkened, not renormalised.
void level_taps(int i, int *emin, std::vector<float> &w)
{
    double s = ldexp(1.0, i);
    int lo = (int)floor(-3.0 * s - 1.0 + 0.5 * s), hi = (int)ceil(3.0 * s + 1.0 + 0.5 * s);
    std::vector<double> wd;
    int first = 0;
    bool have = false;
    for (int e = lo; e <= hi; ++e) {
        double t = e + 0.5 - 0.5 * s;
        if (fabs(t) <= 3.0 * s) {
            if (!have) {
                first = e;
                have = true;
            }
            wd.push_back(exp(-t * t / (2.0 * s * s)));
        }
    }
    double z = 0.0;
    for (double v : wd)
        z += v;
    w.resize(wd.size());
    for (size_t k = 0; k < wd.size(); ++k)
        w[k] = (float)(wd[k] / z);
    *emin = first;
}

}  // namespace

// Scratch of a cloud's build: the partial sums of the density pass, the taps of every level.
struct BuildScratch {
    float2 *part;
    float *pmax;
    unsigned long long *pcnt;
    DensityScan *scan;
    float *taps;
    size_t bytes;
};

static BuildScratch build_scratch(void *ws, size_t taps)
{
    BuildScratch r;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = static_cast<char *>(ws) + off;
        off += (bytes + 255) / 256 * 256;
        return p;
    };
    r.part = reinterpret_cast<float2 *>(take(sizeof(float2) * kMeanBlocks));
    r.pmax = reinterpret_cast<float *>(take(4 * kMeanBlocks));
    r.pcnt = reinterpret_cast<unsigned long long *>(take(8 * kMeanBlocks));
    r.scan = reinterpret_cast<DensityScan *>(take(sizeof(DensityScan)));
    r.taps = reinterpret_cast<float *>(take(taps * 4));
    r.bytes = off;
    return r;
}

static size_t all_taps(int L, std::vector<float> *w, int *emin, int *first)
{
    size_t n = 0;
    std::vector<float> t;
    for (int i = 0; i < L; ++i) {
        int e;
        level_taps(i, &e, t);
        if (w) {
            emin[i] = e;
            first[i] = (int)n;
            w->insert(w->end(), t.begin(), t.end());
        }
        n += t.size();
    }
    if (w)
        first[L] = (int)n;
    return n;
}

size_t cloud_scratch_bytes(int L)
{
    return build_scratch(nullptr, all_taps(L, nullptr, nullptr, nullptr)).bytes;
}

ds_status cloud_scan(hipStream_t s, const void *d, ds_dtype dt, int64_t n, float sigma,
                     void *scratch, DensityScan *host)
{
    const BuildScratch r = build_scratch(scratch, 0);
    k_scan_density<<<kMeanBlocks, kMeanThreads, 0, s>>>(d, dt, n, sigma, r.part, r.pmax, r.pcnt);
    k_scan_final<<<1, kMeanThreads, 0, s>>>(r.part, r.pmax, r.pcnt, kMeanBlocks, r.scan);
    DS_HIP(hipGetLastError());
    DS_HIP(hipMemcpyAsync(host, r.scan, sizeof(*host), hipMemcpyDeviceToHost, s));
    DS_HIP(hipStreamSynchronize(s));
    return DS_OK;
}

ds_status cloud_pyramid(hipStream_t s, const void *d, ds_dtype dt, int nx, int ny, int nz,
                        float scale, float sigma, int L, const Level *lv, float *pyr, float *mu,
                        void *scratch, float *volumes)
{
    std::vector<float> taps;
    XLevels X;
    X.L = L;
    all_taps(L, &taps, X.emin, X.first);
    const BuildScratch r = build_scratch(scratch, taps.size());
    DS_HIP(hipMemcpy(r.taps, taps.data(), taps.size() * sizeof(float), hipMemcpyHostToDevice));
    const int64_t rows = (int64_t)ny * nz;
    int64_t off = 0;
    for (int i = 0; i < L; ++i) {
        X.nout[i] = lv[i].nx;
        X.off[i] = off;
        off += rows * lv[i].nx;
    }
    const int R = (int)std::min<int64_t>(kMaxRow / nx, std::max<int64_t>(1, rows / 1024));
    k_blur_rows<<<(unsigned)((rows + R - 1) / R), 256, 0, s>>>(d, dt, scale, sigma, mu, volumes, nx,
                                                               rows, R, X, r.taps);
    AxisLevels Y, Z;
    LevelRows W;
    for (int i = 0; i < L; ++i) {
        const Level &l = lv[i];
        Y.in[i] = X.off[i];
        Y.out[i] = Z.in[i] = off;
        off += (int64_t)l.nx * l.ny * nz;
        Z.out[i] = l.off;
        Y.na[i] = l.nx;
        Z.na[i] = (int64_t)l.nx * l.ny;
        Y.nj[i] = ny;
        Z.nj[i] = nz;
        Y.nout[i] = l.ny;
        Z.nout[i] = l.nz;
        Y.emin[i] = Z.emin[i] = X.emin[i];
    }
    for (int i = 0; i <= L; ++i)
        Y.first[i] = Z.first[i] = X.first[i];
    int64_t blocks = level_rows(W, L, [&](int i) { return (int64_t)lv[i].ny * nz; },
                                [&](int i) { return Y.na[i]; });
    k_blur_strided<<<(unsigned)blocks, dim3(64, 4), 0, s>>>(volumes, volumes, Y, W, r.taps);
    blocks = level_rows(W, L, [&](int i) { return (int64_t)lv[i].nz; },
                        [&](int i) { return Z.na[i]; });
    k_blur_strided<<<(unsigned)blocks, dim3(64, 4), 0, s>>>(volumes, pyr, Z, W, r.taps);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

// Floats of the partly filtered volumes: every level along x, and along x and y.
int64_t cloud_volume_floats(int ny, int nz, int L, const Level *lv)
{
    int64_t n = 0;
    for (int i = 0; i < L; ++i)
        n += (int64_t)lv[i].nx * (ny + lv[i].ny) * nz;
    return n;
}

ds_status cloud_pack32(hipStream_t s, const float *pyr, int L, const Level *lv, float4 *cells)
{
    for (int i = 0; i < L; ++i) {
        const Level &l = lv[i];
        int64_t n = (int64_t)(l.nx + 2) * (l.ny + 2) * (l.nz + 2);
        k_pack32<<<grid_for(n), 256, 0, s>>>(pyr + l.off, l.nx, l.ny, l.nz,
                                             cells + 2 * l.cell32_off);
    }
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status cloud_pack(hipStream_t s, const float *pyr, int L, const Level *lv, uint4 *cells)
{
    PackLevels X;
    for (int i = 0; i < L; ++i) {
        X.nx[i] = lv[i].nx;
        X.ny[i] = lv[i].ny;
        X.nz[i] = lv[i].nz;
        X.bd[i] = lv[i].bd;
        X.off[i] = lv[i].off;
        X.cell_off[i] = lv[i].cell_off;
    }
    LevelRows W;
    const int64_t blocks = level_rows(
        W, L,
        [&](int i) { return (int64_t)(lv[i].ny + 2 * lv[i].bd) * (lv[i].nz + 2 * lv[i].bd); },
        [&](int i) { return (int64_t)lv[i].nx + 2 * lv[i].bd; });
    k_pack<<<(unsigned)blocks, dim3(64, 4), 0, s>>>(pyr, X, W, cells);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

}  // namespace ds
