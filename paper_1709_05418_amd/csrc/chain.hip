// The network's layers as two chains of small products (Sec. 4.3, Sec. 5.2).  A workgroup
// takes 16 or 32 rows (descriptors) through every layer: wave w owns output features 16 w ..
// 16 w + 15, the rows' activations pass from layer to layer in LDS, the residual stream
// stays in registers, and the weights stream from L2 into registers one group of k chunks
// ahead of their products, which needs no result of the chain.  Rows are independent, so
// nothing crosses workgroups, and one launch replaces a launch (or two) per layer.
//
// What bounds it: a few workgroups are bound by the layers' latency (a wave's products of a
// layer form one chain, and a barrier ends it), many in FP32 by the matrix cores (16 x 1.3 M
// products per 16 rows, 67 us at 157 TFLOP/s over 256 compute units).  Per workgroup the
// 1.3 M parameters of the paper's network pass through a compute unit's vector memory path
// once (5.2 MB, 35 us at 64 B per clock).  K = 10, W = 200, H = 3: 500 rows forward FP32
// 158 us, backward 101 us, 1024 rows BF16 88 and 42 us; loss and gradient of 500 rows
// 1482 us as one GEMM (9 to 13 us) or two and an epilogue per layer, 297 us so; a training
// step of 1024 rows 1364 and 248 us; 50000 rows' forward 2550 and 1853 us (the FP32 matrix
// cores busy for 48 % of it).
#include <algorithm>

#include "internal.h"

namespace ds {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(4))) f4u {  // 16 bytes at any float's address
    float v[4];
};

constexpr int kRows = 16;
constexpr int kGroup = 4;  // k chunks loaded together
// FP32 batches above this take 32 rows per workgroup, which halves the weights' traffic and
// gives a wave two chains of products (50000 rows: 2080 us with 16, 1873 us with 32); up to
// 16 rows on each of the 256 compute units, 32 would leave units idle.
constexpr int64_t kFewRows = 4096;

// A wave's T tiles of 16 rows: four features of one row each per lane.
template <int T> struct Acc {
    f4 v[T];
};

// One lane's share of a chunk: E inputs (16 bytes).  BF16: chunks of 32 inputs, lane 16 g + r
// holds inputs 8 g .. 8 g + 7 of row r.  FP32: chunks of 16 inputs, lane 16 g + r holds
// inputs 4 e + g, e = 0..3, so that step e of the 16x16x4 product adds inputs 4 e .. 4 e + 3
// and the whole sum runs over the inputs in order; LDS keeps a row's inputs in that order
// (place()), so both operands are 16-byte loads.
template <bool BF> struct Form {
    static constexpr int E = 8, CK = 32;
    typedef __bf16 lds_t;
};
template <> struct Form<false> {
    static constexpr int E = 4, CK = 16;
    typedef float lds_t;
};
template <bool BF> using Lds = typename Form<BF>::lds_t;

template <bool BF> __host__ __device__ constexpr int chunks(int n)
{
    return (n + Form<BF>::CK - 1) / Form<BF>::CK;
}

// Row pitch of an LDS operand of n inputs: whole chunks and 16 bytes of skew.
template <bool BF> __host__ __device__ constexpr int pitch(int n)
{
    return chunks<BF>(n) * Form<BF>::CK + Form<BF>::E;
}

// Where input k of a row stands in LDS.
template <bool BF> __device__ __forceinline__ int place(int k)
{
    return BF ? k : (k & ~15) + 4 * (k & 3) + ((k >> 2) & 3);
}

// Inputs of the first layer's matrix: BF16 adds the residual stream's product (operands in
// pairs) to the descriptor's; FP32 takes both in one sum, the descriptor first.
template <bool BF> __host__ __device__ constexpr int first_inputs(int W)
{
    return BF ? kStencil : kStencil + W;
}

// Packed weights: per matrix its fragments in the order the lanes load them, [feature tile]
// [chunk][hi, lo][lane] of 16 bytes, zero past the matrix; the lo parts (BF16 remainders)
// for the W-wide layers' forward products only.  First the K matrices V (FP32: V and W1
// side by side), then the W x W matrices W1 (blocks 2..K; BF16), W2 (blocks 1..K), the
// dense trailing layers and the scalar layer (one feature tile), then the W x W ones
// transposed (for the backward chain).
template <bool BF> struct Pack {
    const uint4 *base;
    int K, W, H, MT;
    __host__ __device__ Pack(const void *p, int k, int w, int h)
        : base(static_cast<const uint4 *>(p)), K(k), W(w), H(h), MT((w + 15) / 16) {}
    __host__ __device__ int nw() const { return 2 * K - 1 + H - 1; }
    __host__ __device__ int64_t sv() const
    {
        return (int64_t)MT * chunks<BF>(first_inputs<BF>(W)) * 64;
    }
    __host__ __device__ int64_t st() const { return (int64_t)MT * chunks<BF>(W) * 64; }
    __host__ __device__ int64_t sw() const { return st() * (BF ? 2 : 1); }
    __host__ __device__ const uint4 *V(int k) const { return base + k * sv(); }
    __host__ __device__ const uint4 *w(int i) const { return base + K * sv() + i * sw(); }
    __host__ __device__ const uint4 *last() const { return w(nw()); }
    __host__ __device__ const uint4 *t(int i) const { return last() + sw() / MT + i * st(); }
    // the index of a W x W matrix
    __host__ __device__ int W1(int k) const { return k - 1; }
    __host__ __device__ int W2(int k) const { return K - 1 + k; }
    __host__ __device__ int hw(int m) const { return 2 * K - 1 + m; }
    __host__ __device__ int64_t total() const
    {
        return K * sv() + nw() * (sw() + st()) + sw() / MT;
    }
};

// A group of chunks of this wave's feature tile in flight.
template <bool X3> struct Weights {
    uint4 v[kGroup][X3 ? 2 : 1];
};

// Loads chunks c0 .. of the tile whose fragments start at p (the same for the whole wave).
template <bool X3>
__device__ __forceinline__ void load(Weights<X3> &w, const uint4 *p, int c0, int nc)
{
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int c = 0; c < kGroup; ++c) {
        const int at = min(c0 + c, nc - 1);  // past the end: a chunk that is not used
        const uint4 *q = p + at * (X3 ? 128 : 64);
#pragma unroll
        for (int h = 0; h < (X3 ? 2 : 1); ++h)
            w.v[c][h] = (q + h * 64)[lane];
    }
}

// acc += the group's chunks times the activations x ([row][input] in LDS; X3: both operands
// as BF16 pairs hi + lo, the activations' remainders at x + lo: hi hi + lo hi + hi lo).
template <bool BF, bool X3, int T>
__device__ __forceinline__ void products(const Weights<X3> &w, const Lds<BF> *x, int ldx, int lo,
                                         int c0, int nc, Acc<T> &acc)
{
    constexpr int CK = Form<BF>::CK;
#pragma unroll
    for (int c = 0; c < kGroup; ++c) {
        if (c0 + c >= nc)
            break;
        const Lds<BF> *p = x + CK * (c0 + c);
        if constexpr (BF) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, w.v[c][0]);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                f4 &d = acc.v[t];
                const bf16x8 b = *reinterpret_cast<const bf16x8 *>(p + t * kRows * ldx);
                d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, d, 0, 0, 0);
                if constexpr (X3) {
                    const bf16x8 al = __builtin_bit_cast(bf16x8, w.v[c][1]);
                    const bf16x8 bl = *reinterpret_cast<const bf16x8 *>(p + t * kRows * ldx + lo);
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b, d, 0, 0, 0);
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, d, 0, 0, 0);
                }
            }
        } else {
            const f4 a = __builtin_bit_cast(f4, w.v[c][0]);
            f4 b[T];
#pragma unroll
            for (int t = 0; t < T; ++t)
                b[t] = *reinterpret_cast<const f4 *>(p + t * kRows * ldx);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < T; ++t)
                    acc.v[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[t][i], acc.v[t], 0, 0, 0);
        }
    }
}

// One matrix's products over n inputs.  Its first group is in `w` on entry (loaded while the
// chain was still busy with the layer before); each further group loads while the one
// before it is multiplied.  split: the sums of the first group and of the rest are formed
// apart and added (the order a small batch's sums have always had, so that a ReLU whose
// argument is a rounding error keeps its side).
template <bool BF, bool X3, int T>
__device__ __forceinline__ Acc<T> matrix(Weights<X3> &w, const uint4 *p, int n, const Lds<BF> *x,
                                         int ldx, int lo, bool split = false)
{
    const int nc = chunks<BF>(n);
    Acc<T> acc = {}, head = {};
#pragma unroll 1
    for (int c0 = 0; c0 < nc; c0 += 2 * kGroup) {
        Weights<X3> u;
        if (c0 + kGroup < nc)
            load(u, p, c0 + kGroup, nc);
        products<BF, X3>(w, x, ldx, lo, c0, nc, acc);
        if (BF && split && c0 == 0) {
            head = acc;
            acc = Acc<T>{};
        }
        if (c0 + kGroup < nc) {
            if (c0 + 2 * kGroup < nc)
                load(w, p, c0 + 2 * kGroup, nc);
            products<BF, X3>(u, x, ldx, lo, c0 + kGroup, nc, acc);
        }
    }
    if (BF && split)
#pragma unroll
        for (int t = 0; t < T; ++t)
            acc.v[t] = head.v[t] + acc.v[t];
    return acc;
}

// Four consecutive features of a row as LDS activations, inputs at + f .. (X3: with
// remainders).
template <bool BF, bool X3>
__device__ __forceinline__ void put(Lds<BF> *x, int lo, int ldx, int n, int at, int f, const f4 &v)
{
    if constexpr (BF) {
        Lds<BF> *p = x + n * ldx + at + f;
        bf16x4 h, l;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = (__bf16)v[i];
            if constexpr (X3)
                l[i] = (__bf16)(v[i] - (float)h[i]);
        }
        *reinterpret_cast<bf16x4 *>(p) = h;
        if constexpr (X3)
            *reinterpret_cast<bf16x4 *>(p + lo) = l;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            x[n * ldx + place<BF>(at + f + i)] = v[i];
    }
}

// Four features f .. f + 3 (those below W) at p[at ..]; p is the same for the whole wave.
__device__ __forceinline__ void store4(float *p, uint32_t at, int f, int W, const f4 &v)
{
    if (f + 4 <= W) {
        f4u q;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q.v[i] = v[i];
        *reinterpret_cast<f4u *>(p + at) = q;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (f + i < W)
                p[at + i] = v[i];
    }
}
__device__ __forceinline__ f4 load4(const float *p, uint32_t at, int f, int W)
{
    f4 v = {0.f, 0.f, 0.f, 0.f};
    if (f + 4 <= W) {
        const f4u q = *reinterpret_cast<const f4u *>(p + at);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[i] = q.v[i];
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (f + i < W)
                v[i] = p[at + i];
    }
    return v;
}
__device__ __forceinline__ void amax_note(unsigned *out, const f4 &v)
{
    float m = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0)
        atomicMax(out, __float_as_uint(m));
}

// Parameters of block k and of trailing layer m in the canonical vector.
struct Params {
    const float *th;
    int K, W;
    __host__ __device__ const float *V(int k) const
    {
        const int64_t w2 = (int64_t)W * W, b = 226 * (int64_t)W + w2 + 2 * W;
        return th + k * b + (k > 1 ? (k - 1) * w2 : 0);
    }
    __host__ __device__ const float *W1(int k) const { return V(k) + 226 * (int64_t)W; }
    __host__ __device__ const float *b1(int k) const { return W1(k) + (k > 0 ? (int64_t)W * W : 0); }
    __host__ __device__ const float *W2(int k) const { return b1(k) + W; }
    __host__ __device__ const float *b2(int k) const { return W2(k) + (int64_t)W * W; }
    __host__ __device__ const float *hw(int m) const
    {
        return V(K) + (int64_t)m * ((int64_t)W * W + W);
    }
};

// Packs every matrix (grid.y: K of V, then the W x W ones, then those transposed, then the
// scalar layer), a thread per 16 bytes of a fragment.
template <bool BF>
__device__ __forceinline__ void pack(const float *theta, int K, int W, int H, uint4 *out)
{
    constexpr int E = Form<BF>::E, CK = Form<BF>::CK;
    const Pack<BF> pk(out, K, W, H);
    const Params P{theta, K, W};
    const int id = blockIdx.y, nw = pk.nw();
    const bool isv = id < K, one = id == K + 2 * nw, tr = id >= K + nw && !one;
    const int wi = isv || one ? 0 : tr ? id - K - nw : id - K;
    const int n1 = isv ? kStencil : W;  // inputs from the matrix m; the others from W1
    const int n = isv && id > 0 ? first_inputs<BF>(W) : n1, ld = isv ? 226 : W;
    const int nc = chunks<BF>(isv ? first_inputs<BF>(W) : W);
    const float *m = isv ? P.V(id) : one ? P.hw(H - 1)
                   : wi < K - 1 ? P.W1(wi + 1) : wi < 2 * K - 1 ? P.W2(wi - K + 1)
                                                                : P.hw(wi - 2 * K + 1);
    const float *m2 = isv ? P.W1(id) : nullptr;
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= (int64_t)(one ? 1 : pk.MT) * nc * 64)
        return;
    const int lane = (int)(u & 63), c = (int)(u / 64 % nc), tile = (int)(u / 64 / nc);
    const int row = 16 * tile + (lane & 15), g = lane >> 4, rows = one ? 1 : W;
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = CK * c + (BF ? E * g + e : 4 * e + g);
        v[e] = 0.f;
        if (row < rows && k < n)
            v[e] = tr ? m[(int64_t)k * ld + row]
                      : k < n1 ? m[(int64_t)row * ld + k] : m2[(int64_t)row * W + k - n1];
    }
    if constexpr (BF) {
        bf16x8 h, l;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h[e] = (__bf16)v[e];
            l[e] = (__bf16)(v[e] - (float)h[e]);
        }
        if (isv || tr) {
            const_cast<uint4 *>(isv ? pk.V(id) : pk.t(wi))[u] = __builtin_bit_cast(uint4, h);
        } else {
            uint4 *p = const_cast<uint4 *>(one ? pk.last() : pk.w(wi)) + (u / 64 * 2) * 64 + lane;
            p[0] = __builtin_bit_cast(uint4, h);
            p[64] = __builtin_bit_cast(uint4, l);
        }
    } else {
        const_cast<uint4 *>(isv ? pk.V(id) : tr ? pk.t(wi) : one ? pk.last() : pk.w(wi))[u] =
            __builtin_bit_cast(uint4, f4{v[0], v[1], v[2], v[3]});
    }
}

// Both packed copies in one launch (grid.z, 13.2 us): apart they took 8.2 and 6.2 us and a
// launch more.
__global__ void __launch_bounds__(256) k_chain_pack(const float *theta, int K, int W, int H, uint4 *f32,
                                                    uint4 *bf16)
{
    if (blockIdx.z == 0)
        pack<false>(theta, K, W, H, f32);
    else
        pack<true>(theta, K, W, H, bf16);
}

template <bool BF>
__device__ __forceinline__ Weights<BF> &one_of(Weights<false> &a, Weights<BF> &b)
{
    if constexpr (BF)
        return b;
    else
        return a;
}

// Forward of T x 16 rows; the BF16 form takes the W-wide layers' operands as pairs (X3).
// FP32 with one tile of rows: 5 waves per SIMD are 96 registers, without a spill (7, two
// workgroups on a compute unit, spill 46 registers: 50000 rows 3105 us, 500 rows 204 us).  The
// BF16 form's 16 waves leave it 128 registers and spill 14 (18 below 13 waves' worth of
// descriptors at once); up to four waves have as many as they need.
// S: the number of waves, which decides how a level's descriptors are loaded (see z_load).
enum Waves { kUpTo4, kUpTo12, kFrom13 };
template <bool BF, int T, Waves S>
__global__ void __launch_bounds__(S == kUpTo4 ? 256 : 1024,
                                  S == kUpTo4 ? (BF ? 2 : 4) : !BF && T == 1 ? 5 : 4)
    k_chain_forward(ChainArgs a)
{
    typedef Lds<BF> X;
    constexpr int kR = T * kRows;  // rows of the workgroup
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int W = a.W, K = a.K, D = kStencil * K + 1;
    const int nf = first_inputs<BF>(W), ldz = pitch<BF>(nf), ldw = pitch<BF>(W), lo = kR * ldw;
    // the first layer's inputs (FP32: the descriptor level, then the residual stream), the
    // second's, and in BF16 the residual stream
    X *zb = reinterpret_cast<X *>(smem), *fb = zb + kR * ldz, *ob = fb + (BF ? 2 : 1) * lo;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int64_t b0 = (int64_t)blockIdx.x * kR;
    // per block gamma weights, b1, b2, then the trailing layers' biases, 16 to a tile: read
    // where a layer ends, when every wave waits for them (from L2 there: 1024 rows BF16
    // 109 us, from LDS 95 us)
    float *const vl = reinterpret_cast<float *>(ob + (BF ? 2 : 0) * lo);
    const int WP = nt / 4, nv = 3 * K + a.H - 1;
    bool in[T];  // this lane's rows n, n + 16, .. below M
#pragma unroll
    for (int t = 0; t < T; ++t)
        in[t] = n + t * kRows < a.M - b0;
    const int f0 = 16 * wave + 4 * g;  // the features this lane computes: f0 .. f0 + 3
    const Params P{a.theta, K, W};
    const Pack<BF> pk(a.pack, K, W, a.H);
    // this wave's tile of a matrix, this lane's place in an LDS operand
    const int tv = wave * chunks<BF>(nf) * 64;
    const int tw = wave * chunks<BF>(W) * (BF ? 2 : 1) * 64;
    const int xz = n * ldz + Form<BF>::E * g, xw = n * ldw + Form<BF>::E * g;
    const int ncw = chunks<BF>(W), ncz = chunks<BF>(nf);

    for (int e = tid; e < (kR * ldz + (BF ? 4 : 1) * lo) * (int)sizeof(X) / 16; e += nt)
        reinterpret_cast<uint4 *>(smem)[e] = uint4{0u, 0u, 0u, 0u};
    for (int e = tid; e < nv * WP; e += nt) {
        const int v = e / WP, f = e - v * WP, k = v / 3;
        float x = 0.f;
        if (f < W)
            x = v >= 3 * K ? P.hw(v - 3 * K)[(int64_t)W * W + f]
                : v - 3 * k == 0 ? P.V(k)[226 * f + 225] : (v - 3 * k == 1 ? P.b1(k) : P.b2(k))[f];
        vl[e] = x;
    }
    __syncthreads();
    // A level's descriptors: unit u holds columns 64 (u & 3) + lane of row u >> 2; a wave takes
    // every waves-th unit, kZ of them in flight at a time.  The first kZ are loaded a layer
    // ahead: all of them with 13 waves or more.  With fewer, a wave loads the others where it
    // stores them, and up to four waves take 16 at a time (one by one, each waiting for HBM, as
    // at first: 65536 rows of 6 x 32 FP32 689 us, of 5 a time 385 us, of 16 209 us; 1 x 16
    // 119, 69 and 48 us).
    constexpr int kZ = S == kUpTo4 ? 16 : 5 * T;
    const int waves = nt >> 6;
    X *const zl = zb + place<BF>(lane);
    float zr[kZ];
    // (past the last row, column or unit: the last one's, so that no load waits on a branch)
    auto z_at = [&](int u, int k, uint32_t at) {
        const int uu = min(u, 4 * kR - 1), c = 64 * (uu & 3);
        const int64_t r = min(b0 + (uu >> 2), a.M - 1);
        return (a.z + r * D + k * kStencil + c)[min(at, (uint32_t)(kStencil - 1 - c))];
    };
    auto z_put = [&](int u, float v) {
        if (u < 4 * kR && lane < kStencil - 64 * (u & 3))
            zl[(u >> 2) * ldz + 64 * (u & 3)] = (X)v;
    };
    auto z_load = [&](int k, uint32_t at, int u0) {
#pragma unroll
        for (int q = 0; q < kZ; ++q)
            zr[q] = z_at(u0 + q * waves, k, at);
    };
    auto z_puts = [&](int u0) {
#pragma unroll
        for (int q = 0; q < kZ; ++q)
            z_put(u0 + q * waves, zr[q]);
    };
    auto z_store = [&](int k) {
        z_puts(wave);
        if (S == kFrom13)
            return;
#pragma unroll 1
        for (int u0 = wave + kZ * waves; u0 < 4 * kR; u0 += kZ * waves) {
            z_load(k, lane, u0);
            z_puts(u0);
        }
    };
    z_load(0, lane, wave);
    z_store(0);
    float gamma[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
        gamma[t] = in[t] ? a.z[(b0 + n + t * kRows) * D + (int64_t)kStencil * K] : 0.f;
    // the first groups of a block's first matrix and of the matrices after it (FP32: one set
    // of registers)
    Weights<false> wv;
    Weights<BF> w2;
    Weights<BF> &w = one_of<BF>(wv, w2);
    load(wv, pk.V(0) + tv, 0, ncz);
    Acc<T> o = {};
    const f4 z4 = {0.f, 0.f, 0.f, 0.f};
    __syncthreads();

#pragma unroll 1
    for (int k = 0; k < K; ++k) {
        // lane offsets that the compiler may not form once for all blocks: kept over the
        // loop, the addresses take more registers than there are
        int f = f0, at = n * W + f0;
        uint32_t zl_at = lane;
        asm volatile("" : "+v"(f), "+v"(at), "+v"(zl_at));
        if (BF)
            load(w, pk.w(k > 0 ? pk.W1(k) : pk.W2(k)) + tw, 0, ncw);
        // FP32: block 1 has no residual stream, its sum ends with the descriptor
        Acc<T> v = matrix<BF, false, T>(wv, pk.V(k) + tv, BF || k == 0 ? kStencil : nf, zb + xz, ldz,
                                        0, a.split_v);
        if (BF && k > 0) {
            const Acc<T> r =
                matrix<BF, BF, T>(w, pk.w(pk.W1(k)) + tw, W, ob + xw, ldw, lo, a.split_w);
#pragma unroll
            for (int t = 0; t < T; ++t)
                v.v[t] = v.v[t] + r.v[t];
        }
        if (!BF || k > 0)
            load(w, pk.w(pk.W2(k)) + tw, 0, ncw);
        if (k + 1 < K)
            z_load(k + 1, zl_at, wave);
        // first layer of the block: the gamma input, bias, ReLU
        {
            const f4 gw = *reinterpret_cast<const f4 *>(vl + 3 * k * WP + f);
            const f4 bias = *reinterpret_cast<const f4 *>(vl + (3 * k + 1) * WP + f);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const float p = fmaf(gamma[t], gw[i], v.v[t][i]) + bias[i];
                    v.v[t][i] = f + i < W ? fmaxf(p, 0.f) : 0.f;
                }
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            put<BF, BF>(fb, lo, ldw, n + t * kRows, 0, f, v.v[t]);
            if (a.F1 && in[t])
                store4(a.F1 + ((int64_t)k * a.M + b0) * W, at + t * kRows * W, f, W, v.v[t]);
            if (a.amax)
                amax_note(a.amax + k, in[t] ? v.v[t] : z4);
        }
        __syncthreads();
        // second layer: bias, residual, ReLU
        v = matrix<BF, BF, T>(w, pk.w(pk.W2(k)) + tw, W, fb + xw, ldw, lo, a.split_w);
        if (k + 1 < K) {
            z_store(k + 1);
            load(wv, pk.V(k + 1) + tv, 0, ncz);
        }
        const f4 bias = *reinterpret_cast<const f4 *>(vl + (3 * k + 2) * WP + f);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            f4 &y = o.v[t];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = (v.v[t][i] + bias[i]) + y[i];
                y[i] = f + i < W ? fmaxf(p, 0.f) : 0.f;
            }
            if (BF)
                put<BF, BF>(ob, lo, ldw, n + t * kRows, 0, f, y);
            else if (f < W)  // past the last feature lies nothing to overwrite but padding
                put<BF, BF>(zb, 0, ldz, n + t * kRows, kStencil, f, y);
            if (a.O && in[t])
                store4(a.O + ((int64_t)k * a.M + b0) * W, at + t * kRows * W, f, W, y);
            if (a.amax)
                amax_note(a.amax + K, in[t] ? y : z4);
        }
        __syncthreads();
    }
    // trailing layers, alternating between two activation buffers; the last one is scalar
    // (the first wave's first feature)
    X *src = BF ? ob : zb, *dst = fb;
    const int f = f0, at = n * W + f0;
    if (!BF) {  // the residual stream again, as a layer's inputs
#pragma unroll
        for (int t = 0; t < T; ++t)
            put<BF, BF>(src, 0, ldw, n + t * kRows, 0, f, o.v[t]);
        __syncthreads();
    }
#pragma unroll 1
    for (int m = 0; m < a.H; ++m) {
        const bool last = m + 1 == a.H;
        if (last && wave > 0)
            return;
        const uint4 *p = last ? pk.last() : pk.w(pk.hw(m)) + tw;
        load(w, p, 0, ncw);
        const Acc<T> v = matrix<BF, BF, T>(w, p, W, src + xw, ldw, lo, last ? a.split_l : a.split_w);
        const float *hb = P.hw(m) + (int64_t)(last ? 1 : W) * W;
        if (last) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (g != 0 || !in[t])
                    continue;
                const int64_t row = b0 + n + t * kRows;
                const float pre = v.v[t][0] + hb[0], out = fmaxf(pre, 0.f);
                if (a.out)
                    a.out[row] = out;
                if (a.pre)
                    a.pre[row] = pre;
                if (a.target) {  // loss on log(1 + g) and its derivative (Sec. 5.2)
                    const float r = log1pf(out) - a.target[row];
                    a.sq[row] = r * r;
                    a.dpre[row] = pre > 0.f ? 2.f * r / ((float)a.M * (1.f + out)) : 0.f;
                }
            }
            return;
        }
        const f4 bias = *reinterpret_cast<const f4 *>(vl + (3 * K + m) * WP + f);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            f4 &y = o.v[t];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float q = v.v[t][i] + bias[i];
                y[i] = f + i < W ? fmaxf(q, 0.f) : 0.f;
            }
            put<BF, BF>(dst, lo, ldw, n + t * kRows, 0, f, y);
            if (a.HO && in[t])
                store4(a.HO + ((int64_t)m * a.M + b0) * W, at + t * kRows * W, f, W, y);
            if (a.amax)
                amax_note(a.amax + K + 1 + m, in[t] ? y : z4);
        }
        __syncthreads();
        X *const t = src;
        src = dst;
        dst = t;
    }
}

// Backward chain: the gradients of every layer's pre-activations, from dpre down to block 1.
template <bool BF>
__global__ void __launch_bounds__(1024) k_chain_backward(ChainArgs a)
{
    typedef Lds<BF> T;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int W = a.W, K = a.K;
    const int ldw = pitch<BF>(W), sz = kRows * ldw;
    T *x0 = reinterpret_cast<T *>(smem), *x1 = x0 + sz;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int64_t b0 = (int64_t)blockIdx.x * kRows, row = b0 + n;
    const bool in = row < a.M;
    const int f = 16 * wave + 4 * g;
    const uint32_t at = n * W + f, read_at = (in ? n : 0) * W + f;  // rows past the last: the first
    const Params P{a.theta, K, W};
    const Pack<BF> pk(a.pack, K, W, a.H);
    const int ncw = chunks<BF>(W), xw = n * ldw + Form<BF>::E * g;
    const int tw = wave * ncw * 64;
    for (int e = tid; e < 2 * sz; e += nt)
        x0[e] = (T)0.f;
    Weights<false> w;
    load(w, pk.t(a.H > 1 ? pk.hw(a.H - 2) : pk.W2(K - 1)) + tw, 0, ncw);
    // gradient of the scalar layer's input (operands rounded once, as in every product)
    f4 d;
    {
        const float dp = in ? a.dpre[row] : 0.f;
        const f4 wl = load4(P.hw(a.H - 1), f, f, W);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            d[i] = BF ? (float)(__bf16)dp * (float)(__bf16)wl[i] : dp * wl[i];
    }
    // d := d where the activation is positive, kept for the weight gradients and as operand
    auto mask = [&](const float *act, float *keep, T *x) {
        const f4 y = load4(act + b0 * W, read_at, f, W);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            d[i] = y[i] > 0.f ? d[i] : 0.f;
        if (in)
            store4(keep + b0 * W, at, f, W, d);
        put<BF, false>(x, 0, ldw, n, 0, f, d);
    };
    __syncthreads();
    const int64_t MW = a.M * W;
#pragma unroll 1
    for (int m = a.H - 2; m >= 0; --m) {
        T *x = (m & 1) ? x1 : x0;
        mask(a.HO + m * MW, a.DY + m * MW, x);
        __syncthreads();
        d = matrix<BF, false, 1>(w, pk.t(pk.hw(m)) + tw, W, x + xw, ldw, 0).v[0];
        load(w, pk.t(m > 0 ? pk.hw(m - 1) : pk.W2(K - 1)) + tw, 0, ncw);
    }
    __syncthreads();
#pragma unroll 1
    for (int k = K - 1;; --k) {
        mask(a.O + k * MW, a.DA + k * MW, x0);
        const f4 da = d;
        __syncthreads();
        d = matrix<BF, false, 1>(w, pk.t(pk.W2(k)) + tw, W, x0 + xw, ldw, 0).v[0];
        if (k > 0)
            load(w, pk.t(pk.W1(k)) + tw, 0, ncw);
        mask(a.F1 + k * MW, a.DH + k * MW, x1);
        if (k == 0)
            break;
        __syncthreads();
        d = da + matrix<BF, false, 1>(w, pk.t(pk.W1(k)) + tw, W, x1 + xw, ldw, 0).v[0];
        load(w, pk.t(pk.W2(k - 1)) + tw, 0, ncw);
    }
}

template <bool BF> size_t forward_lds(int K, int W, int H, int rows)
{
    return rows * (pitch<BF>(first_inputs<BF>(W)) + (BF ? 4 : 1) * pitch<BF>(W)) *
               sizeof(Lds<BF>) +
           (size_t)(3 * K + H - 1) * ((W + 15) / 16 * 16) * sizeof(float);
}

}  // namespace

size_t chain_pack_bytes(int K, int W, int H, bool bf16)
{
    return sizeof(uint4) * (size_t)(bf16 ? Pack<true>(nullptr, K, W, H).total()
                                         : Pack<false>(nullptr, K, W, H).total());
}

ds_status chain_pack(hipStream_t s, const ds_net *net)
{
    const Pack<false> pk(net->chain, net->K, net->W, net->H);  // FP32: the most fragments
    const int64_t n = (int64_t)pk.MT * chunks<false>(first_inputs<false>(net->W)) * 64;
    k_chain_pack<<<dim3((unsigned)((n + 255) / 256), (unsigned)(net->K + 2 * pk.nw() + 1), 2), 256, 0, s>>>(
        net->theta, net->K, net->W, net->H, static_cast<uint4 *>(net->chain),
        static_cast<uint4 *>(net->chain16));
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status chain_forward(hipStream_t s, const ChainArgs &args, bool bf16)
{
    ChainArgs a = args;
    if (a.M <= 0)
        return DS_OK;
    // Small batches form their BF16 sums over more than 128 inputs in two parts, the first 128
    // inputs and the rest: batches of at most 1808 rows whose W-wide outputs make fewer than 64
    // tiles of 64 x 64 (W = 200: 960 rows, W <= 64: 1808), for the scalar layer up to 4032 rows.
    // One sum would do as well, but the two round apart, and a ReLU whose argument is a rounding
    // error then changes sides: the lines lie where they have always been, so that a training
    // run repeats.
    const int64_t rows = (a.M + 63) / 64, cols = (a.W + 63) / 64;
    a.split_v = rows * cols < 64 && a.M <= 1808;
    a.split_w = a.split_v && a.W > 128;
    a.split_l = rows < 64 && a.W > 128;
    const unsigned blocks = (unsigned)((a.M + kRows - 1) / kRows), threads = 64 * ((a.W + 15) / 16);
    // Up to four waves take 16 rows however many there are: a second tile lengthens each wave's
    // loads (65536 rows of 6 x 32 209 us with one, 323 with two; of 6 x 64 271 and 271).
    const Waves S = threads <= 256 ? kUpTo4 : threads <= 768 ? kUpTo12 : kFrom13;
    const int tiles = !bf16 && S != kUpTo4 && a.M > kFewRows ? 2 : 1;
    const auto k =
        S == kUpTo4    ? (bf16 ? k_chain_forward<true, 1, kUpTo4> : k_chain_forward<false, 1, kUpTo4>)
        : S == kUpTo12 ? (bf16         ? k_chain_forward<true, 1, kUpTo12>
                          : tiles == 1 ? k_chain_forward<false, 1, kUpTo12>
                                       : k_chain_forward<false, 2, kUpTo12>)
                       : (bf16         ? k_chain_forward<true, 1, kFrom13>
                          : tiles == 1 ? k_chain_forward<false, 1, kFrom13>
                                       : k_chain_forward<false, 2, kFrom13>);
    k<<<(blocks + tiles - 1) / tiles, threads,
        bf16 ? forward_lds<true>(a.K, a.W, a.H, kRows) : forward_lds<false>(a.K, a.W, a.H, tiles * kRows),
        s>>>(a);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

ds_status chain_backward(hipStream_t s, const ChainArgs &a, bool bf16)
{
    const unsigned blocks = (unsigned)((a.M + kRows - 1) / kRows), threads = 64 * ((a.W + 15) / 16);
    if (bf16)
        k_chain_backward<true>
            <<<blocks, threads, 2 * kRows * pitch<true>(a.W) * sizeof(__bf16), s>>>(a);
    else
        k_chain_backward<false>
            <<<blocks, threads, 2 * kRows * pitch<false>(a.W) * sizeof(float), s>>>(a);
    DS_HIP(hipGetLastError());
    return DS_OK;
}

}  // namespace ds
