// Learned heuristic (a project addition beside the paper's eta = 1/d of
// Sec. 2.1): k-nearest-neighbour edge features, a 8 -> 128 -> 128 -> 1 GELU
// edge-scoring MLP in bfloat16 on MFMA with FP32 accumulation (inference,
// and training by binary cross-entropy with logits and Adam), and the
// installation eta_ij = (1/d_ij) * 2 sigmoid(s_ij) on the 16 nearest cities
// of i; the other edges of i take the multiplier of i's lowest score, so
// s = 0 gives the plain heuristic exactly.
//
// MFMA: v_mfma_f32_16x16x16_bf16 and v_mfma_f32_16x16x32_bf16. With lane l,
// row block q = l / 16 and column c = l % 16: the A operand of lane l is
// A[c][4q .. 4q+3] (row c, four consecutive k; eight with the longer form), the
// B operand is B[4q .. 4q+3][c] (column c), and the result holds D[4q + t][c],
// t = 0..3. Which k a lane's elements stand for is free as long as A and B
// agree.
#include <cmath>
#include <cstddef>
#include <mutex>

#include "device.hpp"
#include "internal.hpp"

namespace mmas {
namespace {

constexpr int kHid = 128;
constexpr int kIn = 16;
constexpr int kK = 16;  // nearest neighbours per city

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// nearest bfloat16, ties to even (finite inputs)
__device__ __forceinline__ uint16_t to_bf16(float x) {
    uint32_t b = __float_as_uint(x);
    b = b + 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// exp in FP32: clamp to [-104, 89], k = rint(x log2 e), r = x - k ln2 (ln2 as
// a 15-bit head and a rounded tail), exp(r) by its Taylor series through r^8,
// times 2^k.
__device__ __forceinline__ float exp_f32(float x) {
    const float kLog2e = __uint_as_float(0x3FB8AA3Bu);
    const float kLn2Hi = __uint_as_float(0x3F317200u);
    const float kLn2Lo = __uint_as_float(0x35BFBE8Eu);
    x = x > 89.0f ? 89.0f : x;
    x = x < -104.0f ? -104.0f : x;
    const float kf = __builtin_rintf(x * kLog2e);
    const float r = (x - kf * kLn2Hi) - kf * kLn2Lo;
    float p = 1.0f / 40320.0f;
    p = 1.0f / 5040.0f + r * p;
    p = 1.0f / 720.0f + r * p;
    p = 1.0f / 120.0f + r * p;
    p = 1.0f / 24.0f + r * p;
    p = 1.0f / 6.0f + r * p;
    p = 0.5f + r * p;
    p = 1.0f + r * p;
    p = 1.0f + r * p;
    return ldexpf(p, (int)kf);
}

__device__ __forceinline__ float sigmoid_f32(float s) { return 1.0f / (1.0f + exp_f32(-s)); }

// GELU(z) = z Phi(z). With t = 1 / (1 + 0.4 |z| / sqrt 2) and E = exp(-z^2/2),
// 1 - Phi(|z|) = h = E (c1 t + .. + c6 t^6) / 2, a form of Abramowitz and
// Stegun 7.1.26 with a degree-6 fit made for this project (reweighted least
// squares of z times the error: 1.5e-8 over the range), E and t by
// v_exp_f32 and v_rcp_f32. 13 instructions and the two transcendentals (the
// derivative 5 more), where the degree-5 form with an IEEE division and a
// Taylor exponential took about 65; against 64 bits over [-8, 8] GELU is off by at most 2.4e-7 and its
// derivative by 2.5e-7 (4.7e-7 and 3.0e-7 before).
struct Normal {
    float h, e;  // 1 - Phi(|z|), exp(-z^2/2)
};
__device__ __forceinline__ Normal normal_tail(float z) {
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.28284271247f, __builtin_fabsf(z), 1.0f));
    const float e = __builtin_amdgcn_exp2f(z * z * -0.72134752044f);
    float p = -0.10188215f;
    p = __builtin_fmaf(p, t, 0.36180096f);
    p = __builtin_fmaf(p, t, -0.19729585f);
    p = __builtin_fmaf(p, t, 0.243770515f);
    p = __builtin_fmaf(p, t, 0.077021965f);
    p = __builtin_fmaf(p, t, 0.116584545f);
    return Normal{p * t * e, e};
}
// (h is 0 long before z = 64: the bound keeps infinity times 0 out of the sum)
__device__ __forceinline__ float gelu_of(float z, const Normal& n) {
    const float u = __builtin_amdgcn_fmed3f(z, -__builtin_inff(), 64.0f);
    return __builtin_fmaf(-__builtin_fabsf(u), n.h, z > 0.0f ? z : 0.0f);
}
// the derivative Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_d_of(float z, const Normal& n) {
    return __builtin_fmaf(z * 0.39894228040f, n.e, 0.5f + __builtin_copysignf(0.5f - n.h, z));
}

// ---- features ----------------------------------------------------------------

// one thread per edge e = 16 i + r: the mean distance of i's neighbours, summed
// left to right by every lane of the row of 16 that holds them, and the
// in-degrees
__global__ __launch_bounds__(256) void k_feat_city(const int32_t* __restrict__ dist, const uint16_t* __restrict__ knn,
                                                   int n, float* __restrict__ dbar, int* __restrict__ indeg) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool in = e < n * kK;
    const int i = in ? e / kK : 0, j = in ? knn[e] : 0;
    const float v = (float)dist[(size_t)i * n + j];
    float s = 0.0f;
    for (int r = 0; r < kK; ++r) s = s + __shfl(v, (lane & 48) + r);
    if (!in) return;
    if (e % kK == 0) dbar[i] = s / 16.0f;
    atomicAdd(&indeg[j], 1);
}

// one thread per directed edge e = 16 i + r; FP32 features in the order of
// operations the oracle uses, then the bfloat16 MLP input row (8 features,
// 8 zeros)
__global__ __launch_bounds__(256) void k_feat_edge(const int32_t* __restrict__ dist, const float* __restrict__ xy,
                                                   const uint16_t* __restrict__ knn, const float* __restrict__ dbar,
                                                   const int* __restrict__ indeg, int n, float* __restrict__ feat,
                                                   uint16_t* __restrict__ X) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * kK) return;
    const int i = e / kK, r = e % kK;
    const int j = knn[e];
    int back = 16;
    for (int t = 0; t < kK; ++t)
        if (knn[j * kK + t] == i) {
            back = t;
            break;
        }
    float f[8];
    f[0] = (float)dist[(size_t)i * n + j] / dbar[i];
    f[1] = (float)r / 15.0f;
    f[2] = (float)back / 16.0f;
    f[3] = (xy[2 * j] - xy[2 * i]) / dbar[i];
    f[4] = (xy[2 * j + 1] - xy[2 * i + 1]) / dbar[i];
    f[5] = (float)indeg[j] / 16.0f;
    f[6] = (float)indeg[i] / 16.0f;
    f[7] = dbar[j] / dbar[i];
    for (int c = 0; c < 8; ++c) {
        if (feat) feat[(size_t)e * 8 + c] = f[c];
        X[(size_t)e * kIn + c] = to_bf16(f[c]);
        X[(size_t)e * kIn + 8 + c] = 0;
    }
}

// ---- parameters ------------------------------------------------------------------
// FP32 master layout: W1 [16][128] | b1 [128] | W2 [128][128] | b2 [128] | w3 [128] | b3

constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kIn * kHid;
constexpr int kOffW2 = kOffB1 + kHid;
constexpr int kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid;
constexpr int kOffB3 = kOffW3 + kHid;
constexpr int kParams = kOffB3 + 1;

// bfloat16 working copies: W1t [128 out][16 in], W2t [128 out][128 in],
// W2n [128 in][128 out], w3 [128]
constexpr int kPkW1t = 0;
constexpr int kPkW2t = kPkW1t + kHid * kIn;
constexpr int kPkW2n = kPkW2t + kHid * kHid;
constexpr int kPkW3 = kPkW2n + kHid * kHid;
constexpr int kPacked = kPkW3 + kHid;

__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ p, uint16_t* __restrict__ pk) {
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < kHid * kHid; t += gridDim.x * blockDim.x) {
        const int a = t / kHid, b = t % kHid;          // W2[a][b], a = in, b = out
        pk[kPkW2n + a * kHid + b] = to_bf16(p[kOffW2 + a * kHid + b]);
        pk[kPkW2t + b * kHid + a] = to_bf16(p[kOffW2 + a * kHid + b]);
        if (t < kIn * kHid) {
            const int k = t / kHid, c = t % kHid;      // W1[k][c]
            pk[kPkW1t + c * kIn + k] = to_bf16(p[kOffW1 + k * kHid + c]);
        }
        if (t < kHid) pk[kPkW3 + t] = to_bf16(p[kOffW3 + t]);
    }
}

// ---- forward / backward ---------------------------------------------------
//
// A wave takes 16 edges, one per column of its MFMAs: every product is formed
// transposed, Z^T = W^T H^T, with the weights as the A operand. A lane then
// holds units 16a + 4q + t of edge c, and what it holds of two unit tiles
// (16a + 4q .. and 16a + 16 + 4q ..), rounded to bfloat16, is the B operand of
// the next layer's product over these 32 units, without an exchange between
// lanes; the weights lie in LDS in the same order of k, one 16-byte piece per
// lane, tile and 32 units ("fragments"), so that a read is without bank
// conflicts.

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kTiles = kHid / 16;                // unit tiles of a layer
constexpr int kFrags = kTiles * (kHid / 32);     // fragments of a 128 x 128 weight matrix
constexpr int kMlpThreads = 512;
constexpr int kMlpEdges = kMlpThreads / kWave * 16;  // edges of a workgroup at a time

// four values as bfloat16 (to nearest, ties to even: v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
    const bf2 lo = __builtin_convertvector(f32x2{a, b}, bf2), hi = __builtin_convertvector(f32x2{c, d}, bf2);
    return make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
}
__device__ __forceinline__ f32x4 mfma32(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(uint2 a, uint2 b, f32x4 c) {
    return mfma16(__builtin_bit_cast(bf16x4, a), __builtin_bit_cast(bf16x4, b), c);
}
// four values at p, which need not be aligned to more than one of them
__device__ __forceinline__ uint2 load4(const uint16_t* p) {
    uint2 v;
    __builtin_memcpy(&v, p, sizeof(v));
    return v;
}
__device__ __forceinline__ uint4 join(uint2 a, uint2 b) { return make_uint4(a.x, a.y, b.x, b.y); }

// Fragments of the row-major 128 x 128 matrix m (row = unit of the result):
// piece (tile a, chunk kt, lane) holds row 16a + c, columns 32kt + 4q .. + 3
// and 32kt + 16 + 4q .. + 3.
__device__ __forceinline__ void load_frags(uint4* frag, const uint16_t* __restrict__ m) {
#pragma unroll
    for (int e = threadIdx.x; e < kFrags * kWave; e += kMlpThreads) {
        const int f = e >> 6, l = e & 63;
        const uint16_t* row = m + (16 * (f >> 2) + (l & 15)) * kHid + 32 * (f & 3) + 4 * (l >> 4);
        frag[e] = join(load4(row), load4(row + 16));
    }
}

struct ForwardSmem {
    uint4 w2t[kFrags * kWave];
    uint2 w1[kTiles * kWave];  // piece (tile a, lane): unit 16a + c, inputs 4q .. + 3
    float b1[kHid], b2[kHid], w3[kHid];
};
__device__ __forceinline__ void load_forward(ForwardSmem& sm, const float* __restrict__ p,
                                             const uint16_t* __restrict__ pk) {
    load_frags(sm.w2t, pk + kPkW2t);
    for (int e = threadIdx.x; e < kTiles * kWave; e += kMlpThreads)
        sm.w1[e] = load4(pk + kPkW1t + (16 * (e >> 6) + (e & 15)) * kIn + 4 * ((e >> 4) & 3));
    for (int t = threadIdx.x; t < kHid; t += kMlpThreads) {
        sm.b1[t] = p[kOffB1 + t];
        sm.b2[t] = p[kOffB2 + t];
        sm.w3[t] = from_bf16(pk[kPkW3 + t]);
    }
}
__device__ __forceinline__ f32x4 lds4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// Forward of the 16 edges whose inputs 4q .. + 3 (edge c) are x: the scores
// without b3, edge c's in every lane of column c. keep_h1(a, h) gets tile a of
// H1 as it is made; kTrain: the derivatives d2 of the second layer's GELUs and
// h2 (rounded).
template <bool kTrain, class Keep>
__device__ __forceinline__ float forward16(const ForwardSmem& sm, uint2 x, int q, int lane, Keep&& keep_h1,
                                           float d2[kTiles][4], uint2 h2[kTiles]) {
    uint2 h[kTiles];
    uint4 h1[kTiles / 2];
#pragma unroll
    for (int a = 0; a < kTiles; ++a) {
        const f32x4 z = mfma16(sm.w1[a * kWave + lane], x, lds4(&sm.b1[16 * a + 4 * q]));
        float g[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            g[t] = gelu_of(z[t], normal_tail(z[t]));
        }
        h[a] = pack4(g[0], g[1], g[2], g[3]);
        keep_h1(a, h[a]);
        if (kTrain || (a & 1)) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int kt = 0; kt < kTiles / 2; ++kt) h1[kt] = join(h[2 * kt], h[2 * kt + 1]);
    float s = 0.0f;
#pragma unroll
    for (int a = 0; a < kTiles; ++a) {
        f32x4 z = lds4(&sm.b2[16 * a + 4 * q]);
#pragma unroll
        for (int kt = 0; kt < kTiles / 2; ++kt) z = mfma32(sm.w2t[(4 * a + kt) * kWave + lane], h1[kt], z);
        float g[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const Normal nt = normal_tail(z[t]);
            g[t] = gelu_of(z[t], nt);
            if (kTrain) d2[a][t] = gelu_d_of(z[t], nt);
        }
        const uint2 r = pack4(g[0], g[1], g[2], g[3]);
        if (kTrain) h2[a] = r;
        const f32x4 w3 = lds4(&sm.w3[16 * a + 4 * q]);
        s = __builtin_fmaf(__uint_as_float(r.x << 16), w3[0], s);
        s = __builtin_fmaf(__uint_as_float(r.x & 0xFFFF0000u), w3[1], s);
        s = __builtin_fmaf(__uint_as_float(r.y << 16), w3[2], s);
        s = __builtin_fmaf(__uint_as_float(r.y & 0xFFFF0000u), w3[3], s);
        // (a tile's weights are read in its turn: read ahead, they would spill)
        if (kTrain || (a & 1)) __builtin_amdgcn_sched_barrier(0);
    }
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    return s;
}

// Bound by the GELUs' vector instructions (64 a lane and 16 edges); eight
// waves a workgroup share the weights' fragments. 60720 edges: 80 -> 16 us
// (activations through LDS rows of 256 bytes, whose reads met in one bank, and
// GELUs of 65 instructions).
__global__ __launch_bounds__(kMlpThreads) void k_mlp_forward(const uint16_t* __restrict__ X,
                                                             const float* __restrict__ p,
                                                             const uint16_t* __restrict__ pk, int64_t E,
                                                             float* __restrict__ s_out) {
    __shared__ ForwardSmem sm;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4, c = lane & 15;
    load_forward(sm, p, pk);
    const float b3 = p[kOffB3];
    __syncthreads();
    for (int64_t e0 = (int64_t)blockIdx.x * kMlpEdges + 16 * wave; e0 < E; e0 += (int64_t)gridDim.x * kMlpEdges) {
        const int64_t e = e0 + c;
        uint2 x = make_uint2(0u, 0u);
        if (e < E) x = load4(X + e * kIn + 4 * q);
        const float s = forward16<false>(sm, x, q, lane, [](int, uint2) {}, nullptr, nullptr) + b3;
        if (q == 0 && e < E) s_out[e] = s;
    }
}

// The training kernel's LDS: both orders of W2 as fragments, and what the
// waves exchange for the weight gradients (below); the column sums at the end
// reuse the exchange.
struct TrainSmem {
    ForwardSmem f;
    uint4 w2n[kFrags * kWave];
    uint4 ex[2][kFrags * kWave];
};

// A 16 x 16 tile held as the B operand of the products above (units 4q .. + 3
// of edge c) turned into units' rows (edges 4q .. + 3 of unit c): as the A
// operand it is the tile's transpose, and the identity as the other operand
// leaves it in the result's order. Exact (one product with 1 per element).
__device__ __forceinline__ uint2 transpose(uint2 v, uint2 identity) {
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const f32x4 d = mfma16(v, identity, zero);
    return pack4(d[0], d[1], d[2], d[3]);
}

// Fused forward and backward over tiles of 128 edges, 16 a wave; each
// workgroup keeps its gradient sums in registers and writes them once to
// partial[blockIdx.x] (kParams floats) plus its loss sum to
// partial[gridDim.x * kParams + b].
// The weight gradients sum over edges, so the waves turn their tiles of H1,
// dZ2, dZ1 and X (an MFMA with the identity each) and exchange them through
// LDS; wave w then owns output columns 16w .. + 15: 64 products for dW2, 4 for
// dW1, and the column sums for the biases with a row of ones. Each GELU of
// the second layer and its derivative come from one evaluation. Bound by the
// chains of vector instructions (2600 per wave and 16 edges) at two waves a
// SIMD, which the LDS leaves: one every 7 clocks of a SIMD. 65536 edges, 256 workgroups: 209 -> 41 us (operands
// gathered from LDS two bytes at a time, three GELU evaluations per unit).
__global__ __launch_bounds__(kMlpThreads) void k_mlp_train(const uint16_t* __restrict__ X, const float* __restrict__ f,
                                                           const float* __restrict__ p,
                                                           const uint16_t* __restrict__ pk, int64_t E,
                                                           float* __restrict__ partial) {
    extern __shared__ __align__(16) uint8_t raw[];
    TrainSmem& sm = *reinterpret_cast<TrainSmem*>(raw);
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    load_forward(sm.f, p, pk);
    load_frags(sm.w2n, pk + kPkW2n);
    const float b3 = p[kOffB3];
    const float invE = 1.0f / (float)E;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr uint32_t kOne = 0x3F80u;
    const uint4 ones = make_uint4(kOne * 0x10001u, kOne * 0x10001u, kOne * 0x10001u, kOne * 0x10001u);
    const uint2 identity = make_uint2((4 * q == c ? kOne : 0u) | (4 * q + 1 == c ? kOne << 16 : 0u),
                                      (4 * q + 2 == c ? kOne : 0u) | (4 * q + 3 == c ? kOne << 16 : 0u));
    // this lane's place for its own tile a of the exchange: pair of waves,
    // tile, lane, half of the 16 bytes
    uint2* const put0 = reinterpret_cast<uint2*>(sm.ex[0]) + ((wave >> 1) * kTiles * kWave + lane) * 2 + (wave & 1);
    uint2* const put1 = reinterpret_cast<uint2*>(sm.ex[1]) + ((wave >> 1) * kTiles * kWave + lane) * 2 + (wave & 1);
    f32x4 gw2[kTiles], gw1 = zero, gb2 = zero, gb1 = zero;
    float gw3[kTiles], gb3 = 0.0f, loss = 0.0f;  // gw3: unit 16a + c over edges 4q .. + 3
#pragma unroll
    for (int a = 0; a < kTiles; ++a) {
        gw2[a] = zero;
        gw3[a] = 0.0f;
    }
    __syncthreads();
    const int64_t tiles = (E + kMlpEdges - 1) / kMlpEdges;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t e = tile * kMlpEdges + 16 * wave + c;
        const bool in = e < E;
        uint2 x = make_uint2(0u, 0u);
        if (in) x = load4(X + e * kIn + 4 * q);
        const float fe = in ? f[e] : 0.0f;
        float d2[kTiles][4];
        uint2 h2[kTiles];
        const float s = forward16<true>(sm.f, x, q, lane,
                                        [&](int a, uint2 h) { put0[a * kWave * 2] = transpose(h, identity); }, d2, h2) + b3;
        // dL/ds of edge c (zero past E)
        float g = 0.0f;
        if (in) {
            g = (sigmoid_f32(s) - fe) * invE;
            if (q == 0) {
                const float sp = s > 0.0f ? s + log1pf(exp_f32(-s)) : log1pf(exp_f32(s));
                loss += sp - fe * s;
                gb3 += g;
            }
        }
        float gt[4];  // g of edges 4q .. + 3
#pragma unroll
        for (int t = 0; t < 4; ++t) gt[t] = __shfl(g, 4 * q + t);
        uint4 z2[kTiles / 2];  // dZ2, fragments by 32 units
        {
            uint2 dz[kTiles];
#pragma unroll
            for (int a = 0; a < kTiles; ++a) {
                const f32x4 w3 = lds4(&sm.f.w3[16 * a + 4 * q]);
                const f32x4 ht = mfma16(h2[a], identity, zero);  // (transposed, as below)
#pragma unroll
                for (int t = 0; t < 4; ++t) gw3[a] = __builtin_fmaf(ht[t], gt[t], gw3[a]);
                dz[a] = pack4(g * w3[0] * d2[a][0], g * w3[1] * d2[a][1], g * w3[2] * d2[a][2], g * w3[3] * d2[a][3]);
                put1[a * kWave * 2] = transpose(dz[a], identity);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int kt = 0; kt < kTiles / 2; ++kt) z2[kt] = join(dz[2 * kt], dz[2 * kt + 1]);
        }
        // dH1^T = W2 dZ2^T, then dZ1 (kept until the exchange is free); the first
        // layer's pre-activations are formed again, which costs less than the
        // registers they would hold since the forward
        uint2 z1[kTiles];
#pragma unroll
        for (int a = 0; a < kTiles; ++a) {
            f32x4 d = zero;
#pragma unroll
            for (int kt = 0; kt < kTiles / 2; ++kt) d = mfma32(sm.w2n[(4 * a + kt) * kWave + lane], z2[kt], d);
            const f32x4 z = mfma16(sm.f.w1[a * kWave + lane], x, lds4(&sm.f.b1[16 * a + 4 * q]));
            float r[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) r[t] = d[t] * gelu_d_of(z[t], normal_tail(z[t]));
            z1[a] = pack4(r[0], r[1], r[2], r[3]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        // dW2 += H1^T dZ2 and its column sums, over the 128 edges
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint4 bz = sm.ex[1][(m * kTiles + wave) * kWave + lane];
            gb2 = mfma32(ones, bz, gb2);
#pragma unroll
            for (int a = 0; a < kTiles; ++a) gw2[a] = mfma32(sm.ex[0][(m * kTiles + a) * kWave + lane], bz, gw2[a]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < kTiles; ++a) put0[a * kWave * 2] = transpose(z1[a], identity);
        put1[0] = transpose(x, identity);
        __syncthreads();
        // dW1 += X^T dZ1
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint4 bz = sm.ex[0][(m * kTiles + wave) * kWave + lane];
            gb1 = mfma32(ones, bz, gb1);
            gw1 = mfma32(sm.ex[1][m * kTiles * kWave + lane], bz, gw1);
        }
        __syncthreads();
    }
    // write this workgroup's partial sums
    float* out = partial + (size_t)blockIdx.x * kParams;
    const int col = 16 * wave + c;
#pragma unroll
    for (int a = 0; a < kTiles; ++a)
#pragma unroll
        for (int t = 0; t < 4; ++t) out[kOffW2 + (16 * a + 4 * q + t) * kHid + col] = gw2[a][t];
#pragma unroll
    for (int t = 0; t < 4; ++t) out[kOffW1 + (4 * q + t) * kHid + col] = gw1[t];
    if (q == 0) {  // (every row of these results is the column sum)
        out[kOffB1 + col] = gb1[0];
        out[kOffB2 + col] = gb2[0];
    }
    // w3, b3 and the loss: over the wave, then over the waves
    float* red = reinterpret_cast<float*>(sm.ex[0]);
    constexpr int kRed = kHid + 2;
#pragma unroll
    for (int a = 0; a < kTiles; ++a) {
        float v = gw3[a];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        if (q == 0) red[wave * kRed + 16 * a + c] = v;
    }
    for (int o = 1; o < 16; o <<= 1) {
        gb3 += __shfl_xor(gb3, o);
        loss += __shfl_xor(loss, o);
    }
    if (lane == 0) {
        red[wave * kRed + kHid] = gb3;
        red[wave * kRed + kHid + 1] = loss;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kRed; t += kMlpThreads) {
        float v = red[t];
        for (int w = 1; w < kMlpThreads / kWave; ++w) v += red[w * kRed + t];
        if (t < kHid)
            out[kOffW3 + t] = v;
        else if (t == kHid)
            out[kOffB3] = v;
        else
            partial[(size_t)gridDim.x * kParams + blockIdx.x] = v;
    }
}

// grad[i] = sum over workgroups of partial[w][i], in a fixed order (eight runs
// of workgroups, each in order, then the runs in order); the loss sum goes to
// grad[kParams]. One wave per 64 parameters and run: 256 workgroups' 19 MB in
// 8.3 us (66 with one thread per parameter).
__global__ __launch_bounds__(512) void k_grad_reduce(const float* __restrict__ partial, int groups,
                                                     float* __restrict__ grad) {
    __shared__ float part[8][kWave];
    const int lane = threadIdx.x & 63, run = threadIdx.x >> 6;
    const int i = blockIdx.x * kWave + lane;
    const int per = (groups + 7) / 8, w0 = run * per, w1 = w0 + per < groups ? w0 + per : groups;
    float s = 0.0f;
    if (i < kParams) {
#pragma unroll 8
        for (int w = w0; w < w1; ++w) s += partial[(size_t)w * kParams + i];
    } else if (i == kParams) {
        for (int w = w0; w < w1; ++w) s += partial[(size_t)groups * kParams + w];
    }
    part[run][lane] = s;
    __syncthreads();
    if (run != 0 || i > kParams) return;
    for (int r = 1; r < 8; ++r) s += part[r][lane];
    grad[i] = s;
}

// Adam in FP32: m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g g;
// p -= lr (m / c1) / (sqrt(v / c2) + eps)
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ v, int count, float lr, float b1, float b2, float eps,
                                              float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float o1 = 1.0f - b1, o2 = 1.0f - b2;
    const float gi = g[i];
    const float mi = b1 * m[i] + o1 * gi;
    const float vi = b2 * v[i] + o2 * (gi * gi);
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// eta_ij = fl(fl(1/d_ij) * fl(2 sigma(s_ij))) on the 16 nearest of i, the
// multiplier of i's lowest score elsewhere; heur = eta^beta. Dense: heur is
// n*n, one workgroup a row: the multipliers are formed once per row (sixteen
// lanes) and the scored cities marked in a bitmask, so an entry costs its
// distance, a bit and the arithmetic; the scored entries are written by the
// sixteen lanes alone. A stream of 8 bytes an entry: n = 3795 106 -> 29 us
// (every entry searched its row's sixteen cities and took their minimum).
__global__ __launch_bounds__(256) void k_install_dense(const int32_t* __restrict__ dist,
                                                       const uint16_t* __restrict__ knn, const float* __restrict__ s,
                                                       int n, int beta, float* __restrict__ heur) {
    __shared__ uint32_t s_scored[2048];  // one bit per city (n <= 65535), set for the scored and i
    const int i = blockIdx.x;
    const int words = (n + 31) >> 5;
    for (int w = threadIdx.x; w < words; w += blockDim.x) s_scored[w] = 0u;
    float smin = s[i * kK];
#pragma unroll
    for (int r = 1; r < kK; ++r) {
        const float v = s[i * kK + r];
        smin = v < smin ? v : smin;
    }
    const float rest = 2.0f * sigmoid_f32(smin);
    const int32_t* drow = dist + (size_t)i * n;
    float* hrow = heur + (size_t)i * n;
    __syncthreads();
    if (threadIdx.x < kK) {
        const int j = knn[i * kK + threadIdx.x];
        // (the first of two equal neighbours counts)
        bool first = j != i && j < n;
        for (int r = 0; r < (int)threadIdx.x; ++r) first = first && knn[i * kK + r] != j;
        if (first) {
            atomicOr(&s_scored[j >> 5], 1u << (j & 31));
            const float x = (1.0f / (float)drow[j]) * (2.0f * sigmoid_f32(s[i * kK + threadIdx.x]));
            hrow[j] = powi(x, beta);
        }
    } else if (threadIdx.x == kK) {
        atomicOr(&s_scored[i >> 5], 1u << (i & 31));
        hrow[i] = 0.0f;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const float x = (1.0f / (float)drow[j]) * rest;
        if (!((s_scored[j >> 5] >> (j & 31)) & 1u)) hrow[j] = powi(x, beta);
    }
}

// the same along the candidate lists (n*cl)
__global__ __launch_bounds__(256) void k_install_cand(const int32_t* __restrict__ dist,
                                                      const uint16_t* __restrict__ knn, const float* __restrict__ s,
                                                      const uint16_t* __restrict__ cand, int n, int cl, int beta,
                                                      float* __restrict__ heur) {
    const size_t total = (size_t)n * cl;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(e / cl);
        const int j = (int)cand[e];
        float h = 0.0f;
        if (i != j) {
            const float eta = 1.0f / (float)dist[(size_t)i * n + j];
            // own score if j is among the 16 nearest, else the lowest score of i
            float smin = s[i * kK], sc = 0.0f;
            bool found = false;
            for (int r = 0; r < kK; ++r) {
                const float v = s[i * kK + r];
                smin = v < smin ? v : smin;
                if (!found && knn[i * kK + r] == j) {
                    sc = v;
                    found = true;
                }
            }
            const float x = eta * (2.0f * sigmoid_f32(found ? sc : smin));
            h = powi(x, beta);
        }
        heur[e] = h;
    }
}

// target of edge (i, knn[i][r]): the share of the R tours that use it
__global__ __launch_bounds__(256) void k_labels(const uint16_t* __restrict__ tours, int R, int n,
                                                const uint16_t* __restrict__ knn, float* __restrict__ label) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * kK) return;
    const int i = e / kK, j = knn[e];
    int hits = 0;
    for (int t = 0; t < R; ++t) {
        const uint16_t* tr = tours + (size_t)t * n;
        // positions of i and j: scan (n is small in training instances)
        int pi = -1, pj = -1;
        for (int k = 0; k < n; ++k) {
            if (tr[k] == i) pi = k;
            if (tr[k] == j) pj = k;
        }
        const int dpos = pi > pj ? pi - pj : pj - pi;
        hits += (dpos == 1 || dpos == n - 1) ? 1 : 0;
    }
    label[e] = (float)hits / (float)R;
}

int grid_of(size_t total) {
    size_t g = (total + 255) / 256;
    if (g > 65536) g = 65536;
    return g < 1 ? 1 : (int)g;
}

}  // namespace

int mlp_param_count() { return kParams; }
int mlp_packed_count() { return kPacked; }

hipError_t launch_features(const int32_t* dist, const float* xy, uint16_t* knn, int n, float* dbar, int* indeg,
                           float* feat, uint16_t* X, hipStream_t st) {
    // the in-degrees are cleared by the kernel that finds the neighbours (a
    // launch of its own took 4.5 us, a memset node would not replay safely)
    hipError_t e = launch_nearest(dist, n, kK, knn, st, indeg);
    if (e != hipSuccess) return e;
    k_feat_city<<<(n * kK + 255) / 256, 256, 0, st>>>(dist, knn, n, dbar, indeg);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_feat_edge<<<(n * kK + 255) / 256, 256, 0, st>>>(dist, xy, knn, dbar, indeg, n, feat, X);
    return hipGetLastError();
}

hipError_t launch_pack(const float* p, uint16_t* pk, hipStream_t st) {
    k_pack<<<64, 256, 0, st>>>(p, pk);
    return hipGetLastError();
}

static hipError_t smem_attr(const void* k, size_t bytes) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_mlp_forward(const uint16_t* X, const float* p, const uint16_t* pk, int64_t E, float* s,
                              hipStream_t st) {
    // (two workgroups a CU, whose 16 waves hide each other's products)
    const int64_t tiles = (E + kMlpEdges - 1) / kMlpEdges;
    const int grid = (int)(tiles < 512 ? tiles : 512);
    k_mlp_forward<<<grid < 1 ? 1 : grid, kMlpThreads, 0, st>>>(X, p, pk, E, s);
    return hipGetLastError();
}

hipError_t launch_mlp_train(const uint16_t* X, const float* f, const float* p, const uint16_t* pk, int64_t E,
                            float* partial, int groups, float* grad, hipStream_t st) {
    hipError_t e = smem_attr((const void*)k_mlp_train, sizeof(TrainSmem));
    if (e != hipSuccess) return e;
    k_mlp_train<<<groups, kMlpThreads, sizeof(TrainSmem), st>>>(X, f, p, pk, E, partial);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_grad_reduce<<<(kParams + kWave) / kWave, 512, 0, st>>>(partial, groups, grad);
    return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, float lr, float b1, float b2, float eps, float c1,
                       float c2, hipStream_t st) {
    k_adam<<<(kParams + 255) / 256, 256, 0, st>>>(p, g, m, v, kParams, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_install(const int32_t* dist, const uint16_t* knn, const float* s, const uint16_t* cand, int n, int cl,
                          int beta, int dense, float* heur, hipStream_t st) {
    if (dense)
        k_install_dense<<<n, 256, 0, st>>>(dist, knn, s, n, beta, heur);
    else
        k_install_cand<<<grid_of((size_t)n * cl), 256, 0, st>>>(dist, knn, s, cand, n, cl, beta, heur);
    return hipGetLastError();
}

hipError_t launch_labels(const uint16_t* tours, int R, int n, const uint16_t* knn, float* label, hipStream_t st) {
    k_labels<<<(n * kK + 255) / 256, 256, 0, st>>>(tours, R, n, knn, label);
    return hipGetLastError();
}

}  // namespace mmas

// ---- scratch for callers that cannot allocate ------------------------------------

// The feature pass's per-city scratch (dbar as FP32, then the in-degree
// counters as int32: 8 bytes per city) for the largest instance the library
// takes, held by every GPU the library runs on until the process ends. Host
// code never passes this name to a kernel (on the host it is only a stand-in
// for the symbol): it uses the device address hipGetSymbolAddress returns.
constexpr int kScratchCities = 65535;
static __device__ __align__(256) uint8_t scratch[8 * (size_t)kScratchCities];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices];  // device address of `scratch`, per device

// The current device's copy of `scratch`, looked up on the first call on
// that device (with it current) and kept.
mmas_status scratch_of_current_device(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return mmas::hip_fail(e, "hipGetDevice (static feature scratch)");
    if (dev < 0 || dev >= kScratchDevices) return MMAS_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return mmas::hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol,
                                                           "hipGetSymbolAddress (static feature scratch)");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MMAS_OK;
}
}  // namespace

// ---- C ABI ----------------------------------------------------------------------

namespace {
hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }
mmas_status st_of(hipError_t e) { return e == hipSuccess ? MMAS_OK : mmas::hip_fail(e, "learned-heuristic kernel"); }
}  // namespace

extern "C" {

int32_t mmas_mlp_param_count(void) { return mmas::mlp_param_count(); }
int32_t mmas_mlp_packed_count(void) { return mmas::mlp_packed_count(); }

mmas_status mmas_mlp_features(const int32_t* dist_dev, const float* xy_dev, int32_t n, void* scratch_dev,
                              uint16_t* knn_dev, float* feat_dev, uint16_t* x_dev, void* hip_stream) {
    if (!dist_dev || !xy_dev || !scratch_dev || !knn_dev || !x_dev || n < 17 || n > 65535) return MMAS_EINVAL;
    hipStream_t st = as_stream(hip_stream);
    float* dbar = reinterpret_cast<float*>(scratch_dev);
    int* indeg = reinterpret_cast<int*>(dbar + n);
    return st_of(mmas::launch_features(dist_dev, xy_dev, knn_dev, n, dbar, indeg, feat_dev, x_dev, st));
}

mmas_status mmas_mlp_features_noalloc(const int32_t* dist_dev, const float* xy_dev, int32_t n, uint16_t* knn_dev,
                                      float* feat_dev, uint16_t* x_dev, void* hip_stream) {
    if (!dist_dev || !xy_dev || !knn_dev || !x_dev || n < 17) return MMAS_EINVAL;
    if (n > kScratchCities) return MMAS_EINVAL;  // beyond the static scratch (and the library's n)
    void* ws = nullptr;
    const mmas_status got = scratch_of_current_device(&ws);
    if (got != MMAS_OK) return got;
    hipStream_t st = as_stream(hip_stream);
    // the in-degree counters are cleared by a kernel inside launch_features
    float* dbar = reinterpret_cast<float*>(ws);
    int* indeg = reinterpret_cast<int*>(dbar + n);
    return st_of(mmas::launch_features(dist_dev, xy_dev, knn_dev, n, dbar, indeg, feat_dev, x_dev, st));
}

mmas_status mmas_mlp_pack(const float* params_dev, uint16_t* packed_dev, void* hip_stream) {
    if (!params_dev || !packed_dev) return MMAS_EINVAL;
    return st_of(mmas::launch_pack(params_dev, packed_dev, as_stream(hip_stream)));
}

mmas_status mmas_mlp_forward(const uint16_t* x_dev, int64_t edges, const float* params_dev, const uint16_t* packed_dev,
                             float* s_dev, void* hip_stream) {
    if (edges < 0 || (edges > 0 && (!x_dev || !params_dev || !packed_dev || !s_dev))) return MMAS_EINVAL;
    if (edges == 0) return MMAS_OK;
    return st_of(mmas::launch_mlp_forward(x_dev, params_dev, packed_dev, edges, s_dev, as_stream(hip_stream)));
}

mmas_status mmas_mlp_grad(const uint16_t* x_dev, const float* target_dev, int64_t edges, const float* params_dev,
                          const uint16_t* packed_dev, float* partial_dev, int32_t groups, float* grad_dev,
                          void* hip_stream) {
    if (edges < 1 || groups < 1 || groups > 4096 || !x_dev || !target_dev || !params_dev || !packed_dev ||
        !partial_dev || !grad_dev)
        return MMAS_EINVAL;
    return st_of(mmas::launch_mlp_train(x_dev, target_dev, params_dev, packed_dev, edges, partial_dev, groups,
                                        grad_dev, as_stream(hip_stream)));
}

mmas_status mmas_mlp_adam(float* params_dev, const float* grad_dev, float* m_dev, float* v_dev, float lr, float beta1,
                          float beta2, float eps, int32_t step, void* hip_stream) {
    if (!params_dev || !grad_dev || !m_dev || !v_dev || step < 1) return MMAS_EINVAL;
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    return st_of(mmas::launch_adam(params_dev, grad_dev, m_dev, v_dev, lr, beta1, beta2, eps, c1, c2,
                                   as_stream(hip_stream)));
}

mmas_status mmas_mlp_labels(const uint16_t* tours_dev, int32_t tours, int32_t n, const uint16_t* knn_dev,
                            float* target_dev, void* hip_stream) {
    if (!tours_dev || !knn_dev || !target_dev || tours < 1 || n < 17) return MMAS_EINVAL;
    return st_of(mmas::launch_labels(tours_dev, tours, n, knn_dev, target_dev, as_stream(hip_stream)));
}

}  // extern "C"
