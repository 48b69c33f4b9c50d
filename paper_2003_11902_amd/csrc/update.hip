// Per-iteration kernels around construction (Alg. 1, Sec. 2.1):
//  - choice_info = tau^alpha * eta^beta, dense and along the candidate lists,
//    and its reciprocal beside both (Sec. 4.2.2: the reciprocal of every
//    weight computed once per iteration, so that a key is a product);
//  - the iteration best, the global best and the trail limits (one workgroup);
//  - evaporation, deposit on both directions of the iteration best's edges (on
//    (i, succ(i)) alone for the asymmetric TSP) and the [tau_min, tau_max] clamp, fused with the refresh of choice_info (the
//    paper's evaporation and deposition kernels in one pass; each entry is
//    independent, so no atomics are needed).
#include "device.hpp"
#include "internal.hpp"

namespace mmas {
namespace {

// dense: one workgroup per row
__global__ __launch_bounds__(256) void k_choice_dense(const float* __restrict__ tau, const float* __restrict__ heur,
                                                      const uint16_t* __restrict__ cand, int n, int cl, int alpha,
                                                      float* __restrict__ choice, float* __restrict__ choice_inv,
                                                      float* __restrict__ chc, float* __restrict__ chc_inv) {
    const size_t i = blockIdx.x;
    const float* trow = tau + i * n;
    const float* hrow = heur + i * n;
    float* crow = choice + i * n;
    float* irow = choice_inv + i * n;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const float c = powi(trow[j], alpha) * hrow[j];
        crow[j] = c;
        irow[j] = 1.0f / c;
    }
    for (int r = threadIdx.x; r < cl; r += blockDim.x) {
        const int j = cand[i * cl + r];
        const float c = powi(trow[j], alpha) * hrow[j];
        chc[i * cl + r] = c;
        chc_inv[i * cl + r] = 1.0f / c;
    }
}

// candidate-only trails: heur is n*cl along the lists
__global__ __launch_bounds__(256) void k_choice_cand(const float* __restrict__ tau, const float* __restrict__ heur,
                                                     size_t count, int alpha, float* __restrict__ chc,
                                                     float* __restrict__ chc_inv) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x) {
        const float c = powi(tau[e], alpha) * heur[e];
        chc[e] = c;
        chc_inv[e] = 1.0f / c;
    }
}

// The shortest tour and its ant, the lowest on ties (every thread of the
// workgroup gets both; any multiple of 64 threads up to 1024).
__device__ __forceinline__ void shortest_tour(const Views& vw, int ants, int64_t& len, int32_t& ant) {
    __shared__ int64_t plen[16];
    __shared__ int32_t pant[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t blen = INT64_MAX;
    int32_t bant = INT32_MAX;
    for (int a = threadIdx.x; a < ants; a += blockDim.x) {
        const int64_t L = vw.lengths[a];
        if (L < blen) {  // ascending a: the first minimum is the lowest ant
            blen = L;
            bant = a;
        }
    }
    for (int o = 32; o >= 1; o >>= 1) {
        const int64_t ol = __shfl_xor(blen, o);
        const int32_t oa = __shfl_xor(bant, o);
        if (ol < blen || (ol == blen && oa < bant)) {
            blen = ol;
            bant = oa;
        }
    }
    if (lane == 0) {
        plen[wave] = blen;
        pant[wave] = bant;
    }
    __syncthreads();
    len = plen[0];
    ant = pant[0];
    for (int w = 1; w < nw; ++w)
        if (plen[w] < len || (plen[w] == len && pant[w] < ant)) {
            len = plen[w];
            ant = pant[w];
        }
}

// Iteration best = shortest tour, lowest ant on ties. If it beats the global
// best (or there is none yet), it becomes the global best and the limits are
// recomputed from its length. Then the successor and predecessor of every
// city along the tour that deposits: the iteration best, or the global best
// (Sec. 2.1 allows either). One workgroup of any size
// (a multiple of 64, at most 1024 threads).
__device__ void best_and_limits(const Views& vw, const Shape& s) {
    __shared__ int s_ib;
    __shared__ int s_improved;
    int64_t L;
    int32_t a;
    shortest_tour(vw, s.ants, L, a);
    if (threadIdx.x == 0) {
        mmas_device_state* st = vw.state;
        st->ib_ant = a;
        st->ib_len = L;
        const int improved = (st->gb_len < 0 || L < st->gb_len) ? 1 : 0;
        if (improved) {
            st->gb_len = L;
            float lo, hi;
            trail_limits(s.rho, L, s.n, s.pdec, &lo, &hi);
            st->tau_min = lo;
            st->tau_max = hi;
        }
        st->delta = (float)(1.0 / (double)(s.deposit == MMAS_DEPOSIT_GLOBAL_BEST ? st->gb_len : L));
        st->updates += 1u;
        s_ib = a;
        s_improved = improved;
    }
    __syncthreads();
    const uint16_t* t = vw.tours + (size_t)s_ib * s.n;
    const int n = s.n;
    if (s.deposit == MMAS_DEPOSIT_GLOBAL_BEST && !s_improved) {
        // the global best deposits and is unchanged: its stored tour
        for (int k = threadIdx.x; k < n; k += blockDim.x) {
            const uint16_t a = vw.gb_tour[k], b = vw.gb_tour[k + 1 == n ? 0 : k + 1];
            vw.succ[a] = b;
            vw.pred[b] = a;
        }
        return;
    }
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const uint16_t a = t[k], b = t[k + 1 == n ? 0 : k + 1];
        vw.succ[a] = b;
        vw.pred[b] = a;
        if (s_improved) vw.gb_tour[k] = a;
    }
}

__global__ __launch_bounds__(1024) void k_best(Views vw, Shape s) { best_and_limits(vw, s); }

__device__ __forceinline__ float evaporate_deposit(float t, bool dep, float keep, float tmin, float tmax,
                                                   float delta) {
    float v = keep * t;
    if (v < tmin) v = tmin;
    if (dep) v = v + delta;
    if (v > tmax) v = tmax;
    return v;
}

// What row i's update needs of the iteration: limits, deposit, and the two
// cities whose edges with i receive it (-1: none).
struct Deposit {
    float tmin, tmax, delta;
    int succ, pred;
};
__device__ __forceinline__ Deposit deposit_of(const Views& vw, const Shape& s, size_t i) {
    const mmas_device_state* st = vw.state;
    return Deposit{st->tau_min, st->tau_max, st->delta, (int)vw.succ[i], s.directed ? -1 : (int)vw.pred[i]};
}

// four consecutive row entries, aligned to one
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

// dense, row i by kWaves waves (threads 0 .. 64 kWaves - 1 of the row as t).
// The candidate entries of chc are computed first from the old trails (each
// thread recomputes its entry's new value), then the row is rewritten, four
// entries a thread at once with kVec. An HBM stream of 20 bytes per entry. In
// a batch a wave takes a row up to kRowWave cities and a workgroup four: the
// search for a row's instance and a workgroup's start for each short row cost
// as much as the stream (160 colonies, n 200-1000: 432 -> 290 us, 4.3 TB/s;
// with longer rows 107 -> 107 us). One colony: four entries at once from
// kRowWave cities on (n = 3795: 55 -> 51 us; at n = 1002 and below one entry a
// thread is as fast, and 1 us faster at n = 198, where one chain of four
// divisions is the kernel's tail).
template <int kWaves, bool kVec>
__device__ __forceinline__ void update_dense_row(const Views& vw, const Shape& s, size_t i, int t, const Deposit& d) {
    const int n = s.n, cl = s.cl;
    const float tmin = d.tmin, tmax = d.tmax, delta = d.delta;
    const float keep = 1.0f - s.rho;
    const int si = d.succ, pi = d.pred;
    float* trow = vw.tau + i * n;
    const float* hrow = vw.heur + i * n;
    float* crow = vw.choice + i * n;
    float* irow = vw.choice_inv + i * n;
    for (int r = t; r < cl; r += kWave * kWaves) {
        const int j = vw.cand[i * cl + r];
        const float tau = evaporate_deposit(trow[j], j == si || j == pi, keep, tmin, tmax, delta);
        const float c = powi(tau, s.alpha) * hrow[j];
        vw.chc[i * cl + r] = c;
        vw.chc_inv[i * cl + r] = 1.0f / c;
    }
    if (kWaves > 1) __syncthreads();
    constexpr int kStep = kVec ? 4 : 1;
    for (int j0 = kStep * t; j0 < n; j0 += kStep * kWave * kWaves) {
        if (kVec && j0 + 4 <= n) {
            f32x4_u tv = *reinterpret_cast<const f32x4_u*>(trow + j0);
            const f32x4_u hv = *reinterpret_cast<const f32x4_u*>(hrow + j0);
            f32x4_u cv, iv;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = j0 + q;
                tv[q] = evaporate_deposit(tv[q], j == si || j == pi, keep, tmin, tmax, delta);
                cv[q] = powi(tv[q], s.alpha) * hv[q];
                iv[q] = 1.0f / cv[q];
            }
            *reinterpret_cast<f32x4_u*>(trow + j0) = tv;
            *reinterpret_cast<f32x4_u*>(crow + j0) = cv;
            *reinterpret_cast<f32x4_u*>(irow + j0) = iv;
        } else {
            for (int j = j0; j < n && j < j0 + kStep; ++j) {
                const float tau = evaporate_deposit(trow[j], j == si || j == pi, keep, tmin, tmax, delta);
                const float c = powi(tau, s.alpha) * hrow[j];
                trow[j] = tau;
                crow[j] = c;
                irow[j] = 1.0f / c;
            }
        }
    }
}

// candidate-only trails, row i (its cl stored entries)
__device__ __forceinline__ void update_cand_row(const Views& vw, const Shape& s, size_t i, int t) {
    const mmas_device_state* st = vw.state;
    const float tmin = st->tau_min, tmax = st->tau_max, delta = st->delta;
    const float keep = 1.0f - s.rho;
    const int si = vw.succ[i], pi = s.directed ? -1 : (int)vw.pred[i];
    for (int r = t; r < s.cl; r += kWave) {
        const size_t e = i * s.cl + r;
        const int j = vw.cand[e];
        const float tau = evaporate_deposit(vw.tau[e], j == si || j == pi, keep, tmin, tmax, delta);
        vw.tau[e] = tau;
        const float c = powi(tau, s.alpha) * vw.heur[e];
        vw.chc[e] = c;
        vw.chc_inv[e] = 1.0f / c;
    }
}

// one workgroup a row
template <bool kVec>
__global__ __launch_bounds__(256) void k_update_dense(Views vw, Shape s) {
    const size_t i = blockIdx.x;
    update_dense_row<4, kVec>(vw, s, i, threadIdx.x, deposit_of(vw, s, i));
}

// The whole update of a small colony in one launch: every workgroup finds the
// iteration best (8 bytes an ant) and its four rows' neighbours in the
// depositing tour for itself, and the last one to finish commits the new
// state and global best, which the others have read before (so none sees a
// half-written one). Saves a launch, its gap and the best's chain of loads:
// n = 198 10.1 -> 8.1 us by events, n = 600 11.6 -> 10.5, n = 1002 14.4 ->
// 14.0; from there on reading the lengths in every workgroup costs more (with
// one row a workgroup the tickets do: n = 1002 21.7 us).
__global__ __launch_bounds__(256) void k_update_small(Views vw, Shape s) {
    constexpr int kRows = 4;
    __shared__ int s_at[kRows][2];
    __shared__ float s_lim[3];
    __shared__ int s_last;
    const int i0 = (int)blockIdx.x * kRows;
    const int n = s.n;
    const mmas_device_state old = *vw.state;
    if (threadIdx.x < 2 * kRows) s_at[threadIdx.x >> 1][threadIdx.x & 1] = -1;
    int64_t L;
    int32_t ib;
    shortest_tour(vw, s.ants, L, ib);
    const bool improved = old.gb_len < 0 || L < old.gb_len;
    const int64_t gb = improved ? L : old.gb_len;
    // the tour that deposits
    const bool stored = s.deposit == MMAS_DEPOSIT_GLOBAL_BEST && !improved;
    const uint16_t* tour = stored ? vw.gb_tour : vw.tours + (size_t)ib * n;
    if (threadIdx.x == 0) {
        float lo = old.tau_min, hi = old.tau_max;
        if (improved) trail_limits(s.rho, L, n, s.pdec, &lo, &hi);
        s_lim[0] = lo;
        s_lim[1] = hi;
        s_lim[2] = (float)(1.0 / (double)(s.deposit == MMAS_DEPOSIT_GLOBAL_BEST ? gb : L));
    }
    for (int k = threadIdx.x; k < n; k += blockDim.x)
        if (const int r = (int)tour[k] - i0; r >= 0 && r < kRows) {
            s_at[r][0] = tour[k + 1 == n ? 0 : k + 1];
            s_at[r][1] = tour[k == 0 ? n - 1 : k - 1];
        }
    __syncthreads();
    const int r = threadIdx.x >> 6;
    if (i0 + r < n)
        update_dense_row<1, true>(vw, s, i0 + r, threadIdx.x & 63,
                                  Deposit{s_lim[0], s_lim[1], s_lim[2], s_at[r][0], s.directed ? -1 : s_at[r][1]});
    if (threadIdx.x == 0) s_last = atomicAdd(vw.ticket, 1u) + 1u == gridDim.x ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    // (every workgroup has read the old state: each did before its ticket)
    if (improved)
        for (int k = threadIdx.x; k < n; k += blockDim.x) vw.gb_tour[k] = tour[k];
    if (threadIdx.x == 0) {
        mmas_device_state* st = vw.state;
        st->ib_ant = ib;
        st->ib_len = L;
        st->gb_len = gb;
        st->tau_min = s_lim[0];
        st->tau_max = s_lim[1];
        st->delta = s_lim[2];
        st->updates = old.updates + 1u;
        *vw.ticket = 0u;
    }
}

// batches: one workgroup per instance for the best, then one per update tile
__global__ __launch_bounds__(1024) void k_batch_best(const BatchItem* __restrict__ items, uint32_t* it_dev,
                                                     uint32_t* queue) {
    best_and_limits(items[blockIdx.x].v, items[blockIdx.x].s);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *it_dev += 1u;  // construction of this iteration is done
        *queue = 0u;    // re-arm the tile queue for the next construction
    }
}

// tile (instance, first row): one row of an instance with more than kRowWave
// cities and dense trails, else four (the last ones of an instance may be
// missing)
__global__ __launch_bounds__(256) void k_batch_update(const BatchItem* __restrict__ items,
                                                      const BatchTile* __restrict__ tiles) {
    const int inst = __builtin_amdgcn_readfirstlane(tiles[blockIdx.x].inst);
    const int row0 = __builtin_amdgcn_readfirstlane(tiles[blockIdx.x].ant0);
    const Views& vw = items[inst].v;
    const Shape& s = items[inst].s;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (s.pher == MMAS_PHER_DENSE && s.n > kRowWave) {
        update_dense_row<4, true>(vw, s, row0, threadIdx.x, deposit_of(vw, s, row0));
        return;
    }
    if (row0 + wave >= s.n) return;
    if (s.pher == MMAS_PHER_DENSE)
        update_dense_row<1, true>(vw, s, row0 + wave, lane, deposit_of(vw, s, row0 + wave));
    else
        update_cand_row(vw, s, row0 + wave, lane);
}

__global__ __launch_bounds__(256) void k_update_cand(Views vw, Shape s) {
    const size_t count = (size_t)s.n * s.cl;
    const mmas_device_state* st = vw.state;
    const float tmin = st->tau_min, tmax = st->tau_max, delta = st->delta;
    const float keep = 1.0f - s.rho;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += (size_t)gridDim.x * blockDim.x) {
        const size_t i = e / s.cl;
        const int j = vw.cand[e];
        const bool dep = j == vw.succ[i] || (!s.directed && j == vw.pred[i]);
        const float t = evaporate_deposit(vw.tau[e], dep, keep, tmin, tmax, delta);
        vw.tau[e] = t;
        const float c = powi(t, s.alpha) * vw.heur[e];
        vw.chc[e] = c;
        vw.chc_inv[e] = 1.0f / c;
    }
}

// Sizes up to which the update is one launch (k_update_small): with more ants
// every workgroup's reading of the lengths costs as much as the launch it saves
// (two launches -> one, 1536 ants: n = 50 10.2 -> 10.2 us, n = 200 10.4 -> 9.4,
// n = 1000 16.5 -> 16.5; 2048 ants: 10.3 -> 10.8, 10.7 -> 9.8, 16.7 -> 17.1).
constexpr int kFusedRows = 1024, kFusedAnts = 1536;

int grid_for(size_t total, int block) {
    size_t g = (total + block - 1) / block;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

}  // namespace

hipError_t launch_choice(const Views& v, const Shape& s, hipStream_t st) {
    if (s.pher == MMAS_PHER_DENSE) {
        k_choice_dense<<<s.n, 256, 0, st>>>(v.tau, v.heur, v.cand, s.n, s.cl, s.alpha, v.choice, v.choice_inv, v.chc,
                                            v.chc_inv);
    } else {
        const size_t count = (size_t)s.n * s.cl;
        k_choice_cand<<<grid_for(count, 256), 256, 0, st>>>(v.tau, v.heur, count, s.alpha, v.chc, v.chc_inv);
    }
    return hipGetLastError();
}

hipError_t launch_batch_update(const BatchItem* items, int count, const BatchTile* tiles, int ntiles, uint32_t* it_dev,
                               uint32_t* queue, hipStream_t st) {
    k_batch_best<<<count, 256, 0, st>>>(items, it_dev, queue);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_batch_update<<<ntiles, 256, 0, st>>>(items, tiles);
    return hipGetLastError();
}

hipError_t launch_update(const Views& v, const Shape& s, hipStream_t st) {
    if (s.pher == MMAS_PHER_DENSE && s.n <= kFusedRows && s.ants <= kFusedAnts) {
        k_update_small<<<(s.n + 3) / 4, 256, 0, st>>>(v, s);
        return hipGetLastError();
    }
    k_best<<<1, 1024, 0, st>>>(v, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (s.pher == MMAS_PHER_DENSE) {
        if (s.n > kRowWave)
            k_update_dense<true><<<s.n, 256, 0, st>>>(v, s);
        else
            k_update_dense<false><<<s.n, 256, 0, st>>>(v, s);
    } else {
        const size_t count = (size_t)s.n * s.cl;
        k_update_cand<<<grid_for(count, 256), 256, 0, st>>>(v, s);
    }
    return hipGetLastError();
}

}  // namespace mmas
