// Set-up kernels (Alg. 1 before its main loop): validation of the distance
// matrix, eta^beta, candidate and neighbour lists, the nearest-neighbour tour,
// the initial trail limits and tau <- tau_max.
#include "device.hpp"
#include "internal.hpp"

namespace mmas {
namespace {

// flags: 1 = asymmetric, 2 = non-zero diagonal, 4 = non-positive off-diagonal.
// 32x32 tiles; the transposed tile is staged in LDS so both reads coalesce.
// With `directed` (ATSP) an asymmetric matrix is valid and flag 1 is not set.
__global__ __launch_bounds__(256) void k_validate(const int32_t* __restrict__ d, int n, int directed,
                                                  uint32_t* __restrict__ flags) {
    __shared__ int32_t tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x, ty = threadIdx.y;
    for (int j = ty; j < 32; j += 8) {
        const int r = by + j, c = bx + tx;
        if (r < n && c < n) tile[j][tx] = d[(size_t)r * n + c];
    }
    __syncthreads();
    uint32_t f = 0;
    for (int j = ty; j < 32; j += 8) {
        const int r = bx + j, c = by + tx;  // element d[r][c]; tile holds d[by+.][bx+.]
        if (r < n && c < n) {
            const int32_t x = d[(size_t)r * n + c];
            const int32_t y = tile[tx][j];  // d[c][r]
            if (x != y && !directed) f |= 1u;
            if (r == c) {
                if (x != 0) f |= 2u;
            } else if (x <= 0) {
                f |= 4u;
            }
        }
    }
    if (f) atomicOr(flags, f);
}

__global__ __launch_bounds__(256) void k_heur_dense(const int32_t* __restrict__ d, int n, int beta,
                                                    float* __restrict__ heur) {
    const size_t total = (size_t)n * n;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(e / n), j = (int)(e % n);
        heur[e] = (i == j) ? 0.0f : heur_from_dist(d[e], beta);
    }
}

__global__ __launch_bounds__(256) void k_heur_cand(const int32_t* __restrict__ d, const uint16_t* __restrict__ cand,
                                                   int n, int cl, int beta, float* __restrict__ heur) {
    const size_t total = (size_t)n * cl;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const size_t i = e / cl;
        heur[e] = heur_from_dist(d[i * n + cand[e]], beta);
    }
}

// Entries of a row that k_nearest sorts at once.
constexpr int kNearCap = 256;

// The k <= 64 nearest other cities of row i by (distance, index), one wave a
// row: the row's entries fall into 128 groups (two per lane); the k-th
// smallest group minimum, or a little more, bounds the k-th smallest entry, so
// a second pass gathers the few entries up to that bound (37 of 3795 on
// average for k = 32) and their ranks among each other are their places.
// A wave's time is its reads' latency (the whole grid is resident at once), so
// a row of up to 64 kRegs cities is read once, all loads in flight, and kept
// in registers; a longer one (kRegs = 0) twice, eight loads in flight (sixteen
// change nothing). k = 16, n = 3795 / 18512: 17.7 / 460 us; 35.0 / 661 with
// four loads and then one in flight, 184 / 4470 by taking the next smallest
// entry k times. (n = 3795: 57.6 MB, 12 us at a copy's rate.)
// Rows with more than kNearCap entries up to the bound (long runs of equal
// distances) look for the least bound that holds k, by bisection over all
// entries, and take of the cities at it the first ones (n = 3795, distances
// 1 to 10: 81 us for the three kernels of the features; 520 by taking the next
// smallest entry k times in the wave, 216 in four waves).
// `clear` (or null): cleared at i, for the kernel that counts in-degrees next.
template <int kRegs>
__global__ __launch_bounds__(256) void k_nearest(const int32_t* __restrict__ d, int n, int k,
                                                 uint16_t* __restrict__ out, int* __restrict__ clear) {
    constexpr int kBatch = kRegs ? kRegs : 8;
    __shared__ uint64_t s_key[4][kNearCap];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int i = (int)blockIdx.x * 4 + wave;
    if (i >= n) return;
    if (clear && lane == 0) clear[i] = 0;
    const int32_t* row = d + (size_t)i * n;
    uint16_t* o = out + (size_t)i * k;
    // the entries of kBatch 64-city pieces from city j0 on (all ones past the
    // row's end and for i itself); the last, partial piece is read once, and
    // pieces past the end read the last full one instead (the first cities
    // again where there is none): scalar bases and one lane offset
    const int full = n >> 6, lc = min(lane, n - 1), self = i >> 6;
    const bool own = lane == (i & 63);
    const uint32_t tail = full * kWave + lane < n ? (uint32_t)row[full * kWave + lane] : ~0u;
    uint32_t x[kBatch];
    auto fetch = [&](int j0) {
        const int p0 = j0 >> 6;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) x[u] = (uint32_t)(row + max(min(p0 + u, full - 1), 0) * kWave)[lc];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            uint32_t v = p0 + u < full ? x[u] : p0 + u == full ? tail : ~0u;
            x[u] = p0 + u == self && own ? ~0u : v;
        }
    };
    uint32_t m0 = ~0u, m1 = ~0u;
    for (int j0 = 0; j0 < n; j0 += kBatch * kWave) {
        fetch(j0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (u & 1)
                m1 = min(m1, x[u]);
            else
                m0 = min(m0, x[u]);
        }
    }
    // the least bound under which at least k group minima lie, or one with up
    // to eight more (bisection; every group but that of i alone has a minimum,
    // and there are at least k such groups)
    uint32_t lo = wave_min_u32<4>(min(m0, m1)), hi = ~0u - 1u;
    {
        const uint32_t g0 = m0 == ~0u ? 0u : m0, g1 = m1 == ~0u ? 0u : m1;
        hi = wave_max_u32<4>(max(g0, g1));
    }
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        const int c = __popcll(__ballot(m0 <= mid)) + __popcll(__ballot(m1 <= mid));
        if (c < k)
            lo = mid + 1;
        else
            hi = mid;
        if (c >= k && c <= k + 8) break;
    }
    // the entries up to the bound
    int m = 0;
    for (int j0 = 0; j0 < n; j0 += kBatch * kWave) {
        if (!kRegs) fetch(j0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint64_t in = __ballot(x[u] <= hi);
            if (in) {
                const int at = m + __popcll(in & ((1ull << lane) - 1ull));
                if (x[u] <= hi && at < kNearCap)
                    s_key[wave][at] = ((uint64_t)x[u] << 32) | (uint32_t)(j0 + u * kWave + lane);
                m += __popcll(in);
            }
        }
    }
    if (__builtin_expect(m > kNearCap, 0)) {
        // the least bound with k entries up to it (or with few enough to sort);
        // `below`: entries up to the bound before it
        uint32_t least = wave_min_u32<4>(min(m0, m1));
        int below = 0;
        while (least < hi) {
            const uint32_t mid = least + (hi - least) / 2;
            int c = 0;
            for (int j0 = 0; j0 < n; j0 += kBatch * kWave) {
                if (!kRegs) fetch(j0);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) c += __popcll(__ballot(x[u] <= mid));
            }
            if (c < k) {
                least = mid + 1;
                below = c;
            } else {
                hi = mid;
                if (c <= kNearCap) break;
            }
        }
        // every entry before the bound, and those at it in index order while
        // there is room (at least k in all)
        const int room = least < hi ? kNearCap : k - below;
        int at_bound = 0;
        m = 0;
        for (int j0 = 0; j0 < n; j0 += kBatch * kWave) {
            if (!kRegs) fetch(j0);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const uint64_t equal = __ballot(x[u] == hi), before = (1ull << lane) - 1ull;
                const bool mine = x[u] < hi || (x[u] == hi && at_bound + __popcll(equal & before) < room);
                const uint64_t in = __ballot(mine);
                if (mine)
                    s_key[wave][m + __popcll(in & before)] =
                        ((uint64_t)x[u] << 32) | (uint32_t)(j0 + u * kWave + lane);
                at_bound += __popcll(equal);
                m += __popcll(in);
            }
        }
    }
    // (one wave's LDS operations complete in order)
    for (int e = lane; e < ((m + kWave - 1) & ~(kWave - 1)); e += kWave) {
        const uint64_t key = e < m ? s_key[wave][e] : ~0ull;
        int rank = 0;
#pragma unroll 8
        for (int q = 0; q < m; ++q) rank += s_key[wave][q] < key ? 1 : 0;
        if (e < m && rank < k) o[rank] = (uint16_t)key;
    }
    // (a matrix that is refused may leave too few: any city keeps the later
    // set-up steps in bounds)
    for (int r = m + lane; r < k; r += kWave) o[r] = 0;
}

// LDS of the nearest-neighbour tour: visited bits, then the first `p` entries
// of every candidate list.
__host__ __device__ inline int nn_tour_bits(int n) { return (((n + 31) >> 5) * 4 + 15) & ~15; }

// The smallest (distance, index) over the unvisited cities of a row, one
// wave's share of it (cities w * 64 + lane, then every 64 nw): (distance, index)
// packed, ~0 if none.
__device__ __forceinline__ uint64_t nn_scan(const int32_t* __restrict__ row, int n, const uint32_t* vis, int w, int nw,
                                            int lane) {
    uint32_t bd = ~0u, bj = ~0u;
    for (int j = w * kWave + lane; j < n; j += kWave * nw) {
        const uint32_t v = (uint32_t)row[j];
        const bool seen = (vis[j >> 5] >> (j & 31)) & 1u;
        if (!seen && v < bd) {  // (ascending j: the first of equal distances)
            bd = v;
            bj = (uint32_t)j;
        }
    }
    const uint32_t m = wave_min_u32<4>(bd);
    const uint32_t jm = wave_min_u32<4>(bd == m ? bj : ~0u);
    return jm == ~0u ? ~0ull : ((uint64_t)m << 32) | jm;
}

// The length of the tour the first wave has written (every thread of the
// workgroup; the barrier before makes the tour visible to them).
__device__ __forceinline__ void nn_length(const int32_t* __restrict__ d, int n, const uint16_t* tour, uint64_t* part,
                                          mmas_device_state* __restrict__ st) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t len = 0;
    for (int k = threadIdx.x; k < n; k += blockDim.x)
        len += d[(size_t)tour[k] * n + tour[k + 1 == n ? 0 : k + 1]];
    len = wave_sum_i64(len);
    if (lane == 0) part[wave] = (uint64_t)len;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nw; ++w) len += (int64_t)part[w];
        st->nn_len = len;
    }
}

// Nearest-neighbour tour from city 0, then its length: one workgroup, whose
// first wave walks. The candidate list is sorted by (d, index) and holds the
// cl nearest cities, so when one of them is unvisited the first such is the
// nearest unvisited city; the first p entries of every list are in LDS (a step
// is then two LDS reads), the rest in global memory; only when all are visited
// do all the waves scan the city's row for the smallest (d, index) (the others
// wait at the barrier for that). n = 1002: 490 -> 240 us, n = 18512: 85 -> 10.4
// ms (one wave, every list and scan from global memory).
__global__ __launch_bounds__(1024) void k_nn_tour(const int32_t* __restrict__ d, const uint16_t* __restrict__ cand,
                                                  int cl, int n, int p, uint16_t* __restrict__ tour,
                                                  mmas_device_state* __restrict__ st) {
    extern __shared__ __align__(16) uint8_t smem[];  // ceil(n/32) words, then the table
    __shared__ uint64_t part[16];
    __shared__ int s_cur;  // the city whose row is to be scanned, -1: the tour is done, -2: it failed
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t* vis = reinterpret_cast<uint32_t*>(smem);
    uint16_t* tab = reinterpret_cast<uint16_t*>(smem + nn_tour_bits(n));
    const int words = (n + 31) >> 5;
    for (int w = threadIdx.x; w < words; w += blockDim.x) vis[w] = w == 0 ? 1u : 0u;
    // (lists and table start 16-byte aligned: eight entries at once where whole
    // lists are kept, four where both lengths are multiples of four)
    int done = 0;
    if (p == cl) {
        const int q = n * cl >> 3;
#pragma unroll 4
        for (int e = threadIdx.x; e < q; e += blockDim.x)
            reinterpret_cast<uint4*>(tab)[e] = reinterpret_cast<const uint4*>(cand)[e];
        done = 8 * q;
    } else if (p > 0 && ((p | cl) & 3) == 0) {
        const int pq = p >> 2, cq = cl >> 2;
#pragma unroll 4
        for (int e = threadIdx.x; e < n * pq; e += blockDim.x)
            reinterpret_cast<uint2*>(tab)[e] = reinterpret_cast<const uint2*>(cand)[(size_t)(e / pq) * cq + e % pq];
        done = n * p;
    }
    for (int e = done + threadIdx.x; e < n * p; e += blockDim.x) tab[e] = cand[(size_t)(e / p) * cl + e % p];
    __syncthreads();
    if (wave > 0) {
        for (;;) {
            __syncthreads();  // a city to scan, or the end
            const int c = __builtin_amdgcn_readfirstlane(s_cur);
            if (c < 0) {
                if (c == -1) nn_length(d, n, tour, part, st);
                return;
            }
            const uint64_t m = nn_scan(d + (size_t)c * n, n, vis, wave, nw, lane);
            if (lane == 0) part[wave] = m;
            __syncthreads();  // the waves' results
        }
    }
    // the nearest unvisited city past the first p candidates (rare)
    auto far_city = [&](int cur) -> int {
        if (p < cl) {
            const uint32_t c = cand[(size_t)cur * cl + (lane < cl ? lane : cl - 1)];
            const bool free = (lane < cl) & !((vis[c >> 5] >> (c & 31)) & 1u);
            const uint64_t m = __ballot(free);
            if (m) return __builtin_amdgcn_readlane((int)c, (int)__builtin_ctzll(m));
        }
        if (lane == 0) s_cur = cur;
        __syncthreads();
        const uint64_t own = nn_scan(d + (size_t)cur * n, n, vis, 0, nw, lane);
        if (lane == 0) part[0] = own;
        __syncthreads();
        const uint64_t r = lane < nw ? part[lane] : ~0ull;
        const uint32_t rd = (uint32_t)(r >> 32), m = wave_min_u32<4>(rd);
        return (int)wave_min_u32<4>(rd == m ? (uint32_t)r : ~0u);  // -1: no unvisited city
    };
    int cur = 0;
    uint32_t tbuf = 0;  // lane (k & 63) holds the city of step k
    bool failed = false;
    const int lp = lane < p ? lane : p - 1;
    const uint64_t listed = p >= 64 ? ~0ull : (1ull << p) - 1ull;
    for (int k = 1; k < n; ++k) {
        uint64_t m = 0ull;
        uint32_t c = 0u, word = 0u;
        if (p > 0) {
            c = tab[cur * p + lp];
            word = vis[c >> 5];
            m = __ballot(__builtin_amdgcn_ubfe(word, c, 1u) == 0u) & listed;
        }
        if (__builtin_expect(m != 0ull, 1)) {
            const int f = (int)__builtin_ctzll(m);
            cur = __builtin_amdgcn_readlane((int)c, f);
            word = (uint32_t)__builtin_amdgcn_readlane((int)word, f);
        } else {
            cur = __builtin_amdgcn_readfirstlane(far_city(cur));
            if (cur < 0) {  // unreachable for k < n
                failed = true;
                break;
            }
            word = (uint32_t)__builtin_amdgcn_readfirstlane((int)vis[cur >> 5]);
        }
        // (the only wave that writes; every lane stores the same word)
        vis[cur >> 5] = word | (1u << (cur & 31));
        if (lane == (k & 63)) tbuf = (uint32_t)cur;
        if ((k & 63) == 63 || k == n - 1) {
            const int at = (k & ~63) + lane;
            if (at <= k) tour[at] = (uint16_t)tbuf;
        }
    }
    if (lane == 0) s_cur = failed ? -2 : -1;
    __syncthreads();  // the others leave the scans
    if (failed) {
        if (lane == 0) atomicOr(&st->flags, 8u);
        return;
    }
    nn_length(d, n, tour, part, st);
}

__global__ void k_init_state(mmas_device_state* st, float rho, int n, double pdec) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        float lo, hi;
        trail_limits(rho, st->nn_len, n, pdec, &lo, &hi);
        st->tau_min = lo;
        st->tau_max = hi;
        st->delta = 0.0f;
        st->ib_ant = -1;
        st->ib_len = -1;
        st->gb_len = -1;
        st->updates = 0u;
    }
}

__global__ __launch_bounds__(256) void k_fill_tau(float* __restrict__ tau, size_t count,
                                                  const mmas_device_state* __restrict__ st) {
    const float v = st->tau_max;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
         e += (size_t)gridDim.x * blockDim.x)
        tau[e] = v;
}

int grid_for(size_t total, int block) {
    size_t g = (total + block - 1) / block;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

}  // namespace

hipError_t launch_validate(const Views& v, const Shape& s, hipStream_t st) {
    const int tiles = (s.n + 31) / 32;
    k_validate<<<dim3(tiles, tiles), dim3(32, 8), 0, st>>>(v.dist, s.n, s.directed, &v.state->flags);
    return hipGetLastError();
}

hipError_t launch_heuristic(const Views& v, const Shape& s, hipStream_t st) {
    if (s.pher == MMAS_PHER_DENSE) {
        const size_t total = (size_t)s.n * s.n;
        k_heur_dense<<<grid_for(total, 256), 256, 0, st>>>(v.dist, s.n, s.beta, v.heur);
    } else {
        const size_t total = (size_t)s.n * s.cl;
        k_heur_cand<<<grid_for(total, 256), 256, 0, st>>>(v.dist, v.cand, s.n, s.cl, s.beta, v.heur);
    }
    return hipGetLastError();
}

hipError_t launch_nearest(const int32_t* dist, int n, int k, uint16_t* out, hipStream_t st, int* clear) {
    if (k <= 0) return hipSuccess;
    const int grid = (n + 3) / 4;
    if (n <= 16 * kWave)
        k_nearest<16><<<grid, 256, 0, st>>>(dist, n, k, out, clear);
    else if (n <= 32 * kWave)
        k_nearest<32><<<grid, 256, 0, st>>>(dist, n, k, out, clear);
    else if (n <= 64 * kWave)
        k_nearest<64><<<grid, 256, 0, st>>>(dist, n, k, out, clear);
    else
        k_nearest<0><<<grid, 256, 0, st>>>(dist, n, k, out, clear);
    return hipGetLastError();
}

hipError_t launch_nn_tour(const Views& v, const Shape& s, hipStream_t st) {
    // as many list entries per city as LDS holds (its static part aside)
    const int bits = nn_tour_bits(s.n), room = max_lds_per_block() - 256 - bits;
    int p = room > 0 ? room / (2 * s.n) : 0;
    if (p > s.cl) p = s.cl;
    if (p < s.cl && p >= 4) p &= ~3;
    const size_t lds = (size_t)bits + 2 * (size_t)p * s.n;
    if (lds > 64 * 1024) {
        const hipError_t e =
            hipFuncSetAttribute((const void*)k_nn_tour, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // (the waves past the first only scan rows: sixteen where rows are long)
    k_nn_tour<<<1, s.n >= 1024 ? 1024 : 256, lds, st>>>(v.dist, v.cand, s.cl, s.n, p, v.nn_tour, v.state);
    return hipGetLastError();
}

hipError_t launch_init_trails(const Views& v, const Shape& s, hipStream_t st) {
    k_init_state<<<1, 64, 0, st>>>(v.state, s.rho, s.n, s.pdec);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t count = s.pher == MMAS_PHER_DENSE ? (size_t)s.n * s.n : (size_t)s.n * s.cl;
    k_fill_tau<<<grid_for(count, 256), 256, 0, st>>>(v.tau, count, v.state);
    return hipGetLastError();
}

}  // namespace mmas
