// 2-opt on every ant's tour with neighbour lists and don't-look bits
// (Sec. 5.7, after Bentley): one workgroup per ant, tour, position, edge
// lengths and don't-look bits in LDS.
//
// The result is that of the sequential first-improvement search: cities are
// examined in index order, cyclically, skipping those whose don't-look bit is
// set, until every bit is set. For city a, the 2k candidate moves (successor
// direction then predecessor direction, neighbours by rank) are evaluated in
// parallel, one per lane; a move counts only while the first partial gain
// g1 = d(a, a') - d(a, c) is positive (it cannot grow with the rank, so this
// is the sequential "stop at the first g1 <= 0"); the lowest lane with a
// positive total gain is the move the sequential search would take. The move
// reverses the shorter of its two paths (the one starting next to a on a
// tie), its four end points get their bits cleared and a is examined again;
// a city without a move gets its bit set. Several cities are evaluated per
// round (see k_two_opt), which changes the speed and not the result.
#include "device.hpp"
#include "internal.hpp"

namespace mmas {
namespace {

constexpr int kMaxWaves = 16;
constexpr int kListCap = 64;  // list entries kept, one per lane of the first wave
// Cities examined in a round, at most: a move is found at the third one on
// average, and every distance read for one behind it is read again (2-opt of
// 64 ants on uniform instances of n = 1002 / 3795 / 18512 with 8, 8 and 16
// waves: 8 cities 1.35 / 5.68 / 33.5 ms, 16: 1.31 / 5.59 / 32.9, 24: 1.38 /
// 5.72 / 33.6, as many as fit 1.39 / 5.78 / 35.1).
constexpr int kExamine = 16;

// A wave's first move and what applying it takes: all of it is worked out by
// the lane that evaluates the move, beside its distance load.
struct alignas(16) Move {
    uint32_t aa1, cc1;  // the city a and its neighbour a1; c and c1 (low, high half)
    int dac, da1c1;     // the new edges' lengths
    uint32_t path;      // first and last position of the reversed path
    uint32_t m12, m3f;  // places of the end points a1, c, c1 merged into the next list; kFlag* from bit 16
    uint32_t found;     // half the path's length, the city's list index from bit 16; kNoMove: none
};
constexpr uint32_t kNoMove = 0xFFFFFFFFu;
// m3f from bit 16: predecessor direction, then the number of end points that
// count as active again, then the number merged (2 bits each)
constexpr int kFlagPred = 16, kFlagAgain = 17, kFlagMerged = 19;

// x + n if x < 0 (as x + n < 2^31, the smaller unsigned value is the one
// wanted), and x - n if x >= n
__device__ __forceinline__ int wrap_up(int x, int n) { return (int)min((uint32_t)x, (uint32_t)(x + n)); }
__device__ __forceinline__ int wrap_down(int x, int n) { return (int)min((uint32_t)x, (uint32_t)(x - n)); }

__device__ __forceinline__ uint32_t dlb_bit(const uint32_t* dlb, int x) { return (dlb[x >> 5] >> (x & 31)) & 1u; }

// The next `count` active cities (don't-look bit clear) from city a0,
// cyclically, into `list`; one wave. Entries in order: the word of a0 from
// bit a0&31, the following words, the word of a0 below bit a0&31; 64 words a
// pass, until `count` cities are listed.
__device__ void list_active(const uint32_t* dlb, int words, uint32_t lastmask, int a0, int count, uint16_t* list,
                            int lane) {
    const int w0 = a0 >> 5, b0 = a0 & 31;
    int found = 0;
    for (int base = 0; base <= words && found < count; base += kWave) {
        const int e = base + lane;
        uint32_t bits = 0u;
        int w = 0;
        if (e <= words) {
            uint32_t m;
            if (e == 0) {
                w = w0;
                m = 0xFFFFFFFFu << b0;
            } else if (e < words) {
                w = w0 + e;
                if (w >= words) w -= words;
                m = 0xFFFFFFFFu;
            } else {
                w = w0;
                m = b0 ? ((1u << b0) - 1u) : 0u;
            }
            if (w == words - 1) m &= lastmask;
            bits = ~dlb[w] & m;
        }
        const int cnt = __popc(bits);
        const int incl = wave_incl_scan(cnt, lane);
        int idx = found + incl - cnt;
        while (bits && idx < count) {
            list[idx++] = (uint16_t)(w * 32 + __ffs(bits) - 1);
            bits &= bits - 1u;
        }
        found += __builtin_amdgcn_readlane(incl, 63);
    }
}

// The 2-opt of one ant per workgroup. kLen: the tour's edge lengths are kept
// in LDS by position (len[p] = d(tour[p], tour[p+1])), so a move evaluation
// reads one distance from HBM instead of three.
//
// A round examines the first E entries of a list of the next active cities
// in cyclic index order (a group of 2k lanes per city, kExamine cities at
// most) against the current tour. The first of them (in that order) with an
// improving move is the city the sequential search reaches next with a move:
// the cities before it have none and get their bits set, its move is applied
// and it is examined again. Without a move all E get their bits set. Any
// prefix of the active cities in cyclic order from the cursor serves as the
// list, so the next list is the old one from the move's city (or from the
// first city not examined) on, with the end points that became active inside
// its range merged in; the don't-look bits are scanned again only when that
// list gets short.
//
// A round is one serial chain (one move: the next one depends on it), so its
// length bounds the kernel: list, positions, tour neighbours from LDS, then
// one distance from HBM; barrier; the winning move from LDS; barrier. All
// that the move's consequences need (path, places of its end points) is
// worked out by every lane beside the distance's load, the first wave then
// keeps the bits and the count, the second the list, the others reverse the
// path. In clock cycles a round at n = 3795 takes 1550 to the first barrier,
// 330 there, 980 of bookkeeping beside 740 of reversal; with those values
// derived by the first waves after the barrier, it was 1585, 363 and 1650
// beside 1140. An iteration of 64 ants, n = 3795: 8.48 -> 6.63 ms; n = 18512:
// 51.7 -> 42.9 ms (reversal 1955 -> 1437 cycles of a round there).
template <bool kLen>
__global__ __launch_bounds__(1024) void k_two_opt(Views vw, Shape s, const int32_t* __restrict__ nnd) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint16_t s_lists[2][kListCap];  // by round parity
    __shared__ int s_count[2];                  // entries of each list (0: the search has ended)
    __shared__ Move s_mv[kMaxWaves];            // each wave's first move
    __shared__ unsigned long long s_len;
    const int n = s.n, k = s.ls_nn;
    const int ant = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63;
    // wave-uniform values are read into scalar registers (readfirstlane), so
    // that the bookkeeping of a round takes scalar branches
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nthr = blockDim.x, nwaves = nthr >> 6;
    int gs = 1;
    while (gs < 2 * k) gs <<= 1;  // lanes per city (power of two <= 64)
    const int lg = __builtin_ctz(gs);
    const int E = min(nthr >> lg, kExamine);  // cities examined per round
    uint16_t* tour = reinterpret_cast<uint16_t*>(smem);
    uint16_t* pos = tour + n;
    const size_t tp_bytes = (4 * (size_t)n + 15) & ~(size_t)15;
    int32_t* elen = reinterpret_cast<int32_t*>(smem + tp_bytes);
    uint32_t* dlb = reinterpret_cast<uint32_t*>(smem + tp_bytes + (kLen ? 4 * (size_t)n : 0));
    const int words = (n + 31) >> 5;
    const uint32_t lastmask = (n & 31) ? ((1u << (n & 31)) - 1u) : 0xFFFFFFFFu;
    const int32_t* dist = vw.dist;
    const uint16_t* nn = vw.lsnn;
    uint16_t* gtour = vw.tours + (size_t)ant * n;
    // after a failed construction the tour may not be a permutation
    if (vw.state->flags & 8u) return;

    for (int i = t; i < n; i += nthr) {
        const uint16_t v = gtour[i];
        tour[i] = v;
        pos[v] = (uint16_t)i;
    }
    for (int w = t; w < words; w += nthr) dlb[w] = 0u;
    if (t == 0) s_len = 0ull;
    __syncthreads();
    if (kLen)
        for (int i = t; i < n; i += nthr) elen[i] = dist[(size_t)tour[i] * n + tour[i + 1 == n ? 0 : i + 1]];

    // Roles after a round's move is known: wave 0 sets and clears the
    // don't-look bits, counts the active cities and tops the next list up from
    // the bits, wave 1 makes the next list from the current one, the other
    // waves reverse the path (with fewer waves, wave 0 also makes the list, and
    // a single wave does everything).
    const int merge_wave = nwaves > 2 ? 1 : 0;
    const int rev_wave0 = nwaves > 2 ? 2 : nwaves - 1;
    int act = n;                    // active cities (kept by the first wave)
    int ca = -1, cc = 0, cdac = 0;  // this lane's last (city, neighbour, distance) from the lists
    // a list shorter than this is topped up from the bits
    const int refill = min(E, 8);
    // every round sets a bit or shortens the tour; the cap only guards
    // against a search that would not end
    const int max_rounds = 256 * n + 4096;
    int rounds = 0;
    // this lane's part of every round: its city's list entry, its neighbour's
    // rank and its direction (step to the tour neighbour, and the same step
    // around the end: the smaller unsigned sum is the position)
    const int g = t >> lg, rl = t & (gs - 1);
    const bool pd = rl >= k;
    const int rank = pd ? rl - k : rl;
    const int step = pd ? -1 : 1, step_wrap = pd ? n - 1 : 1 - n;
    if (wave == 0) {
        list_active(dlb, words, lastmask, 0, min(kListCap, n), s_lists[1], lane);
        if (lane == 0) s_count[1] = min(kListCap, n);
    }
    for (;;) {
        ++rounds;
        const int par = (int)(rounds & 1);
        const uint16_t* s_list = s_lists[par];

        __syncthreads();  // the list, the tour, positions, lengths and bits of this round
        // the list entries are read beside the count: one LDS round trip (the
        // compiler would read them behind the exit)
        int a_l = s_list[g < kListCap ? g : 0];
        int le_l = s_list[lane];
        int count = s_count[par];
        asm volatile("" : "+v"(a_l), "+v"(le_l), "+v"(count));
        count = __builtin_amdgcn_readfirstlane(count);
        if (count == 0) break;
        if (rounds > max_rounds) {
            if (t == 0) atomicOr(&vw.state->flags, 16u);
            return;
        }
        const int ev = min(count, E);
        const int le = lane < count ? le_l : 0;  // the list, one entry a lane
        // places of cities are cyclic distances from the first listed one
        // (the cities between the cursor and it are inactive)
        const int a0 = __builtin_amdgcn_readfirstlane(le_l);
        const int last = __builtin_amdgcn_readlane(le, count - 1);
        auto cyc = [&](int x) { return wrap_up(x - a0, n); };
        const int ql = cyc(last);

        // ---- evaluate every candidate move of the first ev listed cities ----
        bool ok = false;
        Move em;  // (only the lanes with a move fill it and use it)
        if (g < ev && rl < 2 * k) {
            const int a = a_l;
            if (a != ca) {  // the list often starts where the last one did
                cc = nn[(size_t)a * k + rank];
                cdac = nnd[(size_t)a * k + rank];
                ca = a;
            }
            const int c = cc, dac = cdac;
            // both ends' positions, then both tour neighbours and edge lengths
            const int pa = pos[a], pc = pos[c];
            const int pa1 = (int)min((uint32_t)(pa + step), (uint32_t)(pa + step_wrap));
            const int pc1 = (int)min((uint32_t)(pc + step), (uint32_t)(pc + step_wrap));
            const int a1 = tour[pa1], c1 = tour[pc1];
            const int64_t daa1 = kLen ? (int64_t)elen[pd ? pa1 : pa] : (int64_t)dist[(size_t)a * n + a1];
            const int32_t ecc1 = kLen ? elen[pd ? pc1 : pc] : 0;
            const int64_t g1 = daa1 - dac;
            if (g1 > 0 && c != a1 && c1 != a) {
                const int32_t dcc1 = kLen ? ecc1 : dist[(size_t)c * n + c1];
                const int32_t da1c1 = dist[(size_t)a1 * n + c1];
                // beside the distance's load: the end points' don't-look bits
                // and places, whether each counts as active again (inactive
                // before, or listed before a) and is merged into the next list
                // (inactive before and inside (a, last])
                const uint32_t w1 = dlb_bit(dlb, a1), w2 = dlb_bit(dlb, c), w3 = dlb_bit(dlb, c1);
                // the two paths the move may reverse (a1 and c1 sit next to a
                // and c); the shorter one, the first on a tie
                const int i1 = pd ? pa : pa1, j1 = pd ? pc1 : pc;  // a1..c or a..c1
                const int i2 = pd ? pc : pc1, j2 = pd ? pa1 : pa;  // c1..a or c..a1
                const int len1 = wrap_up(j1 - i1, n) + 1;
                const bool first = len1 <= n - len1;
                em.path = (uint32_t)(first ? i1 : i2) | (uint32_t)(first ? j1 : j2) << 16;
                em.found = (uint32_t)((first ? len1 : n - len1) >> 1) | (uint32_t)g << 16;
                const int qa = cyc(a), q1 = cyc(a1), q2 = cyc(c), q3 = cyc(c1);
                const bool b1 = w1 && q1 > qa && q1 <= ql;
                const bool b2 = w2 && q2 > qa && q2 <= ql;
                const bool b3 = w3 && q3 > qa && q3 <= ql;
                const uint32_t again = (w1 | (uint32_t)(q1 < qa)) + (w2 | (uint32_t)(q2 < qa)) + (w3 | (uint32_t)(q3 < qa));
                em.m12 = (uint32_t)(b1 ? q1 : n) | (uint32_t)(b2 ? q2 : n) << 16;
                em.m3f = (uint32_t)(b3 ? q3 : n) | (uint32_t)pd << kFlagPred | again << kFlagAgain |
                         ((uint32_t)b1 + (uint32_t)b2 + (uint32_t)b3) << kFlagMerged;
                em.aa1 = (uint32_t)a | (uint32_t)a1 << 16;
                em.cc1 = (uint32_t)c | (uint32_t)c1 << 16;
                // (kept here: the compiler would move all of it behind the load)
                asm volatile("" : "+v"(em.path), "+v"(em.found), "+v"(em.m12), "+v"(em.m3f), "+v"(em.aa1), "+v"(em.cc1));
                em.dac = dac;
                em.da1c1 = da1c1;
                ok = g1 + (int64_t)dcc1 - (int64_t)da1c1 > 0;
            }
        }
        // the lowest lane with a move: the wave's first city, its first move
        const uint64_t mask = __ballot(ok);
        if (mask == 0ull) {
            if (lane == 0) s_mv[wave].found = kNoMove;
        } else if (lane == __ffsll((unsigned long long)mask) - 1) {
            s_mv[wave] = em;
        }
        __syncthreads();
        // the first move over all waves: that of the first wave with one (the
        // waves' moves are read beside their flags, one a lane)
        Move wm = s_mv[lane & (kMaxWaves - 1)];
        // (read in one go: the compiler would read part of it in the branches)
        asm volatile("" : "+v"(wm.aa1), "+v"(wm.cc1), "+v"(wm.dac), "+v"(wm.da1c1), "+v"(wm.path), "+v"(wm.m12),
                     "+v"(wm.m3f), "+v"(wm.found));
        const uint64_t wmask = __ballot(lane < nwaves && wm.found != kNoMove);
        const bool moved = wmask != 0ull;
        const int bw = moved ? __ffsll((unsigned long long)wmask) - 1 : 0;
        const uint32_t found = __builtin_amdgcn_readlane(wm.found, bw);

        if (wave <= merge_wave) {
            const int gstar = moved ? (int)(found >> 16) : ev;  // the listed cities before it have no move
            const uint32_t aa1 = __builtin_amdgcn_readlane(wm.aa1, bw);
            const uint32_t cc1 = __builtin_amdgcn_readlane(wm.cc1, bw);
            const uint32_t m3f = moved ? __builtin_amdgcn_readlane(wm.m3f, bw) : 0u;
            const int merged = (int)(m3f >> kFlagMerged);
            // kept: the move's city (first) and the entries after it, or the
            // entries not examined; merged end points in cyclic order
            const int head = moved ? 1 : 0, keep0 = gstar + head;
            uint16_t* nl = s_lists[par ^ 1];
            const int ee = lane == 0 ? (int)(aa1 >> 16) : lane == 1 ? (int)(cc1 & 0xFFFFu) : (int)(cc1 >> 16);
            if (wave == merge_wave) {
                const bool keep = lane >= keep0 && lane < count;
                int idx = lane - gstar;
                if (merged) {
                    const uint32_t m12 = __builtin_amdgcn_readlane(wm.m12, bw);
                    const int m1 = (int)(m12 & 0xFFFFu), m2 = (int)(m12 >> 16), m3 = (int)(m3f & 0xFFFFu);
                    const int cx = cyc(le);
                    idx += (int)(m1 < cx) + (int)(m2 < cx) + (int)(m3 < cx);
                    // lanes 0-2: the place of merged end point a1, c, c1
                    const int r1 = __popcll(__ballot(keep && cx < m1));
                    const int r2 = __popcll(__ballot(keep && cx < m2));
                    const int r3 = __popcll(__ballot(keep && cx < m3));
                    const int mm = lane == 0 ? m1 : lane == 1 ? m2 : m3;
                    const int rr = lane == 0 ? r1 : lane == 1 ? r2 : r3;
                    const int ie = head + rr + (int)(m1 < mm) + (int)(m2 < mm) + (int)(m3 < mm);
                    if (lane < 3 && mm < n && ie < kListCap) nl[ie] = (uint16_t)ee;
                }
                // (the move's city is list entry gstar)
                if ((keep || (moved && lane == gstar)) && idx < kListCap) nl[idx] = (uint16_t)le;
            }
            if (wave == 0) {
                // the listed cities before the move's city lose their bits, the
                // end points are all active afterwards (a wave's LDS operations
                // complete in order)
                if (lane < gstar) atomicOr(&dlb[le >> 5], 1u << (le & 31));
                if (moved && lane < 3) atomicAnd(&dlb[ee >> 5], ~(1u << (ee & 31)));
                act = act - gstar + (int)((m3f >> kFlagAgain) & 3u);
                const int cap = min(kListCap, act);
                int len = min(cap, count - gstar + merged);
                if (len < cap && len < refill) {
                    // the next active cities after the last listed one
                    list_active(dlb, words, lastmask, last + 1 == n ? 0 : last + 1, cap - len, nl + len, lane);
                    len = cap;
                }
                if (lane == 0) s_count[par ^ 1] = len;
            }
        }
        if (moved && wave >= rev_wave0) {
            // reverse positions i..j of the tour and i..j-1 of the edge lengths:
            // pair q swaps tour[i+q] and tour[j-q], and elen[i+q] and
            // elen[j-1-q] (for even lengths the middle pair of the lengths is
            // one cell swapped with itself)
            const uint32_t path = __builtin_amdgcn_readlane(wm.path, bw);
            const int mi = (int)(path & 0xFFFFu), mj = (int)(path >> 16);
            const int half = (int)(found & 0xFFFFu);
            const int rt = t - rev_wave0 * kWave, rthr = nthr - rev_wave0 * kWave;
            for (int q = rt; q < half; q += rthr) {
                const int p = wrap_down(mi + q, n);
                const int r = wrap_up(mj - q, n);
                const int r1 = wrap_up(r - 1, n);
                const uint16_t tp = tour[p], tr = tour[r];
                int32_t ep = 0, er = 0;
                if (kLen) {
                    ep = elen[p];
                    er = elen[r1];
                }
                tour[p] = tr;
                tour[r] = tp;
                pos[tr] = (uint16_t)p;
                pos[tp] = (uint16_t)r;
                if (kLen) {
                    elen[p] = er;
                    elen[r1] = ep;
                }
            }
            if (kLen && rt == 0) {
                // the two new edges close the path: in successor direction the
                // city left of it is a (path from a1) or c (path from c1), and
                // {a, c} comes first; else it is a1 or c1
                const bool pd = (__builtin_amdgcn_readlane(wm.m3f, bw) >> kFlagPred) & 1u;
                const int dac = __builtin_amdgcn_readlane(wm.dac, bw), da1c1 = __builtin_amdgcn_readlane(wm.da1c1, bw);
                elen[wrap_up(mi - 1, n)] = pd ? da1c1 : dac;
                elen[mj] = pd ? dac : da1c1;
            }
        }
    }
    __syncthreads();
    // write back; the tour length from the final edges
    int64_t tl = 0;
    for (int i = t; i < n; i += nthr) {
        const uint16_t v = tour[i];
        gtour[i] = v;
        tl += kLen ? (int64_t)elen[i] : (int64_t)dist[(size_t)v * n + tour[i + 1 == n ? 0 : i + 1]];
    }
    tl = wave_sum_i64(tl);
    if (lane == 0) atomicAdd(&s_len, (unsigned long long)tl);
    __syncthreads();
    if (t == 0) vw.lengths[ant] = (int64_t)s_len;
}

// d(i, nn[i][r]) for the 2-opt neighbour lists
__global__ __launch_bounds__(256) void k_nn_dist(const int32_t* __restrict__ dist, const uint16_t* __restrict__ nn,
                                                 int n, int k, int32_t* __restrict__ out) {
    const size_t total = (size_t)n * k;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x)
        out[e] = dist[(e / k) * n + nn[e]];
}

}  // namespace

// dynamic LDS of the 2-opt kernel: tour and position (uint16), the edge
// lengths (int32) when `with_len`, and the don't-look bits
size_t two_opt_lds_bytes(const Shape& s, bool with_len) {
    return (size_t)((4 * s.n + 15) & ~15) + (with_len ? 4 * (size_t)s.n : 0) + 4 * (size_t)((s.n + 31) / 32);
}

hipError_t launch_two_opt_prepare(const Views& v, const Shape& s, int32_t* nnd, hipStream_t st) {
    if (s.ls_nn <= 0) return hipSuccess;
    const size_t total = (size_t)s.n * s.ls_nn;
    int g = (int)((total + 255) / 256);
    if (g > 65536) g = 65536;
    k_nn_dist<<<g, 256, 0, st>>>(v.dist, v.lsnn, s.n, s.ls_nn, nnd);
    return hipGetLastError();
}

hipError_t launch_two_opt(const Views& v, const Shape& s, const int32_t* nnd, hipStream_t st) {
    const bool with_len = two_opt_lds_bytes(s, true) + kTwoOptStaticLds <= (size_t)max_lds_per_block();
    const size_t lds = two_opt_lds_bytes(s, with_len);
    const void* kern = with_len ? (const void*)k_two_opt<true> : (const void*)k_two_opt<false>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    Views vv = v;
    Shape ss = s;
    void* args[] = {(void*)&vv, (void*)&ss, (void*)&nnd};
    // more waves shorten the reversal of long paths and cost a little more
    // at the barriers: 4 below 1024 cities, 8 below 8192, 16 from there (4, 8,
    // 16 waves: n = 500 664, 666, 682 us; 1002 1322, 1305, 1349; 3795 5.84,
    // 5.59, 5.66 ms; 18512 41.4, 33.9, 32.9)
    const int waves = s.two_opt_waves ? s.two_opt_waves : s.n < 1024 ? 4 : s.n < 8192 ? 8 : 16;
    return hipLaunchKernel(kern, dim3(s.ants), dim3(64 * waves), args, lds, st);
}

}  // namespace mmas
