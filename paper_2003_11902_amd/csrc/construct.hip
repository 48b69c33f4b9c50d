// Tour construction (the inner loops of Alg. 1): one ant per wave64.
//
// Each step selects the next city by weighted reservoir sampling (Alg. 4):
// every eligible city v draws u and gets the key ln(u) * (1 / w(cur, v)), the
// reciprocal of the weight computed ahead as Sec. 4.2.2 suggests; the wave
// keeps the largest key, the lowest city among equal keys. Eligible are the
// unvisited cities of the current city's candidate list (Sec. 4.3), one per
// lane, with w = choice_info along the list; when all are visited, every
// unvisited city with w = choice_info[cur][v] (dense trails) or
// tau_min^alpha * eta^beta (candidate-only trails).
//
// The visited set lives in LDS, as a bitmask (one bit per city) or as the
// compact tabu of Sec. 4.1 (one 16-bit entry per city plus the length L).
// Tours are gathered in a register (lane k % 64 holds step k) and stored 64
// cities at a time; tour lengths accumulate at those flushes.
#include <atomic>
#include <cstddef>
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace mmas {
namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;

// pointers typed with their address space, so that an LDS read and a global
// read of the same element are never folded into one generic (flat) load
template <class T>
using LdsPtr = __attribute__((address_space(3))) T*;
template <class T>
using GlbPtr = __attribute__((address_space(1))) T*;
// the LDS address `byte` as a pointer
template <class T>
__device__ __forceinline__ LdsPtr<T> lds_at(uint32_t byte) {
    return (LdsPtr<T>)(uintptr_t)byte;
}
__host__ __device__ inline int align16(int x) { return (x + 15) & ~15; }
// four consecutive row entries, aligned to one
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t i32x4_u __attribute__((ext_vector_type(4), aligned(4)));
constexpr size_t kDrawBytes = 4 * kWave * sizeof(float);  // candidate draws of the next steps
constexpr size_t kScratchBytes = 16;                       // per-ant counter of the fallback list

// x with lane kLane's value replaced by the wave-uniform v. (The compiler's own
// operation, by its name as there is no builtin for it: a vector instruction
// may read a scalar register two wait states after a lane read wrote it at the
// earliest, and the compiler cannot see to that inside inline assembly.)
extern "C" __device__ __attribute__((const)) int lane_write(int v, int lane, int x) __asm__("llvm.amdgcn.writelane.i32");
template <int kLane>
__device__ __forceinline__ int write_lane(int v, int x) {
    return lane_write(__builtin_amdgcn_readfirstlane(v), kLane, x);
}

// ---- tabu variants ---------------------------------------------------------

struct BitmaskTabu {
    uint32_t* bits;
    __device__ void attach(uint8_t* lds, int) { bits = reinterpret_cast<uint32_t*>(lds); }
    __device__ void init(uint8_t* lds, int n, int lane) {
        bits = reinterpret_cast<uint32_t*>(lds);
        const int words = (n + 31) >> 5;
        for (int w = lane; w < words; w += kWave) bits[w] = 0u;
    }
    __device__ __forceinline__ bool visited(uint32_t v) const { return (bits[v >> 5] >> (v & 31u)) & 1u; }
    // ~0 if city v is visited, else 0 (a signed bit-field extract)
    __device__ __forceinline__ uint32_t seen(uint32_t v) const {
        const uint32_t word = bits[__builtin_amdgcn_ubfe(v, 5u, 11u)];
        return (uint32_t)__builtin_amdgcn_sbfe((int)word, v, 1u);  // (the offset is taken mod 32)
    }
    __device__ __forceinline__ void mark(uint32_t v, int lane) {
        if (lane == 0) atomicOr(&bits[v >> 5], 1u << (v & 31u));
    }
};

// Compact tabu: entries[i] for i < L lists the unvisited cities; for i >= L,
// entries[i] is the position of city i if it was moved left, or n once city i
// is visited. City u is visited iff entries[u] > u.
// A mark needs two cells: the marked city's, which the step's visited test has
// read already (mark_at), and the last one of the left part, read ahead after
// the mark before (`tail`), so that a mark waits for no LDS read of its own.
struct CompactTabu {
    uint16_t* entries;
    int L;
    int n;
    uint32_t tail;  // entries[L - 1] (0 once L is 0)
    __device__ void attach(uint8_t* lds, int n_) {
        entries = reinterpret_cast<uint16_t*>(lds);
        n = n_;
        L = n_;
        tail = 0u;
    }
    __device__ void init(uint8_t* lds, int n_, int lane) {
        attach(lds, n_);
        for (int i = lane; i < n_; i += kWave) entries[i] = (uint16_t)i;
        tail = (uint32_t)(n_ - 1);
    }
    __device__ __forceinline__ bool visited(uint32_t v) const { return entries[v] > v; }
    __device__ __forceinline__ uint32_t cell(uint32_t v) const { return entries[v]; }
    __device__ __forceinline__ uint32_t seen(uint32_t v, uint32_t cell_v) const { return cell_v > v ? ~0u : 0u; }
    __device__ __forceinline__ const uint16_t* list() const { return entries; }  // the L unvisited cities
    // u and iu = entries[u] (the position of u in the left part) are
    // wave-uniform, and the whole wave comes here: lane 0 writes the cell at
    // iu, lane 1 the last entry's, the others the marked city's (once more
    // what lane 0 writes where u was not moved), so that no branch is taken
    __device__ __forceinline__ void mark_at(uint32_t u, int iu) {
        const int t = __builtin_amdgcn_readfirstlane((int)tail);
        L = L - 1;
        const bool end = iu == L;
        const int v0 = end ? n : t, v2 = (int)u != iu ? n : v0;
        const int at = write_lane<1>(end ? iu : t, write_lane<0>(iu, (int)u));
        const int val = write_lane<1>(end ? n : iu, write_lane<0>(v0, v2));
        entries[at] = (uint16_t)val;
        tail = entries[L > 0 ? L - 1 : 0];
    }
    __device__ __forceinline__ void mark(uint32_t u, int) {
        mark_at(u, __builtin_amdgcn_readfirstlane((int)entries[u]));
    }
};

// The list tabu of Sec. 4.1 (after Dawson and Stewart, and Uchida et al.):
// unv[0 .. L) lists the unvisited cities, idx[v] is the position of city v
// in unv; marking v swaps it with the last unvisited entry and shortens the
// list (reading C-18: the swap that the worked example of Sec. 4.1 needs), so
// city v is visited iff idx[v] >= L. 4n bytes. Marks as the compact tabu's.
struct ListTabu {
    uint16_t* unv;
    uint16_t* idx;
    int L;
    uint32_t tail;  // unv[L - 1]
    __device__ void attach(uint8_t* lds, int n_) {
        unv = reinterpret_cast<uint16_t*>(lds);
        idx = unv + n_;
        L = n_;
        tail = 0u;
    }
    __device__ void init(uint8_t* lds, int n_, int lane) {
        attach(lds, n_);
        for (int i = lane; i < n_; i += kWave) {
            unv[i] = (uint16_t)i;
            idx[i] = (uint16_t)i;
        }
        tail = (uint32_t)(n_ - 1);
    }
    __device__ __forceinline__ bool visited(uint32_t v) const { return (int)idx[v] >= L; }
    __device__ __forceinline__ uint32_t cell(uint32_t v) const { return idx[v]; }
    __device__ __forceinline__ uint32_t seen(uint32_t, uint32_t cell_v) const { return (int)cell_v >= L ? ~0u : 0u; }
    __device__ __forceinline__ const uint16_t* list() const { return unv; }
    // (idx lies n cells after unv: lanes 0 to 3 write one cell each, the others
    // lane 3's again)
    __device__ __forceinline__ void mark_at(uint32_t u, int iu) {
        const int last = __builtin_amdgcn_readfirstlane((int)tail);
        const int n = (int)(idx - unv);
        L = L - 1;
        int at = write_lane<0>(iu, n + (int)u);
        at = write_lane<1>(n + last, at);
        at = write_lane<2>(L, at);
        int val = write_lane<0>(last, L);
        val = write_lane<1>(iu, val);
        val = write_lane<2>((int)u, val);
        unv[at] = (uint16_t)val;
        tail = unv[L > 0 ? L - 1 : 0];
    }
    __device__ __forceinline__ void mark(uint32_t u, int) {
        mark_at(u, __builtin_amdgcn_readfirstlane((int)idx[u]));
    }
};

// ---- fallback weights --------------------------------------------------------

// The weights themselves (the roulette wheel sums them).
struct DenseWeight {
    const float* row;
    __device__ __forceinline__ float operator()(uint32_t v) const { return row[v]; }
};

struct CandWeight {
    const int32_t* drow;
    float tmin_a;
    int beta;
    __device__ __forceinline__ float operator()(uint32_t v) const {
        return tmin_a * heur_from_dist(drow[v], beta);
    }
};

template <int kTabu>
struct TabuOf;
template <>
struct TabuOf<MMAS_TABU_BITMASK> {
    using type = BitmaskTabu;
};
template <>
struct TabuOf<MMAS_TABU_COMPACT> {
    using type = CompactTabu;
};
template <>
struct TabuOf<MMAS_TABU_LIST> {
    using type = ListTabu;
};

__device__ __forceinline__ void keep_best(uint32_t code, uint32_t node, uint32_t& bcode, uint32_t& bnode) {
    if (code > bcode || (code == bcode && node < bnode)) {
        bcode = code;
        bnode = node;
    }
}

// Entries of the list a one-wave fallback over a bitmask tabu builds in LDS
// (unless the launch allows more): with more unvisited cities the fallback
// goes by draw blocks, so the ant's LDS does not grow with n.
constexpr int kListCap = 512;
__host__ __device__ inline int list_cap(int n, int asked) {
    return asked > 0 ? asked : (n < kListCap ? n : kListCap);
}

// A wave's best (key code, lowest city) packed so that the larger value is
// the better one; 0 if the wave saw no city.
__device__ __forceinline__ unsigned long long share_result(uint32_t bcode, uint32_t bnode) {
    const uint32_t bc = wave_max_u32<4>(bcode);
    if (bc == 0u) return 0ull;
    const uint64_t tied = __ballot(bcode == bc);
    uint32_t node;
    if (__popcll(tied) == 1)
        node = (uint32_t)__builtin_amdgcn_readlane((int)bnode, __ffsll((unsigned long long)tied) - 1);
    else
        node = wave_min_u32<4>(bcode == bc ? bnode : kNone);
    return ((unsigned long long)bc << 32) | (unsigned long long)(~node);
}

// Wave-uniform values that arrive in vector registers (the arguments of an
// outlined function) read back into scalar registers, so that the branches
// and loops over them are scalar.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ float uni(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
__device__ __forceinline__ uint64_t uni(uint64_t x) {
    return ((uint64_t)uni((uint32_t)(x >> 32)) << 32) | uni((uint32_t)x);
}


// A kernel's instance, read through the constant address space (scalar loads):
// an entry of the batch's array, or the first two arguments of a kernel that
// serves one colony. Rare paths read what they need from it again instead of
// keeping it in scalar registers all along.
using ItemPtr = const __attribute__((address_space(4))) BatchItem*;
// (the first two arguments of such a kernel, Views and Shape, are laid out as
// a BatchItem)
__device__ __forceinline__ ItemPtr kernel_item() { return (ItemPtr)__builtin_amdgcn_kernarg_segment_ptr(); }
__device__ __forceinline__ ItemPtr opaque(ItemPtr p) {
    asm volatile("" : "+s"(p));
    return p;
}

// What an all-city fallback of one ant needs, every value wave-uniform. The
// tabu is the bitmask's words, the compact tabu's entries or the list tabu's
// unv (idx follows at n); key factors are irow[v], the reciprocal of the
// weight (dense trails), or 1 / (tmin_a * eta(drow[v])^beta) (candidate-only
// trails). LDS and global pointers carry their address spaces (an outlined
// function would otherwise reach both through flat accesses).
struct Fallback {
    LdsPtr<const uint16_t> tabu;
    int L;  // unvisited cities
    int n, cl, beta;
    GlbPtr<const float> irow;
    GlbPtr<const int32_t> drow;
    float tmin_a;
    uint64_t seed;
    uint32_t it, ant, step;
};

// The fallback's arguments read back into scalar registers (an outlined
// function gets them in vector registers).
__device__ __forceinline__ Fallback uni(const Fallback& v) {
    Fallback q;
    q.tabu = lds_at<const uint16_t>(uni((uint32_t)(uintptr_t)v.tabu));
    q.L = uni(v.L);
    q.n = uni(v.n);
    q.cl = uni(v.cl);
    q.beta = uni(v.beta);
    q.irow = (GlbPtr<const float>)uni((uint64_t)(uintptr_t)v.irow);
    q.drow = (GlbPtr<const int32_t>)uni((uint64_t)(uintptr_t)v.drow);
    q.tmin_a = uni(v.tmin_a);
    q.seed = uni(v.seed);
    q.it = uni(v.it);
    q.ant = uni(v.ant);
    q.step = uni(v.step);
    return q;
}

template <int kTabu>
__device__ __forceinline__ bool fallback_seen(const Fallback& q, uint32_t v) {
    if constexpr (kTabu == MMAS_TABU_BITMASK)
        return (((LdsPtr<const uint32_t>)q.tabu)[v >> 5] >> (v & 31u)) & 1u;
    else if constexpr (kTabu == MMAS_TABU_COMPACT)
        return q.tabu[v] > v;
    else
        return (int)q.tabu[q.n + v] >= q.L;
}

// A fallback key is ln(u) times the reciprocal of the weight (Sec. 4.2.2): read
// from the dense matrix of reciprocals the update writes, or computed from the
// distance (trails kept along the candidate lists only: every other weight is
// tau_min^alpha * eta^beta).
template <int kPher>
__device__ __forceinline__ float exact_factor(const Fallback& q, uint32_t v) {
    if constexpr (kPher == MMAS_PHER_DENSE)
        return q.irow[v];
    else
        return 1.0f / (q.tmin_a * heur_from_dist(q.drow[v], q.beta));
}

// The exact fallback, for the near ties: city v draws slot cl + v, and the
// largest key (the lowest city among equal ones) wins. (Its registers count for
// every kernel that may call it: with the arguments in vector registers the
// candidate-only batches took 65 and lost the eighth wave of a SIMD.)
template <int kTabu, int kPher>
__device__ __attribute__((noinline)) uint32_t fallback_exact(Fallback qv, int lane) {
    const Fallback q = uni(qv);
    uint32_t bcode = 0u, bnode = kNone;
    for (int v0 = 0; v0 < q.n; v0 += kWave) {
        const uint32_t v = (uint32_t)(v0 + lane);
        if (v >= (uint32_t)q.n || fallback_seen<kTabu>(q, v)) continue;
        const uint32_t slot = (uint32_t)q.cl + v;
        const Words4 blk = draw_block(q.seed, q.it, q.ant, q.step, slot);
        const float key = log_u01(u01(pick_word(blk, slot & 3u))) * exact_factor<kPher>(q, v);
        keep_best(ord_key(key), v, bcode, bnode);
    }
    return wave_select<4>(bcode, bnode);
}

// A lane's two best approximate codes (device.hpp) and the best one's city.
struct NearBest {
    uint32_t m1 = 0u, m2 = 0u, node = 0u;
};

// The two largest of four codes (the second: a lane that holds two near the
// wave's best has a near tie of its own).
__device__ __forceinline__ void top_two(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t& m1,
                                        uint32_t& m2) {
    const uint32_t h01 = max(c0, c1), l01 = min(c0, c1), h23 = max(c2, c3), l23 = min(c2, c3);
    m1 = max(h01, h23);
    m2 = max(max(min(h01, h23), l01), l23);
}

// 1 / tmin_a, which the approximate factors of candidate-only trails share.
template <int kPher>
__device__ __forceinline__ float near_scale(const Fallback& q) {
    return kPher == MMAS_PHER_DENSE ? 0.0f : 1.0f / q.tmin_a;
}

// Approximate keys of an all-city fallback, one of two layouts; wave `part`
// of `parts` takes every parts-th round of 64.
//  - by draw blocks: a lane takes the block of slots 4b .. 4b+3, computes it
//    once and keys each of its cities that is unvisited (every city is looked
//    at, but a block serves four): about 85 instructions a round;
//  - by list entries (`list` holds the L unvisited cities): one Philox block
//    and one key per entry, about 58 instructions a round.
template <int kTabu, int kPher>
__device__ __forceinline__ void near_blocks(const Fallback& q, int part, int parts, int lane, NearBest& nb) {
    const int n = q.n, cl = q.cl;
    const float scale = near_scale<kPher>(q);
    const int b_lo = cl >> 2, b_hi = (cl + n - 1) >> 2;  // blocks holding slots cl .. cl + n - 1
    int best_b = 0;
    for (int b0 = b_lo + part * kWave; b0 <= b_hi; b0 += kWave * parts) {
        const int b = b0 + lane, o = 4 * b - cl;  // the block's cities: o .. o + 3
        uint32_t live[4];                         // ~0 for an unvisited city
        float f[4];
        // (the tabu and factor loads go out before the draws)
        if (4 * b0 >= cl && 4 * (b0 + kWave) - cl <= n) {
            // every block of the round lies inside: one read of the bitmask
            // and of the row for all four cities
            if constexpr (kTabu == MMAS_TABU_BITMASK) {
                const LdsPtr<const uint32_t> w = (LdsPtr<const uint32_t>)q.tabu + (o >> 5);
                // (the word after the bitmask is inside the ant's region)
                const uint32_t seen = __builtin_amdgcn_alignbit(w[1], w[0], (uint32_t)o & 31u);
#pragma unroll
                for (int j = 0; j < 4; ++j) live[j] = (uint32_t)((int)(~seen << (31 - j)) >> 31);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) live[j] = fallback_seen<kTabu>(q, (uint32_t)(o + j)) ? 0u : ~0u;
            }
            if constexpr (kPher == MMAS_PHER_DENSE) {
                const f32x4_u r = *(GlbPtr<const f32x4_u>)(q.irow + o);
#pragma unroll
                for (int j = 0; j < 4; ++j) f[j] = r[j];
            } else {
                const i32x4_u r = *(GlbPtr<const i32x4_u>)(q.drow + o);
#pragma unroll
                for (int j = 0; j < 4; ++j) f[j] = powi((float)r[j], q.beta) * scale;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool in = o + j >= 0 && o + j < n;
                const uint32_t v = in ? (uint32_t)(o + j) : 0u;
                live[j] = (in & !fallback_seen<kTabu>(q, v)) ? ~0u : 0u;
                f[j] = kPher == MMAS_PHER_DENSE ? q.irow[v] : powi((float)q.drow[v], q.beta) * scale;
            }
        }
        const Words4 blk = draw_block(q.seed, q.it, q.ant, q.step, (uint32_t)(4 * b));
        uint32_t code[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float key = log2_draw(blk.w[j]) * f[j];
            code[j] = ((~__float_as_uint(key) & ~3u) | (uint32_t)j) & live[j];
        }
        uint32_t t1, t2;
        top_two(code[0], code[1], code[2], code[3], t1, t2);
        nb.m2 = max(max(nb.m2, t2), min(nb.m1, t1));
        best_b = t1 > nb.m1 ? b : best_b;
        nb.m1 = max(nb.m1, t1);
    }
    nb.node = (uint32_t)(4 * best_b - cl) + (nb.m1 & 3u);
}

template <int kPher>
__device__ __forceinline__ void near_list(const Fallback& q, LdsPtr<const uint16_t> list, int part, int parts, int lane,
                                          NearBest& nb) {
    const float scale = near_scale<kPher>(q);
    const int L = q.L;
    // U rounds at once: the factor loads go out before the draws
    auto rounds = [&](auto u_tag, int base) {
        constexpr int U = decltype(u_tag)::value;
        uint32_t v[U];
        float f[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * parts * kWave + lane;
            ok[u] = i < L;
            v[u] = list[ok[u] ? i : 0];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            f[u] = kPher == MMAS_PHER_DENSE ? q.irow[v[u]] : powi((float)q.drow[v[u]], q.beta) * scale;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t slot = (uint32_t)q.cl + v[u];
            const Words4 blk = draw_block(q.seed, q.it, q.ant, q.step, slot);
            const float key = log2_draw(pick_word(blk, slot & 3u)) * f[u];
            const uint32_t code = ok[u] ? ~__float_as_uint(key) : 0u;
            nb.m2 = med3(nb.m1, nb.m2, code);
            nb.node = code > nb.m1 ? v[u] : nb.node;
            nb.m1 = max(nb.m1, code);
        }
    };
    int base = part * kWave;
    const int span = parts * kWave;
    for (; base + span < L; base += 2 * span) rounds(std::integral_constant<int, 2>{}, base);
    if (base < L) rounds(std::integral_constant<int, 1>{}, base);
}

// A wave's share of a fallback as one word, the larger the better: its best
// code, the city and (bit 0) whether the wave cannot tell its best for sure;
// 0 if it saw no city.
template <int kPher>
__device__ __forceinline__ unsigned long long near_share(const Fallback& q, const NearBest& nb) {
    constexpr uint32_t kM = kPher == MMAS_PHER_DENSE ? kNear : kNearPow;
    const uint32_t best = wave_max_bcast(nb.m1);
    if (best == 0u) return 0ull;
    const uint32_t near = near_code<kM>(best);
    const uint64_t tied = __ballot(nb.m1 >= near);
    bool clear = ((tied & (tied - 1)) == 0ull) & (__ballot(nb.m2 >= near) == 0ull);
    if (kPher == MMAS_PHER_CANDIDATES) clear &= (best >= kHuge) & (q.tmin_a <= 1.0f);
    const uint32_t node = (uint32_t)__builtin_amdgcn_readlane((int)nb.node, (int)__builtin_ctzll(tied));
    return ((unsigned long long)best << 32) | (unsigned long long)(node << 1) | (unsigned long long)(clear ? 0u : 1u);
}

// Part `part` of `parts` of a fallback whose tabu keeps the list of unvisited
// cities (compact, list): the cheaper layout by instruction count.
template <int kTabu, int kPher>
__device__ __forceinline__ unsigned long long near_part(const Fallback& q, int part, int parts, int lane) {
    static_assert(kTabu != MMAS_TABU_BITMASK, "the tabu keeps the list of unvisited cities");
    const int nb_ = ((q.cl + q.n - 1) >> 2) - (q.cl >> 2) + 1, span = kWave * parts;
    NearBest nb;
    if (85 * ((nb_ + span - 1) / span) < 58 * ((q.L + span - 1) / span))
        near_blocks<kTabu, kPher>(q, part, parts, lane, nb);
    else
        near_list<kPher>(q, q.tabu, part, parts, lane, nb);
    return near_share<kPher>(q, nb);
}

// The all-city fallback of one wave: by draw blocks or by list, the cheaper by
// instruction count (listing a bitmask's cities costs about 140); a bitmask's
// list must fit in `cap` entries at `list`. At n = 1002 a tour has about 35
// fallbacks over about 200 cities.
template <int kTabu, int kPher>
__device__ __forceinline__ uint32_t fallback_wave(Fallback q, LdsPtr<uint16_t> list, int cap, int lane) {
    constexpr bool kList = kTabu != MMAS_TABU_BITMASK;
    unsigned long long r;
    if constexpr (kList) {
        r = near_part<kTabu, kPher>(q, 0, 1, lane);
    } else {
        const int n = q.n;
        const int nblk = ((q.cl + n - 1) >> 2) - (q.cl >> 2) + 1;
        NearBest nb;
        if (q.L > cap || 85 * ((nblk + kWave - 1) / kWave) < 58 * ((q.L + kWave - 1) / kWave) + 140) {
            near_blocks<kTabu, kPher>(q, 0, 1, lane, nb);
        } else {
            // every unvisited city in ascending order, lane l taking 16-bit
            // halves l, l + 64, ... of the bitmask, so that a lane writes at
            // most 16 entries
            const int nh = (n + 15) >> 4;
            int L = 0;
            for (int h0 = 0; h0 < nh; h0 += kWave) {
                const int hi = h0 + lane;
                uint32_t fr = 0u;
                if (hi < nh) {
                    fr = ~(uint32_t)q.tabu[hi] & 0xFFFFu;
                    if (hi == nh - 1 && (n & 15)) fr &= (1u << (n & 15)) - 1u;
                }
                const int cnt = __popc(fr);
                const int incl = wave_incl_scan(cnt, lane);
                int p = L + incl - cnt;
                while (fr) {
                    const int b = __ffs(fr) - 1;
                    fr &= fr - 1u;
                    list[p++] = (uint16_t)(hi * 16 + b);
                }
                L += __builtin_amdgcn_readlane(incl, 63);
            }
            q.L = L;
            near_list<kPher>(q, list, 0, 1, lane, nb);
        }
        r = near_share<kPher>(q, nb);
    }
    if (__builtin_expect((r & 1ull) == 0ull && r != 0ull, 1)) return (uint32_t)r >> 1;
    return fallback_exact<kTabu, kPher>(q, lane);
}

// ... outlined (it is rare with a list, and one copy serves every step of the
// unrolled step loop).
template <int kTabu, int kPher>
__device__ __attribute__((noinline)) uint32_t fallback_lone(Fallback qv, LdsPtr<uint16_t> list_v, int cap_v, int lane) {
    return fallback_wave<kTabu, kPher>(uni(qv), lds_at<uint16_t>(uni((uint32_t)(uintptr_t)list_v)), uni(cap_v), lane);
}

// The exact choice of a candidate step whose approximate keys nearly tie:
// lane r holds rank r (city `node`, factor w, `live` ~0 or 0) of the list of
// the ant that its half (or the whole wave) serves, and draws slot r. Returns
// this lane's exact code.
__device__ __attribute__((noinline)) uint32_t step_exact_code(uint64_t seed, uint32_t it, uint32_t ant, uint32_t k,
                                                              uint32_t rank, float w, uint32_t live) {
    const Words4 blk = draw_block(seed, it, ant, k, rank);
    const float key = log_u01(u01(pick_word(blk, rank & 3u))) * w;
    return ~__float_as_uint(key) & live;
}

// ---- several waves per ant: the fallback shared by the workgroup ----------

// What the leading wave (the one taking the steps) hands to the helper waves
// of its workgroup for a fallback, and their per-wave results.
struct __align__(16) WideStep {
    int k;               // the step that needs the fallback
    uint32_t cur;        // current city
    int L;               // unvisited count
    int stop;            // the tour is done: every wave leaves
};
// Instructions of one wave for gathering a bitmask's cities in a workgroup
// (the words' bits, an LDS atomic and a barrier), against keying rounds.
constexpr int kGatherCost = 300;

struct WideLds {
    WideStep step;       // written by the leading wave before the first barrier
                         // of a fallback, read by all after it
    uint32_t counter;    // bitmask tabu: list fill counter
    unsigned long long res[16];  // per wave: its near_share
};

// The unvisited cities of a bitmask tabu gathered by the whole workgroup
// (thread t takes words t, t + threads, ...): a wave places its words' cities
// by a prefix sum of their counts and claims room for all of them with one
// LDS atomic; `counter` is 0 on entry.
__device__ void gather_unvisited_block(const BitmaskTabu& tabu, int n, uint16_t* list, uint32_t* counter) {
    const int words = (n + 31) >> 5;
    const int lane = (int)(threadIdx.x & 63);
    for (int w0 = (int)(threadIdx.x & ~63u); w0 < words; w0 += (int)blockDim.x) {
        const int wi = w0 + lane;
        uint32_t fr = 0u;
        if (wi < words) {
            fr = ~tabu.bits[wi];
            if (wi == words - 1 && (n & 31)) fr &= (1u << (n & 31)) - 1u;
        }
        const int cnt = __popc(fr);
        const int incl = wave_incl_scan(cnt, lane);
        const int tot = __builtin_amdgcn_readlane(incl, 63);
        if (tot == 0) continue;
        uint32_t base = 0u;
        if (lane == 0) base = atomicAdd(counter, (uint32_t)tot);
        int p = __builtin_amdgcn_readfirstlane((int)base) + incl - cnt;
        while (fr) {
            const int b = __ffs(fr) - 1;
            fr &= fr - 1u;
            list[p++] = (uint16_t)(wi * 32 + b);
        }
    }
}


// LDS layout of one workgroup: the candidate table of cities 0..R-1 (ids,
// then choice_info), then one region per ant (its draws, its tabu and, for
// the bitmask, room to list the unvisited cities during a fallback).
struct Lds {
    int rows;          // R: rows of the candidate table held in LDS
    int table_bytes;   // bytes of the table part (16-aligned)
    int per_ant;       // bytes of one ant's region
};

// The whole workgroup copies the first R rows of the candidate table (ids,
// then the reciprocals of choice_info) into LDS; the caller synchronises.
__device__ void stage_table(const Views& vw, int cl, int R, uint16_t* tcand, float* tchc) {
    const int ne = R * cl;
    for (int e = threadIdx.x; e < ne; e += blockDim.x) {
        tcand[e] = vw.cand[e];
        tchc[e] = vw.chc_inv[e];
    }
}

// The arguments of an all-city fallback at step k from city cur with L
// unvisited cities, over `tabu` (the bitmask's words, or the other tabus' list).
template <int kPher>
__device__ __forceinline__ Fallback fallback_args(ItemPtr item, uint32_t it, uint32_t ant, int k, uint32_t cur, int L,
                                                  LdsPtr<const void> tabu, float tmin_a) {
    Fallback q;
    const int n = item->s.n;
    // (C-style casts: the only casts that change the address space)
    q.tabu = (LdsPtr<const uint16_t>)tabu;
    q.L = L;
    q.n = n;
    q.cl = item->s.cl;
    q.beta = item->s.beta;
    q.irow = kPher == MMAS_PHER_DENSE ? (GlbPtr<const float>)(item->v.choice_inv + (size_t)cur * n) : nullptr;
    q.drow = kPher == MMAS_PHER_DENSE ? nullptr : (GlbPtr<const int32_t>)(item->v.dist + (size_t)cur * n);
    q.tmin_a = tmin_a;
    q.seed = item->s.seed;
    q.it = it;
    q.ant = ant;
    q.step = (uint32_t)k;
    return q;
}
__device__ __forceinline__ LdsPtr<const void> fallback_tabu(const BitmaskTabu& t) { return (LdsPtr<const void>)t.bits; }
__device__ __forceinline__ LdsPtr<const void> fallback_tabu(const CompactTabu& t) { return (LdsPtr<const void>)t.entries; }
__device__ __forceinline__ LdsPtr<const void> fallback_tabu(const ListTabu& t) { return (LdsPtr<const void>)t.unv; }

// One wave's share of a workgroup-wide fallback at step k from city fcur
// (near_share). A bitmask's unvisited cities are gathered by the whole
// workgroup first, with a barrier, unless keying by draw blocks is cheaper.
template <int kTabu, int kPher, class T>
__device__ unsigned long long wide_share(ItemPtr item, uint32_t it, int ant, int k, uint32_t fcur, int L, T& tabu,
                                         uint16_t* ulist, WideLds* wl, float tmin_a, int lane, int wv, int nw) {
    Fallback q = fallback_args<kPher>(item, it, (uint32_t)ant, k, fcur, L, fallback_tabu(tabu), tmin_a);
    if constexpr (kTabu == MMAS_TABU_BITMASK) {
        NearBest nb;
        const int nblk = ((q.cl + q.n - 1) >> 2) - (q.cl >> 2) + 1, span = kWave * nw;
        if (85 * ((nblk + span - 1) / span) < 58 * ((L + span - 1) / span) + kGatherCost) {
            near_blocks<kTabu, kPher>(q, wv, nw, lane, nb);
        } else {
            gather_unvisited_block(tabu, q.n, ulist, &wl->counter);
            __syncthreads();
            q.L = __builtin_amdgcn_readfirstlane((int)wl->counter);
            near_list<kPher>(q, (LdsPtr<const uint16_t>)ulist, wv, nw, lane, nb);
        }
        return near_share<kPher>(q, nb);
    } else {
        return near_part<kTabu, kPher>(q, wv, nw, lane);
    }
}

// The helper waves of a workgroup-wide ant: they wait at the barrier until
// the leading wave posts a fallback (or the end of its tour), key their share
// and post their best, so the steps without a fallback need no barrier.
template <int kTabu, int kPher>
__device__ __forceinline__ void wide_helpers(ItemPtr item, uint32_t it, int ant, int lane, uint8_t* region, WideLds* wl,
                                             int wv, int nw) {
    const int n = item->s.n;
    typename TabuOf<kTabu>::type tabu;
    tabu.attach(region + kDrawBytes + kScratchBytes, n);
    uint16_t* ulist = reinterpret_cast<uint16_t*>(region + kDrawBytes + kScratchBytes + align16(4 * ((n + 31) / 32)));
    float tmin_a = 0.0f;
    if (kPher == MMAS_PHER_CANDIDATES) tmin_a = powi(item->v.state->tau_min, item->s.alpha);
    for (;;) {
        __syncthreads();  // a posted fallback, or the end
        const WideStep st = wl->step;
        if (__builtin_amdgcn_readfirstlane(st.stop)) return;
        const unsigned long long mine =
            wide_share<kTabu, kPher>(item, it, ant, __builtin_amdgcn_readfirstlane(st.k),
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)st.cur),
                                     __builtin_amdgcn_readfirstlane(st.L), tabu, ulist, wl, tmin_a, lane, wv, nw);
        if (lane == 0) wl->res[wv] = mine;
        __syncthreads();  // the results (read by the leading wave)
    }
}

// The leading wave's side of a workgroup-wide fallback at step k from city
// cur: posts it, keys its share with the helpers, and takes the best over
// the waves (a near tie it settles by the exact keys alone); kNone if none.
template <int kTabu, int kPher, class T>
__device__ uint32_t wide_lead_fallback(ItemPtr item, uint32_t it, int ant, int k, uint32_t cur, T& tabu,
                                       uint16_t* ulist, WideLds* wl, float tmin_a, int lane, int nw) {
    const int L = item->s.n - k;  // unvisited cities
    if (lane == 0) {
        WideStep st;
        st.k = k;
        st.cur = cur;
        st.L = L;
        st.stop = 0;
        wl->step = st;
        if constexpr (kTabu == MMAS_TABU_BITMASK) wl->counter = 0u;
    }
    __syncthreads();
    const unsigned long long mine = wide_share<kTabu, kPher>(item, it, ant, k, cur, L, tabu, ulist, wl, tmin_a, lane, 0, nw);
    if (lane == 0) wl->res[0] = mine;
    __syncthreads();
    // (the record, the counter and the list are read before the second
    // barrier; res is written again only after the next fallback's first)
    const unsigned long long r = lane < nw ? wl->res[lane] : 0ull;
    constexpr uint32_t kM = kPher == MMAS_PHER_DENSE ? kNear : kNearPow;
    const uint32_t hi = (uint32_t)(r >> 32), lo = (uint32_t)r;
    const uint32_t near = near_code<kM>(wave_max_u32<2>(hi));
    const uint64_t tied = __ballot(hi >= near);
    if (__builtin_expect(__popcll(tied) == 1, 1)) {
        const uint32_t pick = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)__builtin_ctzll(tied));
        if (__builtin_expect((pick & 1u) == 0u, 1)) return pick >> 1;
    }
    return fallback_exact<kTabu, kPher>(
        fallback_args<kPher>(item, it, (uint32_t)ant, k, cur, L, fallback_tabu(tabu), tmin_a), lane);
}

// The end of the leading wave's tour: the helpers leave.
__device__ void wide_lead_end(WideLds* wl, int lane) {
    if (lane == 0) {
        WideStep st;
        st.k = 0;
        st.cur = 0u;
        st.L = 0;
        st.stop = 1;
        wl->step = st;
    }
    __syncthreads();
}

// ---- the draw helper of a single-colony ant --------------------------------
//
// A second wave per ant computes the draws (Philox blocks and logarithms) of
// each group of S = 64 / G steps into one of two LDS buffers, a group ahead
// of the ant's wave, which then only reads them. Two counters in LDS hand the
// buffers over: the helper writes group g once group g - 2 is read. Waits are
// bounded: past the limit the ant's wave flags the tour (state flag 32) and
// goes on, and the helper leaves, so no wave can wait for ever. Both waves
// must read the counter the other writes through lds_get (a volatile LDS
// read) and write their own through lds_put. (Sharing the all-city fallbacks
// with the helper pays for no tabu any more: at n = 1002 the compact tabu
// takes 338 us a construction with it and 329 without, the bitmask 297 an
// iteration with and 287 without. Nor do approximate logarithms from the
// helper: the ant's chain then ends in two more instructions, 285 -> 294 us.)
struct HelpLds {
    int made;    // draw groups written (helper)
    int read;    // draw groups read (ant's wave)
    int pad[2];  // (to 16 bytes)
};
static_assert(sizeof(HelpLds) == 16, "cleared by one store");
constexpr size_t kHelpBytes = kDrawBytes + sizeof(HelpLds);  // second draw buffer, then the counters
constexpr int kHelpSpins = 1 << 24;                          // sleeps of 64 clocks before a wait gives up

__device__ __forceinline__ int lds_get(const int* c) {
    return __builtin_amdgcn_readfirstlane(*(LdsPtr<volatile const int>)c);
}
__device__ __forceinline__ void lds_put(int* c, int v) {
    asm volatile("" ::: "memory");
    *(LdsPtr<volatile int>)c = v;
}

// waits until the LDS counter c reaches `want`; false if it gave up
__device__ __forceinline__ bool wait_count(const int* c, int want) {
    for (int spins = 0; spins < kHelpSpins; ++spins) {
        if (lds_get(c) >= want) {
            asm volatile("" ::: "memory");
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

// The helper wave of ant `ant`: `region` is the ant's region (draw buffer 0
// at its start), `help` the helper's part (draw buffer 1, then the HelpLds).
template <int kG>
__device__ __forceinline__ void draw_helper(ItemPtr item, uint32_t it, int ant, int lane, uint8_t* region,
                                            uint8_t* help) {
    constexpr int gsh = kG == 1 ? 0 : kG == 2 ? 1 : kG == 4 ? 2 : kG == 8 ? 3 : 4;
    constexpr int S = kWave >> gsh;
    const int n = item->s.n;
    const uint64_t seed = item->s.seed;
    float* buf0 = reinterpret_cast<float*>(region);
    float* buf1 = reinterpret_cast<float*>(help);
    HelpLds* h = reinterpret_cast<HelpLds*>(help + kDrawBytes);
    const int groups = (n + S - 1) / S;
    for (int g = 0; g < groups; ++g) {
        const Words4 b = draw_block(seed, it, (uint32_t)ant, (uint32_t)(g * S + (lane >> gsh)),
                                    (uint32_t)(4 * (lane & (kG - 1))));
        float4 lv;
        lv.x = log_u01(u01(b.w[0]));
        lv.y = log_u01(u01(b.w[1]));
        lv.z = log_u01(u01(b.w[2]));
        lv.w = log_u01(u01(b.w[3]));
        // (computed before the wait)
        asm volatile("" : "+v"(lv.x), "+v"(lv.y), "+v"(lv.z), "+v"(lv.w));
        // the buffer of group g held group g - 2
        if (g >= 2 && !wait_count(&h->read, g - 1)) return;
        *reinterpret_cast<float4*>(((g & 1) ? buf1 : buf0) + 4 * lane) = lv;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the draws are in LDS before the count
        lds_put(&h->made, g + 1);
    }
}

// One ant's tour (one wave64, the batched kernel's step): start city, n - 1
// selection steps, tour and length stores. `region` is the ant's LDS region;
// rows 0..R-1 of the candidate table are in LDS at tcand / tchc.
template <int kTabu, int kPher>
__device__ __forceinline__ void construct_ant(ItemPtr item, uint32_t it, int ant, int lane, uint8_t* region,
                                              const uint16_t* tcand, const float* tchc, int R) {
    const int n = item->s.n, cl = item->s.cl;
    const uint64_t seed = item->s.seed;

    // per-ant LDS: the draws of the next steps (256 floats), then the tabu
    float* lnbuf = reinterpret_cast<float*>(region);
    typename TabuOf<kTabu>::type tabu;
    tabu.init(region + kDrawBytes + kScratchBytes, n, lane);
    uint16_t* ulist = reinterpret_cast<uint16_t*>(region + kDrawBytes + kScratchBytes + align16(4 * ((n + 31) / 32)));

    float tmin_a = 0.0f;
    if (kPher == MMAS_PHER_CANDIDATES) tmin_a = powi(item->v.state->tau_min, item->s.alpha);
    // (C-style casts: the only casts that change the address space)
    const LdsPtr<const uint16_t> lds_cand = (LdsPtr<const uint16_t>)tcand;
    const LdsPtr<const float> lds_chc = (LdsPtr<const float>)tchc;
    const GlbPtr<const uint16_t> glb_cand = (GlbPtr<const uint16_t>)item->v.cand;
    const GlbPtr<const float> glb_chc = (GlbPtr<const float>)item->v.chc_inv;  // reciprocals

    // start city: floor(x * n / 2^32) of draw (step 0, slot 0)
    const uint32_t x0 = draw_block(seed, it, (uint32_t)ant, 0u, 0u).w[0];
    const uint32_t start = (uint32_t)(((uint64_t)x0 * (uint64_t)n) >> 32);
    tabu.mark(start, lane);

    // Candidate draws are generated ahead, S steps at a time: lane l computes
    // the Philox block of step k + l/G and slots 4(l%G)..4(l%G)+3 and stores
    // their logarithms at lnbuf[4l..4l+3]; step k + j then reads slot r at
    // lnbuf[4jG + r]. G = 4-slot groups per step (a power of two), S = 64/G.
    const int gsh = cl <= 4 ? 0 : cl <= 8 ? 1 : cl <= 16 ? 2 : cl <= 32 ? 3 : 4;
    const int G = 1 << gsh;
    const int S = kWave >> gsh;

    uint16_t* tour_out = item->v.tours + (size_t)ant * n;
    const int32_t* dist = item->v.dist;
    uint32_t tbuf = start;   // lane (k & 63) holds the city of step k
    uint32_t prev_last = 0;  // last city of the previous 64-step chunk
    int64_t len = 0;
    int64_t fb_steps = 0, fb_nodes = 0;
    uint32_t cur = start;

    for (int k = 1; k < n; ++k) {
        uint32_t next = kNone;
        if (cl > 0) {
            // candidate phase: lane r holds rank r of cur's list
            // every lane loads a valid entry (lanes past the list repeat the
            // last one and get no key); the row comes from LDS or from global
            // memory through separate, address-space-typed loads
            uint32_t node;
            float w;
            const int cs = __builtin_amdgcn_readfirstlane((int)cur);
            const int e = cs * cl + (lane < cl ? lane : cl - 1);
            if (cs < R) {
                node = lds_cand[e];
                w = lds_chc[e];
            } else {
                node = glb_cand[e];
                w = glb_chc[e];
            }
            const int j = (k - 1) & (S - 1);
            if (j == 0) {
                // (steps past n - 1 draw values nobody reads; no lane is masked)
                const int ks = k + (lane >> gsh);
                const Words4 b = draw_block(seed, it, (uint32_t)ant, (uint32_t)ks, (uint32_t)(4 * (lane & (G - 1))));
                float4 lv;
                lv.x = log2_draw(b.w[0]);
                lv.y = log2_draw(b.w[1]);
                lv.z = log2_draw(b.w[2]);
                lv.w = log2_draw(b.w[3]);
                *reinterpret_cast<float4*>(lnbuf + 4 * lane) = lv;
            }
            // branch-free: every lane of the list computes its key; visited
            // cities and lanes past the list contribute no key
            const float lnu = lnbuf[4 * j * G + (lane & (4 * G - 1))];
            // the visited-bit load is issued first, so that the product overlaps it
            const bool seen = tabu.visited(node);
            float key = lnu * w;  // (w holds 1 / choice_info)
            asm volatile("" : "+v"(key));
            const bool live = (lane < cl) & !seen;  // no short circuit: no exec mask
            // (approximate keys: device.hpp)
            const uint32_t code = live ? ~__float_as_uint(key) : 0u;
            // (all four rows even for cl <= 32: lanes past the list hold no key,
            // and one code path is faster than two)
            const uint32_t best = wave_max_u32<4>(code);
            if (best != 0u) {
                const uint64_t tied = __ballot(code >= near_code(best));
                next = (uint32_t)__builtin_amdgcn_readlane((int)node, (int)__builtin_ctzll(tied));
                if (__builtin_expect((tied & (tied - 1)) != 0ull, 0)) {
                    const uint32_t c = step_exact_code(seed, it, (uint32_t)ant, (uint32_t)k, (uint32_t)lane, w,
                                                       live ? ~0u : 0u);
                    const uint32_t top = wave_max_u32<4>(c);
                    next = wave_min_u32<4>(c == top ? node : kNone);
                }
            }
        }
        if (next == kNone) {
            fb_steps += 1;
            fb_nodes += n - k;
            next = fallback_lone<kTabu, kPher>(
                fallback_args<kPher>(opaque(item), it, (uint32_t)ant, k, cur, n - k, fallback_tabu(tabu), tmin_a),
                (LdsPtr<uint16_t>)ulist, list_cap(n, item->s.list_cap), lane);
        }
        next = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
        if (next >= (uint32_t)n) {
            // unreachable with a validated instance (some unvisited city always
            // has a key); report it instead of indexing out of bounds
            if (lane == 0) atomicOr(&item->v.state->flags, 8u);
            break;
        }
        tabu.mark(next, lane);
        const int slot = k & 63;
        if (lane == slot) tbuf = next;
        cur = next;
        if (slot == 63 || k == n - 1) {
            // flush the chunk of steps k0 .. k; lane l holds step k0 + l
            const int k0 = k - slot;
            const uint32_t prev = __shfl_up(tbuf, 1);
            if (lane <= slot) {
                tour_out[k0 + lane] = (uint16_t)tbuf;
                // edge entering step k0 + l (none for step 0)
                const uint32_t from = lane == 0 ? prev_last : prev;
                if (k0 + lane > 0) len += dist[(size_t)from * n + tbuf];
            }
            prev_last = (uint32_t)__builtin_amdgcn_readlane((int)tbuf, slot);
        }
    }
    if (lane == 0) len += dist[(size_t)cur * n + start];  // closing edge
    len = wave_sum_i64(len);
    if (lane == 0) {
        item->v.lengths[ant] = len;
        item->v.fallback[ant] = fb_steps;
        item->v.fallback[item->s.ants + ant] = fb_nodes;
    }
}

// One ant per wave64 for the single colony, where every wave sits alone on
// its SIMD and the time per step is the length of the step's instruction
// chain. The same selection as construct_ant, laid out so that the chain
// stays short: the current and the next city are wave-uniform (scalar
// registers and scalar branches, no exec-mask bookkeeping around the step);
// the steps run in groups of S (one draw generation per group, no per-step
// test for it) inside chunks of 64 (one tour flush per chunk); the visited
// test folds into the key code as a mask; and for cl <= 32 (kRows = 2) the
// argmax reduces only the two rows that hold the list.
// kWide: the wave leads a workgroup whose other waves share its fallbacks
// (wide_helpers), nw waves in all. kHelp (kG > 0): a draw helper wave
// (draw_helper) fills the draw buffers; `help` is its part of the region
// (second buffer, counters).
template <int kTabu, int kPher, int kRows, int kG, bool kWide = false, bool kHelp = false>
__device__ __forceinline__ void construct_lone(ItemPtr item, uint32_t it, int ant, int lane, uint8_t* region,
                                               const uint16_t* tcand, const float* tchc, int R, WideLds* wl = nullptr,
                                               int nw = 1, uint8_t* help = nullptr) {
    // the draws' logarithms: approximate where this wave computes them, exact
    // from the draw helper (whose time is not on the ant's chain)
    constexpr bool kApprox = !kHelp;
    const int n = item->s.n, cl = item->s.cl;
    const uint64_t seed = item->s.seed;
    float* lnbuf = reinterpret_cast<float*>(region);
    typename TabuOf<kTabu>::type tabu;
    tabu.init(region + kDrawBytes + kScratchBytes, n, lane);
    uint16_t* ulist = reinterpret_cast<uint16_t*>(region + kDrawBytes + kScratchBytes + align16(4 * ((n + 31) / 32)));

    float tmin_a = 0.0f;
    if (kPher == MMAS_PHER_CANDIDATES) tmin_a = powi(item->v.state->tau_min, item->s.alpha);
    const LdsPtr<const uint16_t> lds_cand = (LdsPtr<const uint16_t>)tcand;
    const LdsPtr<const float> lds_chc = (LdsPtr<const float>)tchc;
    const GlbPtr<const uint16_t> glb_cand = (GlbPtr<const uint16_t>)item->v.cand;
    const GlbPtr<const float> glb_chc = (GlbPtr<const float>)item->v.chc_inv;  // reciprocals
    LdsPtr<const float> lds_ln = (LdsPtr<const float>)lnbuf;

    const uint32_t x0 = draw_block(seed, it, (uint32_t)ant, 0u, 0u).w[0];
    const int start = __builtin_amdgcn_readfirstlane((int)(((uint64_t)x0 * (uint64_t)n) >> 32));
    tabu.mark((uint32_t)start, lane);

    // Draws ahead: G 4-slot groups per step, S = 64 / G steps per generation.
    // The generation for the group of steps k0 .. k0 + S - 1 (k0 a multiple
    // of S; step 0 is the start and reads none) has lane l compute the Philox
    // block of step k0 + l / G, slots 4(l % G) .. 4(l % G) + 3, and store
    // their logarithms at lnbuf[4l .. 4l + 3]; step k0 + j reads slot r at
    // lnbuf[4jG + r].
    // (kG > 0: G fixed at compile time, with the draws pipelined below)
    const int gsh = kG == 1 ? 0 : kG == 2 ? 1 : kG == 4 ? 2 : kG == 8 ? 3 : kG == 16 ? 4
                  : cl <= 4 ? 0 : cl <= 8 ? 1 : cl <= 16 ? 2 : cl <= 32 ? 3 : 4;
    const int G = 1 << gsh;
    const int S = kWave >> gsh;
    const int lr = lane < cl ? lane : cl - 1;       // lanes past the list repeat the last entry
    uint32_t lane_ok = lane < cl ? ~0u : 0u;        // ... and never hold a key
    const int ln_lane = lane & (4 * G - 1);
    const uint32_t cells = (uint32_t)(uintptr_t)(LdsPtr<uint8_t>)region + (uint32_t)(kDrawBytes + kScratchBytes);
    // bitmask marks: LDS byte address of each lane's OR (see below)
    uint32_t mark_mask = lane == 0 ? ~0u : 0u;
    uint32_t mark_base = (uint32_t)(uintptr_t)(LdsPtr<uint8_t>)region +
                         (lane == 0 ? (uint32_t)(kDrawBytes + kScratchBytes) : 4u * (uint32_t)lane);
    // (opaque to the compiler, which would otherwise turn the arithmetic
    // below back into lane-0 selects)
    asm volatile("" : "+v"(mark_mask), "+v"(mark_base), "+v"(lane_ok));

    uint16_t* tour_out = item->v.tours + (size_t)ant * n;
    const int32_t* dist = item->v.dist;
    uint32_t tbuf = (uint32_t)start;  // lane (k & 63) holds the city of step k
    uint32_t prev_last = 0;           // city of the last step of the previous chunk
    int64_t len = 0;
    int64_t fb_steps = 0, fb_nodes = 0;
    int cur = start;
    bool bad = false;
    bool bad_help = false;  // a wait for the draw helper gave up
    HelpLds* hl = kHelp ? reinterpret_cast<HelpLds*>(help + kDrawBytes) : nullptr;

    // the all-city fallback of step k from city cur (rare with a list)
    auto fallback = [&](int k) -> uint32_t {
        // (k laundered so that n - k is not kept as a 64-bit induction
        // variable on every step)
        int kk = k;
        if constexpr (kWide)
            kk = __builtin_amdgcn_readfirstlane(kk);
        else
            asm volatile("" : "+s"(kk));
        fb_steps += 1;
        fb_nodes += n - kk;
        uint32_t pick;
        if constexpr (kWide) {
            pick = wide_lead_fallback<kTabu, kPher>(opaque(item), it, ant, kk, (uint32_t)cur, tabu, ulist, wl, tmin_a, lane, nw);
        } else {
            const ItemPtr im = opaque(item);
            pick = fallback_lone<kTabu, kPher>(
                fallback_args<kPher>(im, it, (uint32_t)ant, kk, (uint32_t)cur, n - kk, fallback_tabu(tabu), tmin_a),
                (LdsPtr<uint16_t>)ulist, list_cap(n, im->s.list_cap), lane);
        }
        const uint32_t next = (uint32_t)__builtin_amdgcn_readfirstlane((int)pick);
        // no city is unreachable with a validated instance; were it not,
        // report it after the tour and go on with city 0 (the tour is void)
        // rather than index out of bounds
        bad |= next >= (uint32_t)n;
        return next < (uint32_t)n ? next : 0u;
    };

    // marks the chosen city, records it as step k and moves there
    auto advance = [&](uint32_t next, int at, int k) {
        if constexpr (kTabu == MMAS_TABU_BITMASK) {
            // every lane issues the OR, so that no exec mask is set up around
            // it: lane 0 into the city's word, the others a 0 into their own
            // word of the draw buffer (no change)
            const uint32_t addr = mark_base + (((next >> 5) << 2) & mark_mask);
            __hip_atomic_fetch_or(lds_at<uint32_t>(addr), (1u << (next & 31u)) & mark_mask,
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
            tabu.mark_at(next, at);
        }
        if (lane == (k & 63)) tbuf = next;
        cur = __builtin_amdgcn_readfirstlane((int)next);
    };

    // The row entry of this lane for city c (rank lr of its candidate list),
    // loaded one step ahead: as soon as the next city is known, before it is
    // marked, so the loads are not queued behind the mark.
    // (typed as a 16-bit float only so that its bits are never widened)
    _Float16 node_next = 0;
    float w_next = 0.0f;
    uint32_t lds_cand_l = (uint32_t)(uintptr_t)lds_cand + 2u * (uint32_t)lr;
    uint32_t lds_chc_l = (uint32_t)(uintptr_t)lds_chc + 4u * (uint32_t)lr;
    asm volatile("" : "+v"(lds_cand_l), "+v"(lds_chc_l));
    auto load_row_near = [&](int c) {
        const uint32_t e = (uint32_t)(c * cl);
        node_next = *lds_at<const _Float16>(lds_cand_l + 2u * e);
        w_next = *lds_at<const float>(lds_chc_l + 4u * e);
    };
    auto load_row_far = [&](int c) {
        const uint32_t e = (uint32_t)(c * cl);
        node_next = ((GlbPtr<const _Float16>)glb_cand + e)[(uint32_t)lr];
        w_next = (glb_chc + e)[(uint32_t)lr];
    };
    auto load_row = [&](int c) {
        if (__builtin_expect(c < R, 1))
            load_row_near(c);
        else
            load_row_far(c);
    };

    // One candidate-phase step k reading its draws at lnbuf[4jG + r] and the
    // row loaded ahead for the current city; `mid` runs before the row's
    // first use (independent work that fills the loads' latency).
    auto cand_step = [&](int k, int j, auto&& mid) {
        // (a bitmask's visited test does not look at the bits above 16, so the
        // city is not widened on its chain)
        uint32_t node_raw, node_word = 0u;
        if constexpr (kTabu == MMAS_TABU_BITMASK) {
            asm("v_bfe_u32 %0, %1, 5, 11" : "=v"(node_word) : "v"(node_next));
            asm("v_mov_b32 %0, %1" : "=v"(node_raw) : "v"(node_next));
        } else {
            asm("v_and_b32 %0, 0xffff, %1" : "=v"(node_raw) : "v"(node_next));
        }
        const float w = w_next;
        mid();
        const float lnu = lds_ln[4 * j * G + ln_lane];
        uint32_t seen = 0u, cell = 0u;
        if constexpr (kTabu == MMAS_TABU_BITMASK)
            seen = (uint32_t)__builtin_amdgcn_sbfe((int)*lds_at<const uint32_t>(cells + 4u * node_word), node_raw, 1u);
        else
            cell = tabu.cell(node_raw);
        if constexpr (kTabu != MMAS_TABU_BITMASK) {
            // (both LDS reads go out before the product waits for the first)
            __builtin_amdgcn_sched_barrier(0);
            seen = tabu.seen(node_raw, cell);
        }
        float key = lnu * w;  // (w holds 1 / choice_info)
        asm volatile("" : "+v"(key));
        // ln(u) < 0 and w >= 0 give a key with the sign bit set (a negative
        // number, -0 or -inf), whose order code is ~bits (kApprox: the key is
        // approximate, and the exact ones settle a near tie)
        const uint32_t code = ~__float_as_uint(key) & ~seen & lane_ok;
        // (for cl <= 32 only the first half's maximum counts: lanes past the
        // list have no code, so none of them holds or is near it)
        const uint32_t top = rows_max_lanes<kRows>(code);
        const uint64_t tied = __ballot(kApprox ? code >= near_code(top) : code == top) & (kRows == 2 ? 0xFFFFFFFFull : ~0ull);
        const int first = (int)__builtin_ctzll(tied | (1ull << 63));
        uint32_t next = (uint32_t)__builtin_amdgcn_readlane((int)node_raw, first) & 0xFFFFu;
        // the chosen city's cell (compact and list tabus)
        int at = __builtin_amdgcn_readlane((int)cell, first);
        if (__builtin_expect(__popcll(tied) != 1, 0)) {
            const uint32_t node = node_raw & 0xFFFFu;
            const uint32_t best = (uint32_t)__builtin_amdgcn_readfirstlane((int)top);
            if (best == 0u) {
                next = fallback(k);
            } else {
                uint32_t c = code, t = best;
                if constexpr (kApprox) {
                    c = step_exact_code(opaque(item)->s.seed, it, (uint32_t)ant, (uint32_t)k, (uint32_t)lane, w,
                                        ~seen & lane_ok);
                    t = wave_max_u32<kRows>(c);
                }
                next = wave_min_u32<kRows>(c == t ? node : kNone);
            }
            if constexpr (kTabu != MMAS_TABU_BITMASK) at = __builtin_amdgcn_readfirstlane((int)tabu.cell(next));
        }
        // (the move is written out for both kinds of row: as one piece of code
        // after the loads it cost the compiler two more branches a step)
        if (__builtin_expect((int)next < R, 1)) {
            load_row_near((int)next);
            advance(next, at, k);
        } else {
            load_row_far((int)next);
            advance(next, at, k);
        }
    };

    // after the steps before ke: at the end of a 64-step chunk or of the
    // tour, store the chunk's cities and add the lengths of the edges into them
    auto flush = [&](int ke) {
        if ((ke & 63) == 0 || ke == n) {
            // steps c0 .. ke - 1; lane l holds step c0 + l
            const int c0 = (ke - 1) & ~63;
            const int last = ke - 1 - c0;
            const uint32_t prev = __shfl_up(tbuf, 1);
            if (lane <= last) {
                tour_out[c0 + lane] = (uint16_t)tbuf;
                // edge entering step c0 + l (none for step 0)
                const uint32_t from = lane == 0 ? prev_last : prev;
                if (c0 + lane > 0) len += dist[(size_t)from * n + tbuf];
            }
            prev_last = (uint32_t)__builtin_amdgcn_readlane((int)tbuf, last);
        }
    };

    // the draws of the group of steps k0 .. k0 + S - 1, all at once
    auto draws_now = [&](int k0) {
        const Words4 b = draw_block(seed, it, (uint32_t)ant, (uint32_t)(k0 + (lane >> gsh)),
                                    (uint32_t)(4 * (lane & (G - 1))));
        float4 lv;
        lv.x = log2_draw(b.w[0]);
        lv.y = log2_draw(b.w[1]);
        lv.z = log2_draw(b.w[2]);
        lv.w = log2_draw(b.w[3]);
        *reinterpret_cast<float4*>(lnbuf + 4 * lane) = lv;
    };

    // steps kb .. ke - 1 of the group starting at k0 (draws in place)
    auto steps_plain = [&](int k0, int kb, int ke) {
        for (int k = kb; k < ke; ++k) cand_step(k, k - k0, [] {});
    };

    if (cl == 0) {
        for (int k = 1; k < n; ++k) {
            const uint32_t next = fallback(k);
            int at = 0;
            if constexpr (kTabu != MMAS_TABU_BITMASK) at = __builtin_amdgcn_readfirstlane((int)tabu.cell(next));
            advance(next, at, k);
            flush(k + 1);
        }
    } else if constexpr (kG > 0 && kHelp) {
        // draws from the helper wave: group g in buffer g & 1
        const LdsPtr<const float> buf0 = (LdsPtr<const float>)lnbuf;
        const LdsPtr<const float> buf1 = (LdsPtr<const float>)reinterpret_cast<float*>(help);
        constexpr int S = kWave / kG;
        load_row(cur);
        int g = 0;
        for (int k0 = 0; k0 < n; k0 += S, ++g) {
            if (!bad_help) bad_help = !wait_count(&hl->made, g + 1);  // (after one timeout, no more waits)
            lds_ln = (g & 1) ? buf1 : buf0;
            const int ke = k0 + S < n ? k0 + S : n;
            steps_plain(k0, k0 > 0 ? k0 : 1, ke);
            lds_put(&hl->read, g + 1);  // after the group's last read of its buffer
            flush(ke);
        }
    } else if constexpr (kG > 0) {
        load_row(cur);
        // Draws computed one group ahead, spread over the steps of the group
        // before in seven pieces (three of Philox rounds, the last round with
        // the first logarithm, one logarithm each) that fill the latency of
        // the steps' row loads, and stored after that group's last read.
        constexpr int S = kWave / kG;
        static_assert(S == 8 || S == 16, "pieces are laid out for 8 or 16 steps a group");
        const uint32_t k0s = (uint32_t)seed, k1s = (uint32_t)(seed >> 32);
        draws_now(0);
        steps_plain(0, 1, S < n ? S : n);
        flush(S < n ? S : n);
        if (S < n) draws_now(S);
        int k0 = S;
        for (; k0 + S <= n; k0 += S) {
            Words4 c;
            float lv[4];
            const int kn = k0 + S;  // the group whose draws are computed here
#pragma unroll
            for (int j = 0; j < S; ++j) {
                // piece q of the next group's draws runs at step j = q * S / 8
                auto piece = [&] {
                    if (j * 8 % S != 0) return;
                    const int q = j * 8 / S;
                    // (each piece's results pass through an empty asm in this
                    // step, which keeps the compiler from sinking the piece to
                    // the end of the group, where its results are stored)
                    if (q == 0) {
                        c = Words4{{(uint32_t)(lane & (kG - 1)) | ((uint32_t)(kn + (lane >> gsh)) << 16),
                                    (uint32_t)ant, it, 0u}};
                        philox_rounds<0, 3>(c, k0s, k1s);
                    } else if (q == 1) {
                        philox_rounds<3, 6>(c, k0s, k1s);
                    } else if (q == 2) {
                        philox_rounds<6, 9>(c, k0s, k1s);
                    } else if (q == 3) {
                        philox_rounds<9, 10>(c, k0s, k1s);
                        lv[0] = log2_draw(c.w[0]);
                        asm volatile("" : "+v"(lv[0]));
                    } else if (q < 7) {
                        lv[q - 3] = log2_draw(c.w[q - 3]);
                        asm volatile("" : "+v"(lv[q - 3]));
                    }
                    if (q < 4) asm volatile("" : "+v"(c.w[0]), "+v"(c.w[1]), "+v"(c.w[2]), "+v"(c.w[3]));
                };
                cand_step(k0 + j, j, piece);
            }
            // after the group's last read of the buffer
            *reinterpret_cast<float4*>(lnbuf + 4 * lane) = make_float4(lv[0], lv[1], lv[2], lv[3]);
            flush(k0 + S);
        }
        if (k0 < n) {
            steps_plain(k0, k0, n);
            flush(n);
        }
    } else {
        load_row(cur);
        for (int k0 = 0; k0 < n; k0 += S) {
            draws_now(k0);
            const int ke = k0 + S < n ? k0 + S : n;
            steps_plain(k0, k0 > 0 ? k0 : 1, ke);
            flush(ke);
        }
    }
    if constexpr (kWide) wide_lead_end(wl, lane);
    if (bad && lane == 0) atomicOr(&item->v.state->flags, 8u);
    if (bad_help && lane == 0) atomicOr(&item->v.state->flags, 32u);
    if (lane == 0) len += dist[(size_t)cur * n + start];  // closing edge
    len = wave_sum_i64(len);
    if (lane == 0) {
        item->v.lengths[ant] = len;
        item->v.fallback[ant] = fb_steps;
        item->v.fallback[item->s.ants + ant] = fb_nodes;
    }
}

// Per-half wave64 reductions for two ants per wave (lanes 0-31: first ant,
// 32-63: second): the maximum (minimum) of each half, as two scalars.
__device__ __forceinline__ void half_max_u32(uint32_t x, uint32_t& lo, uint32_t& hi) {
    x = max(x, dpp<0xB1>(x));
    x = max(x, dpp<0x4E>(x));
    x = max(x, dpp<0x141>(x));
    x = max(x, dpp<0x140>(x));
    lo = max((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16));
    hi = max((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48));
}
__device__ __forceinline__ void half_min_u32(uint32_t x, uint32_t& lo, uint32_t& hi) {
    x = min(x, dpp<0xB1>(x));
    x = min(x, dpp<0x4E>(x));
    x = min(x, dpp<0x141>(x));
    x = min(x, dpp<0x140>(x));
    lo = min((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16));
    hi = min((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48));
}

// The all-node fallback of one ant on the whole wave (outlined: its arguments
// are wave-uniform and arrive in vector registers).
template <int kTabu, int kPher>
__device__ __attribute__((noinline)) uint32_t fallback_item(ItemPtr item_v, LdsPtr<uint8_t> region_v, uint32_t it,
                                                            uint32_t ant, int k_v, uint32_t cur_v, float tmin_a,
                                                            int lane) {
    const ItemPtr item = (ItemPtr)uni((uint64_t)(uintptr_t)item_v);
    const uint32_t region = uni((uint32_t)(uintptr_t)region_v);
    const int k = uni(k_v), n = item->s.n;
    const size_t row = (size_t)uni(cur_v) * n;
    Fallback q;
    q.tabu = lds_at<const uint16_t>(region + (uint32_t)(kDrawBytes + kScratchBytes));
    q.L = n - k;
    q.n = n;
    q.cl = item->s.cl;
    q.beta = item->s.beta;
    // (C-style casts: the only casts that change the address space)
    q.irow = kPher == MMAS_PHER_DENSE ? (GlbPtr<const float>)(item->v.choice_inv + row) : nullptr;
    q.drow = kPher == MMAS_PHER_DENSE ? nullptr : (GlbPtr<const int32_t>)(item->v.dist + row);
    q.tmin_a = uni(tmin_a);
    q.seed = item->s.seed;
    q.it = uni(it);
    q.ant = uni(ant);
    q.step = (uint32_t)k;
    const int cap = list_cap(n, item->s.list_cap);
    return fallback_wave<kTabu, kPher>(
        q, lds_at<uint16_t>(region + (uint32_t)(kDrawBytes + kScratchBytes) + (uint32_t)align16(4 * ((n + 31) / 32))),
        cap, lane);
}

// The visited test of a lane's candidate in a wave serving two ants: half h
// reads the tabu of its own ant, whose cells start at LDS byte `cells` (~0 if
// visited, else 0).
template <int kTabu>
__device__ __forceinline__ uint32_t seen_pair(uint32_t cells, int n, int L, uint32_t v) {
    if constexpr (kTabu == MMAS_TABU_BITMASK) {
        const uint32_t word = *lds_at<const uint32_t>(cells + 4u * __builtin_amdgcn_ubfe(v, 5u, 11u));
        return (uint32_t)__builtin_amdgcn_sbfe((int)word, v, 1u);
    } else if constexpr (kTabu == MMAS_TABU_COMPACT) {
        return *lds_at<const uint16_t>(cells + 2u * v) > v ? ~0u : 0u;
    } else {
        return (int)*lds_at<const uint16_t>(cells + 2u * ((uint32_t)n + v)) >= L ? ~0u : 0u;
    }
}
__device__ __forceinline__ int pair_left(const BitmaskTabu&, const BitmaskTabu&, int) { return 0; }
template <class T>
__device__ __forceinline__ int pair_left(const T& a, const T& b, int h) { return h ? b.L : a.L; }

// Two ants per wave64 (1 <= cl <= 32): lanes 0-31 serve ant `ant0`, lanes
// 32-63 ant `ant0 + 1` (without one, ant0 again in the second region, its
// results not stored). Both take their candidate steps together: lane 32h + r
// holds rank r of ant h's current row, the keys and the per-half argmax are
// those of construct_ant. A step in which an ant has no unvisited candidate
// runs that ant's fallback on the whole wave. Same draws, same choices, same
// tours as one ant per wave. With eight waves on a SIMD the step is bound by
// instruction issue, so what is wave-uniform (ant0, both cities, the
// selection) stays in scalar registers and instructions, rows are addressed
// by 32-bit offsets, and whatever only the rare paths need (a near tie, a
// fallback) is read again there: about 38 vector instructions a step (75 with
// the instance held in spilled scalar registers), 14 more for a quarter of the
// draws' Philox block and logarithms, and no spilled register inside the loop.
// kTable: some rows are in LDS.
template <int kTabu, int kPher, bool kTable>
__device__ __forceinline__ void construct_pair(ItemPtr item, uint32_t it, int ant0, int lane, uint8_t* regA, uint8_t* regB,
                               const uint16_t* tcand, const float* tchc, int R) {
    using Tabu = typename TabuOf<kTabu>::type;
    const int n = item->s.n, cl = item->s.cl;
    const int h = lane >> 5, hl = lane & 31;
    const bool hasB = ant0 + 1 < item->s.ants;
    const uint32_t antA = (uint32_t)ant0, antB = hasB ? antA + 1u : antA;
    const uint32_t my_ant = h ? antB : antA;

    Tabu tabA, tabB;
    tabA.init(regA + kDrawBytes + kScratchBytes, n, lane);
    tabB.init(regB + kDrawBytes + kScratchBytes, n, lane);
    float* lnbuf = reinterpret_cast<float*>(h ? regB : regA);
    const uint32_t cells = (uint32_t)(uintptr_t)(LdsPtr<float>)lnbuf + (uint32_t)(kDrawBytes + kScratchBytes);

    float tmin_a = 0.0f;
    if (kPher == MMAS_PHER_CANDIDATES) tmin_a = powi(item->v.state->tau_min, item->s.alpha);
    const LdsPtr<const uint16_t> lds_cand = (LdsPtr<const uint16_t>)tcand;
    const LdsPtr<const float> lds_chc = (LdsPtr<const float>)tchc;
    const GlbPtr<const uint8_t> glb_cand = (GlbPtr<const uint8_t>)item->v.cand;
    const GlbPtr<const uint8_t> glb_chc = (GlbPtr<const uint8_t>)item->v.chc_inv;  // reciprocals
    uint32_t k0s = (uint32_t)item->s.seed, k1s = (uint32_t)(item->s.seed >> 32);

    // start cities: floor(x * n / 2^32) of draw (step 0, slot 0) of each ant
    const uint32_t x0 = draw_block(item->s.seed, it, my_ant, 0u, 0u).w[0];
    const uint32_t st_l = (uint32_t)(((uint64_t)x0 * (uint64_t)n) >> 32);
    const int startA = __builtin_amdgcn_readlane((int)st_l, 0);
    const int startB = __builtin_amdgcn_readlane((int)st_l, 32);
    tabA.mark((uint32_t)startA, lane);
    tabB.mark((uint32_t)startB, lane ^ 32);

    // draws ahead, S = 32/G steps at a time, each half for its own ant
    const int gsh = cl <= 4 ? 0 : cl <= 8 ? 1 : cl <= 16 ? 2 : 3;
    const int G = 1 << gsh;
    const int S = 32 >> gsh;
    const int lr = hl < cl ? hl : cl - 1;
    uint32_t lane_ok = hl < cl ? ~0u : 0u;
    const uint32_t ln_lane = (uint32_t)(uintptr_t)(LdsPtr<float>)lnbuf + 4u * (uint32_t)(hl & (4 * G - 1));
    // bitmask marks, both in one LDS OR issued by every lane: lane 0 sets A's
    // bit, lane 32 B's, the others OR zero into their own word of the draw
    // buffer (a field of no bits gives them offset 0, and their "bit" is 0)
    uint32_t mark_bits = hl == 0 ? 11u : 0u, mark_one = hl == 0 ? 1u : 0u;
    uint32_t mark_base = hl == 0 ? cells : (uint32_t)(uintptr_t)(LdsPtr<float>)lnbuf + 4u * (uint32_t)hl;
    asm volatile("" : "+v"(mark_bits), "+v"(mark_one), "+v"(mark_base), "+v"(lane_ok));

    uint32_t tbuf = (uint32_t)(h ? startB : startA);  // lane 32h + (k & 31) holds the city of step k
    uint32_t prev_last = 0;
    int64_t len = 0;
    uint32_t fbA_steps = 0, fbA_nodes = 0, fbB_steps = 0, fbB_nodes = 0;
    int curA = startA, curB = startB;
    bool bad = false;

    // an ant without an unvisited candidate (no city at all is unreachable with
    // a validated instance; were it so, report it after the tour and go on with
    // city 0: the tour is void)
    auto fallback = [&](uint32_t ant, int cur, int k, uint8_t* reg) -> uint32_t {
        const uint32_t pick = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)fallback_item<kTabu, kPher>(opaque(item), (LdsPtr<uint8_t>)reg, it, ant, k, (uint32_t)cur, tmin_a, lane));
        bad |= pick >= (uint32_t)n;
        return pick < (uint32_t)n ? pick : 0u;
    };

    for (int k0 = 0; k0 < n; k0 += S) {
        {
            // (the round keys are formed anew: kept, they would be spilled)
            asm volatile("" : "+s"(k0s), "+s"(k1s));
            const Words4 b = philox4x32_10((uint32_t)(hl & (G - 1)) | ((uint32_t)(k0 + (hl >> gsh)) << 16), my_ant, it,
                                           0u, k0s, k1s);
            float4 lv;
            lv.x = log2_draw(b.w[0]);
            lv.y = log2_draw(b.w[1]);
            lv.z = log2_draw(b.w[2]);
            lv.w = log2_draw(b.w[3]);
            *reinterpret_cast<float4*>(lnbuf + 4 * hl) = lv;
        }
        const int kb = k0 > 0 ? k0 : 1;
        const int ke = k0 + S < n ? k0 + S : n;
        for (int k = kb; k < ke; ++k) {
            const uint32_t offA = (uint32_t)(curA * cl), offB = (uint32_t)(curB * cl);
            const uint32_t e = (h ? offB : offA) + (uint32_t)lr;
            uint32_t node;
            float w;
            if constexpr (kTable) {
                const int cur_l = h ? curB : curA;
                if (cur_l >= R) {
                    node = *(GlbPtr<const uint16_t>)(glb_cand + 2u * e);
                    w = *(GlbPtr<const float>)(glb_chc + 4u * e);
                } else {
                    node = lds_cand[e];
                    w = lds_chc[e];
                }
            } else {
                node = *(GlbPtr<const uint16_t>)(glb_cand + 2u * e);
                w = *(GlbPtr<const float>)(glb_chc + 4u * e);
            }
            const float lnu = *lds_at<const float>(ln_lane + (uint32_t)(16 * (k - k0) * G));
            const uint32_t seen = seen_pair<kTabu>(cells, n, pair_left(tabA, tabB, h), node);
            float key = lnu * w;  // (w holds 1 / choice_info)
            asm volatile("" : "+v"(key));
            // log2(u) < 0 and w >= 0: the key's sign bit is set, its order code
            // is ~bits (approximate keys: device.hpp)
            const uint32_t code = ~__float_as_uint(key) & ~seen & lane_ok;
            // (no code is near a best of 0)
            const uint64_t tied = __ballot(code >= near_code(half_max_lanes(code)));
            const uint32_t tA = (uint32_t)tied, tB = (uint32_t)(tied >> 32);
            uint32_t nextA = (uint32_t)__builtin_amdgcn_readlane((int)node, __builtin_ctz(tA | 0x80000000u));
            uint32_t nextB = (uint32_t)__builtin_amdgcn_readlane((int)node, 32 + __builtin_ctz(tB | 0x80000000u));
            const int cntA = __builtin_popcount(tA), cntB = __builtin_popcount(tB);
            if (__builtin_expect(((cntA ^ 1) | (cntB ^ 1)) != 0, 0)) {
                if (cntA > 1 || cntB > 1) {
                    const uint32_t c = step_exact_code(opaque(item)->s.seed, it, my_ant, (uint32_t)k, (uint32_t)hl, w,
                                                       ~seen & lane_ok);
                    uint32_t topA, topB, mA, mB;
                    half_max_u32(c, topA, topB);
                    half_min_u32(c == (h ? topB : topA) ? node : kNone, mA, mB);
                    if (cntA > 1) nextA = mA;
                    if (cntB > 1) nextB = mB;
                }
                if (cntA == 0) {
                    fbA_steps += 1;
                    fbA_nodes += (uint32_t)(n - k);
                    nextA = fallback(antA, curA, k, regA);
                }
                if (cntB == 0) {
                    fbB_steps += 1;
                    fbB_nodes += (uint32_t)(n - k);
                    nextB = fallback(antB, curB, k, regB);
                }
            }
            const uint32_t nx = h ? nextB : nextA;
            if constexpr (kTabu == MMAS_TABU_BITMASK) {
                const uint32_t addr = mark_base + 4u * __builtin_amdgcn_ubfe(nx, 5u, mark_bits);
                __hip_atomic_fetch_or(lds_at<uint32_t>(addr), mark_one << (nx & 31u), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                tabA.mark(nextA, lane);
                tabB.mark(nextB, lane ^ 32);
            }
            if (hl == (k & 31)) tbuf = nx;
            curA = (int)nextA;
            curB = (int)nextB;
        }
        if ((ke & 31) == 0 || ke == n) {
            // flush steps c0 .. ke - 1; lane 32h + l holds step c0 + l of ant h
            const int c0 = (ke - 1) & ~31;
            const int last = ke - 1 - c0;
            const ItemPtr im = opaque(item);
            uint16_t* tour_out = im->v.tours + (size_t)my_ant * n;
            const int32_t* dist = im->v.dist;
            const uint32_t prev = __shfl_up(tbuf, 1);
            if (hl <= last && (h == 0 || hasB)) {
                tour_out[c0 + hl] = (uint16_t)tbuf;
                const uint32_t from = hl == 0 ? prev_last : prev;
                if (c0 + hl > 0) len += dist[(size_t)from * n + tbuf];
            }
            const uint32_t plA = (uint32_t)__builtin_amdgcn_readlane((int)tbuf, last);
            const uint32_t plB = (uint32_t)__builtin_amdgcn_readlane((int)tbuf, 32 + last);
            prev_last = h ? plB : plA;
        }
    }
    const ItemPtr im = opaque(item);
    if (bad && lane == 0) atomicOr(&im->v.state->flags, 8u);
    if (hl == 0) len += im->v.dist[(size_t)(h ? curB : curA) * n + (h ? startB : startA)];  // closing edges
    for (int o = 16; o >= 1; o >>= 1) len += __shfl_xor(len, o);
    if (hl == 0 && (h == 0 || hasB)) {
        im->v.lengths[my_ant] = len;
        im->v.fallback[my_ant] = h ? fbB_steps : fbA_steps;
        im->v.fallback[im->s.ants + my_ant] = h ? fbB_nodes : fbA_nodes;
    }
}

// kRows: 16-lane rows the argmax of a one-ant-per-wave step reduces (2 for
// cl <= 32, else 4); kG: 4-slot draw groups per step when fixed (4 for
// 9 <= cl <= 16, 8 for 17 <= cl <= 32: the draws are then pipelined), else 0.
// Both unused with two ants per wave. kHelp (one ant per wave, kG > 0): the
// workgroup has a draw helper wave per ant (waves apb .. 2 apb - 1 for the
// ants of waves 0 .. apb - 1); each region ends with the helper's part.
template <int kTabu, int kPher, bool kPair, int kRows = 4, int kG = 0, bool kHelp = false>
__global__ __launch_bounds__(1024) void k_construct(Views vw, Shape s, uint32_t it, int ants_per_block, Lds lds) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const ItemPtr item = kernel_item();
    const int R = lds.rows;
    uint16_t* tcand = reinterpret_cast<uint16_t*>(smem);
    float* tchc = reinterpret_cast<float*>(smem + align16(R * s.cl * 2));
    uint8_t* regions = smem + lds.table_bytes;
    if (R > 0) stage_table(vw, s.cl, R, tcand, tchc);
    if constexpr (kHelp) {
        // every ant's HelpLds starts at 0
        if ((int)threadIdx.x < ants_per_block)
            *reinterpret_cast<int4*>(regions + (size_t)(threadIdx.x + 1) * lds.per_ant - sizeof(HelpLds)) =
                make_int4(0, 0, 0, 0);
    }
    if (R > 0 || kHelp) __syncthreads();
    const bool helper = kHelp && wave >= ants_per_block;
    const int aw = helper ? wave - ants_per_block : wave;
    const int ant = blockIdx.x * ants_per_block + (kPair ? 2 * aw : aw);
    if (ant >= s.ants) return;  // whole waves leave together
    if constexpr (kHelp) {
        uint8_t* region = regions + (size_t)aw * lds.per_ant;
        uint8_t* help = region + lds.per_ant - kHelpBytes;
        if (helper)
            draw_helper<kG>(item, it, ant, lane, region, help);
        else
            construct_lone<kTabu, kPher, kRows, kG, false, true>(item, it, ant, lane, region, tcand, tchc, R,
                                                                 nullptr, 1, help);
        return;
    }
    if constexpr (kPair) {
        construct_pair<kTabu, kPher, true>(item, it, ant, lane, regions + (size_t)(2 * wave) * lds.per_ant,
                                           regions + (size_t)(2 * wave + 1) * lds.per_ant, tcand, tchc, R);
    }
    else
        construct_lone<kTabu, kPher, kRows, kG>(item, it, ant, lane, regions + (size_t)wave * lds.per_ant, tcand,
                                                tchc, R);
}

// One ant per workgroup of several waves: the leading wave takes the steps
// as in the single colony (construct_lone), the others share its
// fallbacks. LDS: the table part, then the ant's region. kRows, kG as for
// k_construct.
template <int kTabu, int kPher, int kRows = 4, int kG = 0>
__global__ __launch_bounds__(1024) void k_construct_wide(Views vw, Shape s, uint32_t it, Lds lds) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ WideLds wl;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nw = (int)(blockDim.x >> 6);
    const ItemPtr item = kernel_item();
    const int R = lds.rows;
    uint16_t* tcand = reinterpret_cast<uint16_t*>(smem);
    float* tchc = reinterpret_cast<float*>(smem + align16(R * s.cl * 2));
    if (R > 0) stage_table(vw, s.cl, R, tcand, tchc);
    __syncthreads();
    uint8_t* region = smem + lds.table_bytes;
    if (wave > 0) {
        wide_helpers<kTabu, kPher>(item, it, (int)blockIdx.x, lane, region, &wl, wave, nw);
        return;
    }
    // the leading wave: the single-colony step, its fallbacks shared
    construct_lone<kTabu, kPher, kRows, kG, true>(item, it, (int)blockIdx.x, lane, region, tcand, tchc, R, &wl, nw);
}

// Without candidate lists, up to 4096 cities: a team of W waves per ant and no
// shared tabu. Every step keys all unvisited cities (Alg. 4 over all of them,
// as the fallback does), by draw blocks: wave w, lane l takes blocks
// 64 w + l + 64 W r, r < kBlocks (cities 4 b .. 4 b + 3 of block b), keeps
// their visited bits in a register, computes each block once and keys its
// four words approximately (device.hpp). With W > 1 each wave posts its best
// and whether its second best is near it, and after one barrier all waves
// take the same winner; with one wave there is no exchange. A near tie (about
// one step in 10^5) is settled by the exact keys. Bound by issue: about 78
// instructions a block (half of them the Philox rounds) and 90 a step and
// wave. n = 1002, 1002 ants: 2.55 ms -> 0.95 ms (four waves that all computed
// every Philox block, exact keys with 25 instructions a logarithm, before);
// n = 198: 130 -> 79 us; n = 3795, 3795 ants: 71 -> 35 ms.
// (a row is read four floats at a time: the last block's read may pass the
// row's end by at most three floats, into the next row or, after the last
// row, into the padding of the view to 256 bytes, which is at least that long
// whenever n is not a multiple of 4)
template <int W, int kBlocks>
__global__ __launch_bounds__(64 * W) void k_construct_team(Views vw, Shape s, uint32_t it) {
    static_assert(kBlocks <= 4, "a city's place in the lane takes four code bits");
    constexpr uint32_t kId = kBlocks == 1 ? 3u : kBlocks == 2 ? 7u : 15u;  // those low bits
    __shared__ unsigned long long res[2][W];  // by step parity: each wave's best
    __shared__ unsigned long long resx[W];    // the exact keys' best
    const int lane = threadIdx.x & 63;
    const int wave = W > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int ant = blockIdx.x;
    const int n = s.n;
    const uint64_t seed = s.seed;
    const int b0 = kWave * wave + lane;  // this lane's first draw block; the others follow at 64 W
    const uint32_t x0 = draw_block(seed, it, (uint32_t)ant, 0u, 0u).w[0];
    const int start = __builtin_amdgcn_readfirstlane((int)(((uint64_t)x0 * (uint64_t)n) >> 32));
    // bit 4 r + j: city j of block r is live; cities past n count as visited
    uint32_t live = 0u;
    uint32_t row_off[kBlocks];  // bytes into the row of factors
#pragma unroll
    for (int r = 0; r < kBlocks; ++r) {
        const int left = n - 4 * (b0 + kWave * W * r);
        live |= (left >= 4 ? 0xFu : left > 0 ? (1u << left) - 1u : 0u) << (4 * r);
        row_off[r] = left > 0 ? 16u * (uint32_t)(b0 + kWave * W * r) : 0u;
    }
    auto mark = [&](int c) {
        const int cb = c >> 2;
        live &= ~((cb & (kWave * W - 1)) == b0 ? 1u << (4 * (cb / (kWave * W)) + (c & 3)) : 0u);
    };
    mark(start);

    uint16_t* tour_out = vw.tours + (size_t)ant * n;
    const int32_t* dist = vw.dist;
    uint32_t tbuf = (uint32_t)start;  // first wave: lane (k & 63) holds the city of step k
    uint32_t prev_last = 0;
    int64_t len = 0;
    int cur = start;
    for (int k = 1; k < n; ++k) {
        // the factors first, then the draws
        const uint8_t* row = reinterpret_cast<const uint8_t*>(vw.choice_inv + (size_t)cur * n);
        float f[kBlocks][4];
#pragma unroll
        for (int r = 0; r < kBlocks; ++r) __builtin_memcpy(f[r], row + row_off[r], sizeof(f[r]));
        uint32_t m1 = 0u, m2 = 0u;
#pragma unroll
        for (int r = 0; r < kBlocks; ++r) {
            const Words4 blk =
                draw_block(seed, it, (uint32_t)ant, (uint32_t)k, (uint32_t)(4 * (b0 + kWave * W * r)));
            uint32_t code[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int id = 4 * r + j;
                const float key = log2_draw(blk.w[j]) * f[r][j];
                const uint32_t m = (uint32_t)((int)(live << (31 - id)) >> 31);  // ~0 if live
                code[j] = ((~__float_as_uint(key) & ~kId) | (uint32_t)id) & m;
            }
            uint32_t t1, t2;
            top_two(code[0], code[1], code[2], code[3], t1, t2);
            m2 = max(max(m2, t2), min(m1, t1));
            m1 = max(m1, t1);
        }
        const uint32_t best = wave_max_bcast(m1);
        const uint32_t near = near_code(best);
        const uint64_t tied = __ballot(m1 >= near);
        // (none is near when the wave has no city left: best is 0, and its city,
        // which no wave takes then, that of the last lane)
        const int first = (int)__builtin_ctzll(tied | (1ull << 63));
        const bool one = __popcll(tied) == 1, alone = __ballot(m2 >= near) == 0ull;
        bool clear = one & alone;
        const uint32_t id = best & kId;
        uint32_t next = 4u * (uint32_t)(kWave * (W * (int)(id >> 2) + wave) + first) + (id & 3u);
        if constexpr (W > 1) {
            if (lane == 0)
                res[k & 1][wave] = ((unsigned long long)best << 32) | (unsigned long long)(next << 1) |
                                   (unsigned long long)(clear ? 0u : 1u);
            __syncthreads();
            // every wave takes the same winner (res[k & 1] is written again two
            // steps later, after the next barrier)
            const unsigned long long rr = res[k & 1][lane < W ? lane : 0];
            const uint32_t hi = (uint32_t)(rr >> 32), lo = (uint32_t)rr;
            uint32_t mx = max(hi, dpp<0xB1>(hi));
            if (W > 2) mx = max(mx, dpp<0x4E>(mx));
            if (W > 4) mx = max(mx, dpp<0x141>(mx));
            if (W > 8) mx = max(mx, dpp<0x140>(mx));
            const uint32_t top = near_code((uint32_t)__builtin_amdgcn_readfirstlane((int)mx));
            const uint64_t held = __ballot(hi >= top) & ((1ull << W) - 1ull);
            const uint32_t pick = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)__builtin_ctzll(held | (1ull << 63)));
            next = pick >> 1;
            const bool one_wave = __popcll(held) == 1, sure = (pick & 1u) == 0u;
            clear = one_wave & sure;
        }
        if (__builtin_expect(!clear, 0)) {
            // the exact keys (every wave of the team comes here)
            uint32_t bcode = 0u, bnode = kNone;
#pragma unroll
            for (int r = 0; r < kBlocks; ++r) {
                const uint32_t c = 4u * (uint32_t)(b0 + kWave * W * r);
                const Words4 blk = draw_block(seed, it, (uint32_t)ant, (uint32_t)k, c);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    keep_best((live >> (4 * r + j)) & 1u ? ord_key(log_u01(u01(blk.w[j])) * f[r][j]) : 0u,
                              c + (uint32_t)j, bcode, bnode);
            }
            unsigned long long r = share_result(bcode, bnode);
            if constexpr (W > 1) {
                if (lane == 0) resx[wave] = r;
                __syncthreads();
                // (written again after the next step's barrier at the earliest)
                r = resx[0];
#pragma unroll
                for (int w = 1; w < W; ++w) r = resx[w] > r ? resx[w] : r;
            }
            next = (uint32_t)__builtin_amdgcn_readfirstlane((int)(r ? ~(uint32_t)r : kNone));
        }
        if (next >= (uint32_t)n) {
            // unreachable with a validated instance; every wave leaves
            if (wave == 0 && lane == 0) atomicOr(&vw.state->flags, 8u);
            break;
        }
        mark((int)next);
        cur = (int)next;
        if (wave == 0) {
            const int slot = k & 63;
            if (lane == slot) tbuf = next;
            if (slot == 63 || k == n - 1) {
                // flush the chunk of steps k0 .. k; lane l holds step k0 + l
                const int k0 = k - slot;
                const uint32_t prev = __shfl_up(tbuf, 1);
                if (lane <= slot) {
                    tour_out[k0 + lane] = (uint16_t)tbuf;
                    const uint32_t from = lane == 0 ? prev_last : prev;
                    if (k0 + lane > 0) len += dist[(size_t)from * n + tbuf];
                }
                prev_last = (uint32_t)__builtin_amdgcn_readlane((int)tbuf, slot);
            }
        }
    }
    if (wave != 0) return;
    if (lane == 0) len += dist[(size_t)cur * n + start];  // closing edge
    len = wave_sum_i64(len);
    if (lane == 0) {
        vw.lengths[ant] = len;
        vw.fallback[ant] = n - 1;                                 // every step is a fallback
        vw.fallback[s.ants + ant] = (int64_t)n * (n - 1) / 2;     // over n - k cities at step k
    }
}

static_assert(offsetof(BatchItem, v) == 0 && offsetof(BatchItem, s) == sizeof(Views) && alignof(Shape) == alignof(Views),
              "kernel_item reads the kernel's first two arguments");

// Batched construction: a persistent grid pulls tiles (instance, first ant of
// a group of ants_per_block ants) from a queue ordered by decreasing n. Each
// tile stages as many candidate rows of its instance as fit in the table part
// of LDS, then every wave builds one ant's tour (two with kPair).
// kTable: the launch has a table part.
template <int kTabu, int kPher, bool kPair, bool kTable>
// (limited to 64 VGPRs, which lets eight waves share a SIMD: the persistent
// batch is bound by instruction issue, and the extra waves hide more latency
// than the few registers cost that are spilled around the steps)
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_batch_construct(const BatchItem* __restrict__ items,
                                                          const BatchTile* __restrict__ tiles, int ntiles,
                                                          uint32_t* __restrict__ queue, const uint32_t* __restrict__ it_dev,
                                                          int ants_per_block, int table_bytes, int per_ant) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ int s_tile;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t it = *it_dev;
    for (;;) {
        if (threadIdx.x == 0) s_tile = (int)atomicAdd(queue, 1u);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(s_tile);
        if (t >= ntiles) break;  // every wave of the workgroup leaves here
        const int inst = __builtin_amdgcn_readfirstlane(tiles[t].inst);
        const Views& vw = items[inst].v;
        const Shape& s = items[inst].s;
        int R = 0;
        if (kTable && s.cl > 0) {
            R = (table_bytes - 16) / (s.cl * 6);
            if (R > s.n) R = s.n;
            while (R > 0 && align16(R * s.cl * 2) + R * s.cl * 4 > table_bytes) --R;
        }
        uint16_t* tcand = reinterpret_cast<uint16_t*>(smem);
        float* tchc = reinterpret_cast<float*>(smem + align16(R * s.cl * 2));
        if (R > 0) stage_table(vw, s.cl, R, tcand, tchc);
        __syncthreads();
        const int ant = __builtin_amdgcn_readfirstlane(tiles[t].ant0) + (kPair ? 2 * wave : wave);
        uint8_t* regions = smem + table_bytes;
        if (ant < s.ants) {
            if constexpr (kPair)
                construct_pair<kTabu, kPher, kTable>((ItemPtr)&items[inst], it, ant, lane,
                                                     regions + (size_t)(2 * wave) * per_ant,
                                                     regions + (size_t)(2 * wave + 1) * per_ant, tcand, tchc, R);
            else
                construct_ant<kTabu, kPher>((ItemPtr)&items[inst], it, ant, lane, regions + (size_t)wave * per_ant, tcand, tchc, R);
        }
        __syncthreads();  // the next tile reuses the table part
    }
}

}  // namespace

// Per-device attributes, read once per device (up to 64 devices).
namespace {
constexpr int kMaxDevices = 64;
std::atomic<int> g_lds[kMaxDevices];
std::atomic<int> g_simds[kMaxDevices];
std::atomic<int> g_cus[kMaxDevices];

int device_attr(std::atomic<int>* cache, hipDeviceAttribute_t attr, int scale, int fallback) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return fallback;
    int v = cache[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    int a = 0;
    v = hipDeviceGetAttribute(&a, attr, dev) == hipSuccess && a > 0 ? a * scale : fallback;
    cache[dev].store(v, std::memory_order_relaxed);
    return v;
}
}  // namespace

int max_lds_per_block() { return device_attr(g_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, 1, 65536); }
int compute_units() { return device_attr(g_cus, hipDeviceAttributeMultiprocessorCount, 1, 0); }

namespace {

// Two ants per wave when asked for and 1 <= cl <= 32 (the candidate row fits
// in a half wave).
bool pair_ok(const Shape& s) { return s.lanes_per_ant == 32 && s.cl >= 1 && s.cl <= 32; }

template <int kTabu, int kPher, bool kPair, int kRows = 4, int kG = 0>
hipError_t launch_t(const Views& v, const Shape& s0, uint32_t it, hipStream_t st) {
    // one colony: a workgroup per four ants rarely shares a CU, so the fallback
    // lists every unvisited city in one pass
    Shape s = s0;
    s.list_cap = s.n;
    // a draw helper wave per ant (one ant per wave with pipelined draws) by
    // default while every ant's wave has a SIMD of its own, which the helper
    // then shares; not with one wave per ant asked for
    const bool help = !kPair && kG > 0 && s.construct_waves == 0 &&
                      s.ants <= device_attr(g_simds, hipDeviceAttributeMultiprocessorCount, 4, 0);
    const int per_ant = (int)construct_lds_per_ant(s) + (help ? (int)kHelpBytes : 0);
    const int budget = max_lds_per_block();
    int apb = s.ants_per_block > 0 ? s.ants_per_block : 4;
    const int step = kPair ? 2 : 1;  // ants per wave
    if (apb < step) apb = step;
    if (help && apb > 8) apb = 8;  // two waves per ant, at most 16 a workgroup
    while (apb > step && per_ant * apb > budget) apb -= step;
    if (per_ant * apb > budget) return hipErrorInvalidValue;
    // as many rows of the candidate table as fit next to the ants' regions;
    // by default only in one workgroup's share of a CU's LDS when the grid
    // needs several per CU (a full table would leave one resident workgroup
    // per CU: 3795 ants at n = 3795 took 8.9 ms instead of 3.5 ms)
    const int blocks = (s.ants + apb - 1) / apb;
    int lds_wg = budget;
    const int cus = device_attr(g_cus, hipDeviceAttributeMultiprocessorCount, 1, 0);
    if (cus > 0 && s.table_rows < 0) {
        const int waves = apb / step * (help ? 2 : 1);
        int per_cu = (blocks + cus - 1) / cus;
        const int most = waves < 32 ? 32 / waves : 1;  // eight waves per SIMD
        if (per_cu > most) per_cu = most;
        if (per_cu > 1) lds_wg = budget / per_cu;
    }
    Lds lds{};
    lds.per_ant = per_ant;
    const int row_bytes = s.cl * 6;
    int rows = 0;
    if (s.cl > 0) {
        rows = (lds_wg - apb * per_ant - 32) / row_bytes;
        if (rows > s.n) rows = s.n;
        if (s.table_rows >= 0 && rows > s.table_rows) rows = s.table_rows;
        while (rows > 0 && align16(rows * s.cl * 2) + align16(rows * s.cl * 4) + apb * per_ant > budget) --rows;
        if (rows < 0) rows = 0;
    }
    lds.rows = rows;
    lds.table_bytes = align16(rows * s.cl * 2) + align16(rows * s.cl * 4);
    const size_t bytes = (size_t)lds.table_bytes + (size_t)apb * per_ant;
    auto kern = k_construct<kTabu, kPher, kPair, kRows, kG>;
    if constexpr (!kPair && kG > 0) {
        if (help) kern = k_construct<kTabu, kPher, false, kRows, kG, true>;
    }
    if (bytes > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    kern<<<blocks, 64 * (apb / step) * (help ? 2 : 1), bytes, st>>>(v, s, it, apb, lds);
    return hipGetLastError();
}

// Waves per ant for the construction: the launch option, or (0) a choice by
// where the all-city fallback dominates the step, the only part the helper
// waves share. With n >= 8192 (long fallbacks) and SIMDs to spare: as many
// as the SIMDs left over by one wave per ant allow, a power of two up to 16.
// Without a candidate list (past the team kernel's n): four (the bitmask
// tabu's cities are then gathered by the workgroup, one LDS atomic per wave).
// Otherwise one: the per-step barriers then cost more than the shared
// fallbacks save (measured at n = 198, 1002 and 3795 with lists).
int construct_waves(const Shape& s) {
    if (s.construct_waves > 0) return s.construct_waves;
    if (s.n >= 8192) {
        // four SIMDs per compute unit
        const int simds = device_attr(g_simds, hipDeviceAttributeMultiprocessorCount, 4, 0);
        int w = 1;
        while (w < 16 && 2 * w * s.ants <= simds) w *= 2;
        return w;
    }
    if (s.cl == 0) return 4;
    return 1;
}

template <int kTabu, int kPher>
hipError_t launch_wide(const Views& v, const Shape& s, uint32_t it, int waves, hipStream_t st) {
    const int per_ant = (int)wide_lds_per_ant(s);
    const int budget = max_lds_per_block() - (int)sizeof(WideLds) - 64;
    if (per_ant > budget) return hipErrorInvalidValue;
    Lds lds{};
    lds.per_ant = per_ant;
    int rows = 0;
    if (s.cl > 0) {
        rows = (budget - per_ant - 32) / (s.cl * 6);
        if (rows > s.n) rows = s.n;
        if (s.table_rows >= 0 && rows > s.table_rows) rows = s.table_rows;
        while (rows > 0 && align16(rows * s.cl * 2) + align16(rows * s.cl * 4) + per_ant > budget) --rows;
        if (rows < 0) rows = 0;
    }
    lds.rows = rows;
    lds.table_bytes = align16(rows * s.cl * 2) + align16(rows * s.cl * 4);
    const size_t bytes = (size_t)lds.table_bytes + (size_t)per_ant;
    auto kern = s.cl > 16 && s.cl <= 32 ? k_construct_wide<kTabu, kPher, 2, 8>
                : s.cl > 8 && s.cl <= 16 ? k_construct_wide<kTabu, kPher, 2, 4>
                : s.cl <= 32             ? k_construct_wide<kTabu, kPher, 2>
                                         : k_construct_wide<kTabu, kPher, 4>;
    if (bytes > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    kern<<<s.ants, 64 * waves, bytes, st>>>(v, s, it, lds);
    return hipGetLastError();
}

// The team kernel (no list, n <= 4096, whichever tabu: it keeps the visited
// bits in registers), by default or asked for with four waves per ant.
bool team_ok(const Shape& s) {
    if (s.cl != 0 || s.n > 4096) return false;
    return s.construct_waves == 0 || s.construct_waves == 4;
}

// Waves per ant and blocks per lane, by q = ceil(blocks / 64) waves of blocks.
// While q waves per ant load each SIMD at most twice, one block a lane: the
// blocks run side by side and the barrier costs less than a second block
// (n = 1002: 64 to 256 ants 0.56 ms with four waves, 0.90 with one; 512 ants
// 0.73 and 0.92). Past that the waves share the issue slots and the fewest
// waves win, whose exchange and selection are paid once per ant (1002 ants:
// 1.07 ms with four waves, 0.95 with one and no exchange; n = 3795, 3795
// ants: 62 and 35 ms with sixteen and four). Up to two blocks a lane one wave
// is as good at any ant count (n = 512: 64 ants 0.28 ms with two waves, 0.29
// with one; 512 ants 0.36 and 0.31).
template <int W, int kBlocks>
hipError_t launch_team_t(const Views& v, const Shape& s, uint32_t it, hipStream_t st) {
    k_construct_team<W, kBlocks><<<s.ants, kWave * W, 0, st>>>(v, s, it);
    return hipGetLastError();
}

hipError_t launch_team(const Views& v, const Shape& s, uint32_t it, hipStream_t st) {
    const int q = (((s.n + 3) >> 2) + kWave - 1) / kWave;
    if (q <= 1) return launch_team_t<1, 1>(v, s, it, st);
    if (q <= 2) return launch_team_t<1, 2>(v, s, it, st);
    const int waves = q <= 4 ? 4 : q <= 8 ? 8 : 16;
    if ((int64_t)s.ants * waves <= 2 * (int64_t)device_attr(g_simds, hipDeviceAttributeMultiprocessorCount, 4, 0))
        return waves == 4   ? launch_team_t<4, 1>(v, s, it, st)
               : waves == 8 ? launch_team_t<8, 1>(v, s, it, st)
                            : launch_team_t<16, 1>(v, s, it, st);
    if (q <= 3) return launch_team_t<1, 3>(v, s, it, st);
    if (q <= 4) return launch_team_t<1, 4>(v, s, it, st);
    if (q <= 6) return launch_team_t<2, 3>(v, s, it, st);
    if (q <= 8) return launch_team_t<2, 4>(v, s, it, st);
    if (q <= 12) return launch_team_t<4, 3>(v, s, it, st);
    return launch_team_t<4, 4>(v, s, it, st);
}

template <int kTabu, int kPher>
hipError_t launch_tp(const Views& v, const Shape& s, uint32_t it, hipStream_t st) {
    if (kPher == MMAS_PHER_DENSE && team_ok(s)) return launch_team(v, s, it, st);
    if (pair_ok(s)) return launch_t<kTabu, kPher, true>(v, s, it, st);
    const int waves = construct_waves(s);
    if (waves > 1) return launch_wide<kTabu, kPher>(v, s, it, waves, st);
    if (s.cl > 16 && s.cl <= 32) return launch_t<kTabu, kPher, false, 2, 8>(v, s, it, st);
    if (s.cl > 8 && s.cl <= 16) return launch_t<kTabu, kPher, false, 2, 4>(v, s, it, st);
    if (s.cl <= 32) return launch_t<kTabu, kPher, false, 2>(v, s, it, st);
    return launch_t<kTabu, kPher, false, 4>(v, s, it, st);
}

// the persistent batched kernel for a configuration
template <int kTabu, int kPher>
const void* batch_kernel_t(bool pair, bool table) {
    if (pair)
        return table ? (const void*)k_batch_construct<kTabu, kPher, true, true>
                     : (const void*)k_batch_construct<kTabu, kPher, true, false>;
    return table ? (const void*)k_batch_construct<kTabu, kPher, false, true>
                 : (const void*)k_batch_construct<kTabu, kPher, false, false>;
}

const void* batch_kernel(int tabu, int pher, bool pair, bool table) {
    const bool dense = pher == MMAS_PHER_DENSE;
    if (tabu == MMAS_TABU_BITMASK)
        return dense ? batch_kernel_t<MMAS_TABU_BITMASK, MMAS_PHER_DENSE>(pair, table)
                     : batch_kernel_t<MMAS_TABU_BITMASK, MMAS_PHER_CANDIDATES>(pair, table);
    if (tabu == MMAS_TABU_COMPACT)
        return dense ? batch_kernel_t<MMAS_TABU_COMPACT, MMAS_PHER_DENSE>(pair, table)
                     : batch_kernel_t<MMAS_TABU_COMPACT, MMAS_PHER_CANDIDATES>(pair, table);
    return dense ? batch_kernel_t<MMAS_TABU_LIST, MMAS_PHER_DENSE>(pair, table)
                 : batch_kernel_t<MMAS_TABU_LIST, MMAS_PHER_CANDIDATES>(pair, table);
}

}  // namespace

size_t construct_lds_per_ant(const Shape& s) {
    // draws; tabu (bitmask words, or compact entries); for the bitmask, the
    // list of unvisited cities built in a fallback
    const int bits = align16(4 * ((s.n + 31) / 32));
    const int tab = s.tabu == MMAS_TABU_BITMASK ? bits + align16(2 * list_cap(s.n, s.list_cap))
                    : s.tabu == MMAS_TABU_COMPACT ? align16(2 * s.n) : align16(4 * s.n);
    return kDrawBytes + kScratchBytes + tab;
}

size_t wide_lds_per_ant(const Shape& s) {
    // as construct_lds_per_ant, with room to list every unvisited city at once
    const int bits = align16(4 * ((s.n + 31) / 32));
    const int list = align16(2 * s.n);
    const int tab = s.tabu == MMAS_TABU_BITMASK ? bits + list : s.tabu == MMAS_TABU_COMPACT ? list : align16(4 * s.n);
    return kDrawBytes + kScratchBytes + tab;
}

hipError_t launch_batch_construct(const BatchItem* items, const BatchTile* tiles, int ntiles, uint32_t* queue,
                                  const uint32_t* it_dev, int tabu, int pher, int ants_per_block, int lanes_per_ant,
                                  int table_bytes, int per_ant, int grid, hipStream_t st) {
    const size_t bytes = (size_t)table_bytes + (size_t)ants_per_block * per_ant;
    const bool pair = lanes_per_ant == 32;
    const void* kern = batch_kernel(tabu, pher, pair, table_bytes > 0);
    // the LDS limit was raised by batch_construct_grid for this footprint (a
    // graph capture must not need it here)
    void* args[] = {(void*)&items, (void*)&tiles, (void*)&ntiles, (void*)&queue, (void*)&it_dev,
                    (void*)&ants_per_block, (void*)&table_bytes, (void*)&per_ant};
    return hipLaunchKernel(kern, dim3(grid), dim3(64 * (pair ? ants_per_block / 2 : ants_per_block)), args, bytes, st);
}

int batch_construct_grid(int tabu, int pher, int ants_per_block, int lanes_per_ant, int table_bytes, int per_ant) {
    const int lds_bytes = table_bytes + ants_per_block * per_ant;
    const bool pair = lanes_per_ant == 32;
    const void* kern = batch_kernel(tabu, pher, pair, table_bytes > 0);
    if (lds_bytes > 64 * 1024 &&
        hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes) != hipSuccess) {
        (void)hipGetLastError();  // do not leave the error for the next launch check
        return 0;
    }
    int per_cu = 0, dev = 0, cus = 0;
    const int threads = 64 * (pair ? ants_per_block / 2 : ants_per_block);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, lds_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return per_cu * cus;
}

namespace {

// ---- the parallel roulette wheel (Sec. 4.2.1), the paper's baseline ---------

// Inclusive prefix sum of FP32 values over the wave: a log-step scan within
// each row of 16 (lanes below the shift add 0), then every row adds the
// totals of the rows before it, in a fixed order.
__device__ __forceinline__ float wave_scan_f32(float x, int lane) {
    x = x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xF, 0xF, false));
    x = x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xF, 0xF, false));
    x = x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xF, 0xF, false));
    x = x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xF, 0xF, false));
    const float t0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 15));
    const float t1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 31));
    const float t2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 47));
    const int row = lane >> 4;
    float add = 0.0f;
    if (row >= 1) add = t0;
    if (row >= 2) add = add + t1;
    if (row >= 3) add = add + t2;
    return x + add;
}

// The wheel over entries 0 .. m-1 of `list` with weights wt(list[i]): 64
// chunks of ceil(len/64) a stage (chunk sums left to right), their prefix
// sums, target u times the total, the first chunk whose prefix exceeds it
// (the last with a positive sum if rounding leaves none), the target less the
// prefix before it, and again inside that chunk until a chunk is one entry.
// Returns the entry; 0 if every weight is 0.
template <class W>
__device__ int prwm_list(const uint16_t* list, int m, const W& wt, float u, int lane) {
    int lo = 0, len = m;
    float target = 0.0f;
    bool first = true;
    for (;;) {
        const int c = (len + 63) >> 6;
        float a = 0.0f;
        const int q1 = (lane + 1) * c < len ? (lane + 1) * c : len;
        for (int q = lane * c; q < q1; ++q) a = a + wt((uint32_t)list[lo + q]);
        const float P = wave_scan_f32(a, lane);
        if (first) {
            const uint64_t pos = __ballot(a > 0.0f);
            if (pos == 0ull) return 0;
            target = u * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(P), 63));
            first = false;
        }
        const uint64_t over = __ballot((P > target) & (a > 0.0f));
        const uint64_t pos = __ballot(a > 0.0f);
        const int win = over ? (int)__builtin_ctzll(over) : pos ? 63 - (int)__builtin_clzll(pos) : 0;
        if (win > 0) target = target - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(P), win - 1));
        lo += win * c;
        if (c == 1) return lo;
        len = len - win * c < c ? len - win * c : c;
    }
}

// One ant per wave, bitmask tabu and the full list of unvisited cities in
// LDS (the wheel's chunks follow the ascending city order), rows read from
// global memory. One draw per step (slot 0).
template <int kPher>
__global__ __launch_bounds__(256) void k_construct_prwm(Views vw, Shape s, uint32_t it, int ants_per_block,
                                                        int per_ant) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ant = blockIdx.x * ants_per_block + wave;
    if (ant >= s.ants) return;
    const int n = s.n, cl = s.cl;
    uint8_t* region = smem + (size_t)wave * per_ant;
    BitmaskTabu tabu;
    tabu.init(region, n, lane);
    uint16_t* ulist = reinterpret_cast<uint16_t*>(region + align16(4 * ((n + 31) / 32)));
    float tmin_a = 0.0f;
    if (kPher == MMAS_PHER_CANDIDATES) tmin_a = powi(vw.state->tau_min, s.alpha);
    const uint32_t x0 = draw_block(s.seed, it, (uint32_t)ant, 0u, 0u).w[0];
    const uint32_t start = (uint32_t)(((uint64_t)x0 * (uint64_t)n) >> 32);
    tabu.mark(start, lane);
    uint16_t* tour_out = vw.tours + (size_t)ant * n;
    const int32_t* dist = vw.dist;
    uint32_t tbuf = start, prev_last = 0, cur = start;
    int64_t len = 0, fb_steps = 0, fb_nodes = 0;
    for (int k = 1; k < n; ++k) {
        const float u = u01(draw_block(s.seed, it, (uint32_t)ant, (uint32_t)k, 0u).w[0]);
        uint32_t next = kNone;
        if (cl > 0) {
            const int e = (int)cur * cl + (lane < cl ? lane : cl - 1);
            const uint32_t node = vw.cand[e];
            const float w = vw.chc[e];
            const float a = ((lane < cl) & !tabu.visited(node)) ? w : 0.0f;
            const uint64_t pos = __ballot(a > 0.0f);
            if (pos) {
                const float P = wave_scan_f32(a, lane);
                const float target = u * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(P), 63));
                const uint64_t over = __ballot((P > target) & (a > 0.0f));
                const int win = over ? (int)__builtin_ctzll(over) : 63 - (int)__builtin_clzll(pos);
                next = (uint32_t)__builtin_amdgcn_readlane((int)node, win);
            }
        }
        if (next == kNone) {
            fb_steps += 1;
            fb_nodes += n - k;
            // every unvisited city, ascending (one pass: the list has room for n)
            const int words = (n + 31) >> 5;
            int L = 0;
            for (int w0 = 0; w0 < words; w0 += kWave) {
                const int wi = w0 + lane;
                uint32_t fr = 0u;
                if (wi < words) {
                    fr = ~tabu.bits[wi];
                    if (wi == words - 1 && (n & 31)) fr &= (1u << (n & 31)) - 1u;
                }
                const int cnt = __popc(fr);
                const int incl = wave_incl_scan(cnt, lane);
                int p = L + incl - cnt;
                while (fr) {
                    const int b = __ffs(fr) - 1;
                    fr &= fr - 1u;
                    ulist[p++] = (uint16_t)(wi * 32 + b);
                }
                L += __builtin_amdgcn_readlane(incl, 63);
            }
            int pick;
            if constexpr (kPher == MMAS_PHER_DENSE) {
                const DenseWeight wt{vw.choice + (size_t)cur * n};
                pick = prwm_list(ulist, L, wt, u, lane);
            } else {
                const CandWeight wt{dist + (size_t)cur * n, tmin_a, s.beta};
                pick = prwm_list(ulist, L, wt, u, lane);
            }
            next = L > 0 ? (uint32_t)ulist[pick] : kNone;
        }
        next = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
        if (next >= (uint32_t)n) {
            if (lane == 0) atomicOr(&vw.state->flags, 8u);
            return;
        }
        tabu.mark(next, lane);
        const int slot = k & 63;
        if (lane == slot) tbuf = next;
        cur = next;
        if (slot == 63 || k == n - 1) {
            const int k0 = k - slot;
            const uint32_t prev = __shfl_up(tbuf, 1);
            if (lane <= slot) {
                tour_out[k0 + lane] = (uint16_t)tbuf;
                const uint32_t from = lane == 0 ? prev_last : prev;
                if (k0 + lane > 0) len += dist[(size_t)from * n + tbuf];
            }
            prev_last = (uint32_t)__builtin_amdgcn_readlane((int)tbuf, slot);
        }
    }
    if (lane == 0) len += dist[(size_t)cur * n + start];
    len = wave_sum_i64(len);
    if (lane == 0) {
        vw.lengths[ant] = len;
        vw.fallback[ant] = fb_steps;
        vw.fallback[s.ants + ant] = fb_nodes;
    }
}

template <int kPher>
hipError_t launch_prwm(const Views& v, const Shape& s, uint32_t it, hipStream_t st) {
    const int per_ant = align16(4 * ((s.n + 31) / 32)) + align16(2 * s.n);
    const int budget = max_lds_per_block();
    int apb = 4;
    while (apb > 1 && apb * per_ant > budget) --apb;
    if (apb * per_ant > budget) return hipErrorInvalidValue;
    const size_t bytes = (size_t)apb * per_ant;
    auto kern = k_construct_prwm<kPher>;
    if (bytes > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    kern<<<(s.ants + apb - 1) / apb, 64 * apb, bytes, st>>>(v, s, it, apb, per_ant);
    return hipGetLastError();
}

// One wave marks marks[0 .. count) in a fresh tabu of n cities, in order, then
// writes visited[v] for every city, the tabu's cells (bitmask: its 32-bit
// words as pairs of 16-bit halves, low first; compact: entries[0 .. n); list:
// unv[0 .. n) then idx[0 .. n)) and the unvisited count (-1 if a mark was out
// of range or already visited: the marking stops there).
template <int kTabu>
__global__ __launch_bounds__(64) void k_eval_tabu(int n, const int32_t* __restrict__ marks, int count,
                                                  uint8_t* __restrict__ visited, uint16_t* __restrict__ state,
                                                  int32_t* __restrict__ left) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x;
    typename TabuOf<kTabu>::type tabu;
    tabu.init(smem, n, lane);
    int bad = 0;
    for (int q = 0; q < count; ++q) {
        const int u = __builtin_amdgcn_readfirstlane(marks[q]);
        if (u < 0 || u >= n || tabu.visited((uint32_t)u)) {
            bad = 1;
            break;
        }
        tabu.mark((uint32_t)u, lane);
    }
    for (int v = lane; v < n; v += kWave) visited[v] = tabu.visited((uint32_t)v) ? 1 : 0;
    if constexpr (kTabu == MMAS_TABU_BITMASK) {
        for (int w = lane; w < (n + 31) / 32; w += kWave) {
            state[2 * w] = (uint16_t)(tabu.bits[w] & 0xFFFFu);
            state[2 * w + 1] = (uint16_t)(tabu.bits[w] >> 16);
        }
    } else if constexpr (kTabu == MMAS_TABU_COMPACT) {
        for (int v = lane; v < n; v += kWave) state[v] = tabu.entries[v];
    } else {
        for (int v = lane; v < n; v += kWave) {
            state[v] = tabu.unv[v];
            state[n + v] = tabu.idx[v];
        }
    }
    if (lane == 0) *left = bad ? -1 : n - count;
}

}  // namespace

hipError_t launch_eval_tabu(int tabu, int n, const int32_t* marks, int count, uint8_t* visited, uint16_t* state,
                            int32_t* left, hipStream_t st) {
    const size_t bytes = tabu == MMAS_TABU_BITMASK ? (size_t)align16(4 * ((n + 31) / 32))
                                                   : (size_t)align16((tabu == MMAS_TABU_COMPACT ? 2 : 4) * n);
    if (tabu == MMAS_TABU_BITMASK)
        k_eval_tabu<MMAS_TABU_BITMASK><<<1, kWave, bytes, st>>>(n, marks, count, visited, state, left);
    else if (tabu == MMAS_TABU_COMPACT)
        k_eval_tabu<MMAS_TABU_COMPACT><<<1, kWave, bytes, st>>>(n, marks, count, visited, state, left);
    else
        k_eval_tabu<MMAS_TABU_LIST><<<1, kWave, bytes, st>>>(n, marks, count, visited, state, left);
    return hipGetLastError();
}

hipError_t launch_construct(const Views& v, const Shape& s, uint32_t it, hipStream_t st) {
    if (s.select == MMAS_SELECT_PRWM)
        return s.pher == MMAS_PHER_DENSE ? launch_prwm<MMAS_PHER_DENSE>(v, s, it, st)
                                         : launch_prwm<MMAS_PHER_CANDIDATES>(v, s, it, st);
    if (s.tabu == MMAS_TABU_BITMASK) {
        return s.pher == MMAS_PHER_DENSE ? launch_tp<MMAS_TABU_BITMASK, MMAS_PHER_DENSE>(v, s, it, st)
                                         : launch_tp<MMAS_TABU_BITMASK, MMAS_PHER_CANDIDATES>(v, s, it, st);
    }
    if (s.tabu == MMAS_TABU_COMPACT) {
        return s.pher == MMAS_PHER_DENSE ? launch_tp<MMAS_TABU_COMPACT, MMAS_PHER_DENSE>(v, s, it, st)
                                         : launch_tp<MMAS_TABU_COMPACT, MMAS_PHER_CANDIDATES>(v, s, it, st);
    }
    return s.pher == MMAS_PHER_DENSE ? launch_tp<MMAS_TABU_LIST, MMAS_PHER_DENSE>(v, s, it, st)
                                     : launch_tp<MMAS_TABU_LIST, MMAS_PHER_CANDIDATES>(v, s, it, st);
}

}  // namespace mmas
