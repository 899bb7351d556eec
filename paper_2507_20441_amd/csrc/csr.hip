// Graph build: validation, the canonical edge order and the per-vertex lists.
//
// The paper stores the graph as per-vertex in/out edge lists sorted by time,
// searched by binary search (Sec. 4, storage paragraph), with timestamps
// shifted to start at 0.  Here every list is built by stable LSD radix sorts
// so that the order inside each list is the canonical eid order; each sort
// carries the edge fields its lists need (time, eid, neighbour), so the list
// arrays come out of the sorts in order and only the two inverse
// permutations (an edge's T position) are written or read at random.
#include <algorithm>
#include <cstdio>
#include <cstring>

#include "tm_primitives.h"

namespace {

enum : int { kBadRange = 1, kSelfLoop = 2, kDup = 4 };

// The build's words on the device: the flags above, the sorts' error word, the
// edges of long runs (decode_ties_kernel).
enum : int { kFlags, kSortErr, kLongEdges, kFlagWords };

__device__ __forceinline__ u64 order_key(int64_t t) { return (u64)t ^ 0x8000000000000000ull; }

// Per workgroup: flags and the time range of its edges, as one partial each
// (part[3 b] = min, part[3 b + 1] = max, part[3 b + 2] = flags).
__global__ void __launch_bounds__(kBlock)
validate_kernel(const int32_t* src, const int32_t* dst, const int64_t* t, int64_t m, int32_t n, u64* part) {
    u64 lo = ~0ull, hi = 0;
    int f = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * kBlock) {
        const int32_t u = src[i], v = dst[i];
        if (u < 0 || u >= n || v < 0 || v >= n) f |= kBadRange;
        if (u == v) f |= kSelfLoop;
        const u64 k = order_key(t[i]);
        lo = k < lo ? k : lo;
        hi = k > hi ? k : hi;
    }
    for (int d = 32; d > 0; d >>= 1) {
        const u64 a = __shfl_xor(lo, d, 64), b = __shfl_xor(hi, d, 64);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
        f |= __shfl_xor(f, d, 64);
    }
    // one partial per block: the waves meet in LDS first
    __shared__ u64 slo[kWaves], shi[kWaves];
    __shared__ int sf[kWaves];
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        slo[wave] = lo;
        shi[wave] = hi;
        sf[wave] = f;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWaves; ++w) {
            lo = slo[w] < lo ? slo[w] : lo;
            hi = shi[w] > hi ? shi[w] : hi;
            f |= sf[w];
        }
        part[3 * blockIdx.x] = lo;
        part[3 * blockIdx.x + 1] = hi;
        part[3 * blockIdx.x + 2] = (u64)(uint32_t)f;
    }
}

// Times at pseudo-random edges: how many repeat one before them tells how many
// edges share a time (see graph_build).  Four times as many for large graphs,
// where few of them would repeat.
constexpr int kTieSamples = 4096;

constexpr double kTieMean = 20;

int tie_samples(int64_t m) { return m < ((int64_t)1 << 23) ? kTieSamples / 4 : kTieSamples; }

__device__ __forceinline__ int repeated_times(const int64_t* t, int64_t m, int samples) {
    constexpr int kSlots = 2 * kTieSamples;
    __shared__ uint32_t table[kSlots];  // 32 bits of a time's hash; 0: empty
    __shared__ int repeats;
    for (int i = threadIdx.x; i < kSlots; i += kBlock) table[i] = 0;
    if (threadIdx.x == 0) repeats = 0;
    __syncthreads();
    int mine = 0;
    for (int i = threadIdx.x; i < samples; i += kBlock) {
        const u64 at = __umul64hi((u64)(i + 1) * 0x9E3779B97F4A7C15ull, (u64)m);
        const u64 hash = (u64)t[at] * 0x9E3779B97F4A7C15ull;
        const uint32_t x = (uint32_t)(hash >> 32) | 1u;
        // at most kTieSamples of the kSlots fill: the probe ends
        for (uint32_t h = (uint32_t)(hash >> 40) % kSlots;; h = (h + 1) % kSlots) {
            const uint32_t old = atomicCAS(&table[h], 0u, x);
            if (old == 0) break;
            if (old == x) {
                ++mine;
                break;
            }
        }
    }
    if (mine) atomicAdd(&repeats, mine);
    __syncthreads();
    return repeats;
}

// One workgroup: the partials of nb workgroups into *flags, *tmin, *tmax, and
// *rep, the repeated times among `samples` ones.
__global__ void __launch_bounds__(kBlock)
validate_reduce_kernel(const u64* part, int nb, const int64_t* t, int64_t m, int samples, int* flags, u64* tmin,
                       u64* tmax, u64* rep) {
    const int repeats = repeated_times(t, m, samples);
    u64 lo = ~0ull, hi = 0;
    uint32_t f = 0;
    for (int b = threadIdx.x; b < nb; b += kBlock) {
        lo = part[3 * b] < lo ? part[3 * b] : lo;
        hi = part[3 * b + 1] > hi ? part[3 * b + 1] : hi;
        f |= (uint32_t)part[3 * b + 2];
    }
    for (int d = 32; d > 0; d >>= 1) {
        const u64 a = __shfl_xor(lo, d, 64), c = __shfl_xor(hi, d, 64);
        lo = a < lo ? a : lo;
        hi = c > hi ? c : hi;
        f |= (uint32_t)__shfl_xor((int)f, d, 64);
    }
    __shared__ u64 slo[kWaves], shi[kWaves];
    __shared__ uint32_t sf[kWaves];
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        slo[wave] = lo;
        shi[wave] = hi;
        sf[wave] = f;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWaves; ++w) {
            lo = slo[w] < lo ? slo[w] : lo;
            hi = shi[w] > hi ? shi[w] : hi;
            f |= sf[w];
        }
        *tmin = lo;
        *tmax = hi;
        *rep = (u64)repeats;
        *flags = (int)f;
    }
}

// Sort keys for the canonical order (t, u, v): one packed key t << 2bn |
// u << bn | v when it fits 64 bits, else the key u << bn | v with the time
// carried beside it (a second sort then orders by time).
__global__ void canon_keys_kernel(const int32_t* src, const int32_t* dst, const int64_t* t, int64_t m, int64_t tmin,
                                  int bn, int one_key, u64* keys, u64* times) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= m) return;
    u64 k = ((u64)(uint32_t)src[i] << bn) | (u64)(uint32_t)dst[i];
    if (one_key)
        k |= (u64)(t[i] - tmin) << (2 * bn);
    else
        times[i] = (u64)(t[i] - tmin);
    keys[i] = k;
}

// Edge arrays from the sorted packed keys, and the duplicate check on
// neighbours.
// (ot32, when not null: the times again in 32 bits, for the list sorts)
__global__ void decode_packed_kernel(const u64* key, int64_t m, int bn, int32_t* osrc, int32_t* odst, int64_t* ot,
                                     uint32_t* ot32, int* flags) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    const u64 k = key[e];
    const u64 mask = (1ull << bn) - 1;
    osrc[e] = (int32_t)((k >> bn) & mask);
    odst[e] = (int32_t)(k & mask);
    ot[e] = (int64_t)(k >> (2 * bn));
    if (ot32) ot32[e] = (uint32_t)(k >> (2 * bn));
    if (e > 0 && key[e - 1] == k) atomicOr(flags, kDup);
}

// Edge arrays from keys in time order only: an edge's place among the edges of
// its time is the number of smaller (u, v) there, counted by reading them all
// (the average time of the graphs that come here holds a few edges).  The edges
// of a time with more than kTieMax go to a list instead, counted in
// words[kLongEdges] and kept while it holds at most cap, which the caller
// sorts (decode_long_kernel).  Every edge of a run of equal times finds its
// length, or that it exceeds kTieMax, so a run is placed or listed as a whole.
// key: the packed keys (uv null), or the times with the (u, v) keys beside.
constexpr int kTieMax = 256;

__global__ void __launch_bounds__(kBlock)
decode_ties_kernel(const u64* key, const u64* uv, int64_t m, int bn, int32_t* osrc, int32_t* odst, int64_t* ot,
                   uint32_t* ot32, int* words, u64* lkey, u64* luv, int64_t cap) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int tshift = uv ? 0 : 2 * bn;
    const u64* order = uv ? uv : key;  // equal times: order by these
    const bool edge = e < m;
    const u64 t = edge ? key[e] >> tshift : 0, k = edge ? order[e] : 0;
    int64_t l = e - 1, r = e + 1;
    int less = 0;
    bool dup = false;
    // a run that reaches kTieMax further on a side shows there at once
    bool over = edge && ((e >= kTieMax && (key[e - kTieMax] >> tshift) == t) ||
                         (e + kTieMax < m && (key[e + kTieMax] >> tshift) == t));
    // (of equal keys, an error, the earlier one comes first: every position of
    // the edge arrays is written, whatever the input)
    for (; edge && !over && l >= 0 && (key[l] >> tshift) == t; --l) {
        over = r - l > kTieMax;  // e, those between and l
        less += order[l] <= k ? 1 : 0;
        dup = dup || order[l] == k;
    }
    for (; edge && !over && r < m && (key[r] >> tshift) == t; ++r) {
        over = r - l > kTieMax;
        less += order[r] < k ? 1 : 0;
        dup = dup || order[r] == k;
    }
    // one atomic per wave
    if (__ballot(dup && !over) && lane == 0) atomicOr(&words[kFlags], kDup);
    if (const u64 overs = __ballot(over)) {
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(reinterpret_cast<uint32_t*>(&words[kLongEdges]), (uint32_t)__popcll(overs));
        const int64_t at = (int64_t)__shfl(base, 0, 64) + __popcll(overs & (lane ? ~0ull >> (64 - lane) : 0ull));
        if (over && at < cap) {
            lkey[at] = key[e];
            if (luv) luv[at] = k;
        }
    }
    if (!edge || over) return;
    const int64_t at = l + 1 + less;  // inside the edges looked at
    const u64 mask = (1ull << bn) - 1;
    osrc[at] = (int32_t)((k >> bn) & mask);
    odst[at] = (int32_t)(k & mask);
    ot[at] = (int64_t)t;
    if (ot32) ot32[at] = (uint32_t)t;
}

// The first of n keys in time order whose time is at or past t.
__device__ __forceinline__ int64_t first_at(const u64* key, int64_t n, int tshift, u64 t) {
    int64_t a = 0;
    while (n > 0) {
        const int64_t h = n >> 1;
        const bool up = (key[a + h] >> tshift) < t;
        a = up ? a + h + 1 : a;
        n = up ? n - h - 1 : h;
    }
    return a;
}

// The c listed edges of long runs, in canonical order (lkey, luv), to their
// places: as far after the first edge of their time among all edges (key, in
// time order) as after the first of it in the list.
__global__ void __launch_bounds__(kBlock)
decode_long_kernel(const u64* lkey, const u64* luv, int64_t c, const u64* key, int64_t m, int bn, int32_t* osrc,
                   int32_t* odst, int64_t* ot, uint32_t* ot32, int* words) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= c) return;
    const int tshift = luv ? 0 : 2 * bn;
    const u64* order = luv ? luv : lkey;
    const u64 t = lkey[j] >> tshift, k = order[j];
    if (j > 0 && order[j - 1] == k && (lkey[j - 1] >> tshift) == t) atomicOr(&words[kFlags], kDup);
    const int64_t at = first_at(key, m, tshift, t) + (j - first_at(lkey, c, tshift, t));
    if (at < 0 || at >= m) return;  // (a broken order must not write outside)
    const u64 mask = (1ull << bn) - 1;
    osrc[at] = (int32_t)((k >> bn) & mask);
    odst[at] = (int32_t)(k & mask);
    ot[at] = (int64_t)t;
    if (ot32) ot32[at] = (uint32_t)t;
}

// Edge arrays from the sorted times and the (u, v) keys carried with them.
__global__ void decode_split_kernel(const u64* tsorted, const u64* uv, int64_t m, int bn, int32_t* osrc,
                                    int32_t* odst, int64_t* ot, uint32_t* ot32, int* flags) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    const u64 k = uv[e], t = tsorted[e];
    const u64 mask = (1ull << bn) - 1;
    osrc[e] = (int32_t)(k >> bn);
    odst[e] = (int32_t)(k & mask);
    ot[e] = (int64_t)t;
    if (ot32) ot32[e] = (uint32_t)t;
    if (e > 0 && uv[e - 1] == k && tsorted[e - 1] == t) atomicOr(flags, kDup);
}

// out[from .. to) = v for every lane of the wave (an empty range writes
// nothing): short ranges lane by lane, long ones by the whole wave.  Every
// lane of the wave calls it.
__device__ __forceinline__ void wave_fill(int32_t* out, int64_t from, int64_t to, int32_t v) {
    const bool big = to - from > 64;
    if (!big)
        for (int64_t i = from; i < to; ++i) out[i] = v;
    for (u64 todo = __ballot(big); todo; todo &= todo - 1) {
        const int src = __ffsll(todo) - 1;
        const int64_t f = __shfl((long long)from, src, 64), t = __shfl((long long)to, src, 64);
        const int32_t w = __shfl(v, src, 64);
        for (int64_t i = f + (threadIdx.x & 63); i < t; i += 64) out[i] = w;
    }
}

// Search guide of one list order (see DevGraph): position p writes the
// entries after the previous position's slice up to its own, the last
// position also those after it.  own: the list owners in order, key(p) the
// time or neighbour at p.
template <typename F>
__device__ __forceinline__ void guide_fill(const uint32_t* own, const int32_t* off, int64_t m, int32_t n, int64_t p,
                                           const F& key, int bits, uint32_t mul, int32_t* guide) {
    auto entry = [&](int64_t i) -> int64_t {
        // (clamped: a broken order must not write outside the guide)
        const int32_t g = own[i] < (uint32_t)n ? (int32_t)own[i] : n - 1;
        const int32_t a = off[g], b = off[g + 1];
        const int32_t ns = guide_slices(a, b);
        const int64_t at = guide_first(g, a) + slice_of(slice_frac(key(i), bits, mul), ns > 0 ? ns : 1);
        const int64_t last = guide_first(n, (int32_t)m);
        return at < 0 ? 0 : (at > last ? last : at);
    };
    int64_t to = 0, end = 0;
    if (p < m) {
        to = entry(p) + 1;
        if (p == m - 1) end = guide_first(n, (int32_t)m) + 1;
    }
    // the previous position's is the lane's before (the wave's first looks itself)
    int64_t from = __shfl_up((long long)to, 1, 64);
    if ((threadIdx.x & 63) == 0) from = p == 0 || p >= m ? 0 : entry(p - 1) + 1;
    if (p >= m) from = 0;
    wave_fill(guide, from, to, (int32_t)p);
    wave_fill(guide, to, end, (int32_t)m);
}

// What follows a T-order sort, in one pass over the positions of each
// direction (blockIdx.y): the (neighbour, time) records of 32-bit lists, and by
// eid the edge's position (the inverse of leid); each where it is asked for.
//
// The positions' scattered writes are its time.  Up to 2^26 edges everything
// goes in one launch; above, where an array of positions no longer fits the
// 256 MB cache behind the L2s, the records' stream and the other direction's
// writes push it out, and the four parts go one after the other (1e8 edges 6.0
// and 4.8 ms, 2e7 0.60 and 0.73 ms).
constexpr int64_t kFinishTogether = (int64_t)1 << 26;

template <typename TT>
struct ListFinish {
    const int32_t* leid;
    const uint32_t* nbr;
    const TT* t;
    int32_t* pos;
    uint2* nt;
};

template <typename TT>
__global__ void __launch_bounds__(kBlock) list_finish_kernel(ListFinish<TT> f0, ListFinish<TT> f1, int64_t m) {
    const int y = blockIdx.y;
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= m) return;
    const int32_t e = pick_arg(f0.leid, f1.leid, y)[p];
    uint2* nt = pick_arg(f0.nt, f1.nt, y);
    if (nt) nt[p] = make_uint2(pick_arg(f0.nbr, f1.nbr, y)[p], (uint32_t)pick_arg(f0.t, f1.t, y)[p]);
    int32_t* pos = pick_arg(f0.pos, f1.pos, y);
    if (pos && (uint32_t)e < (uint64_t)m) pos[e] = (int32_t)p;
}

// N order (of one direction, or of both: blockIdx.y): the packed key from the
// carried neighbour and time (time: the carried times, which may be nkey
// itself), each entry's position in the direction's T order, and the guides by
// neighbour and by time.  own: the owners, the same sequence in both orders;
// tt: the T order's times.
//
// The positions are random reads and the kernel's time; the guides' own reads
// and stores pass beside them (2e7 edges, per direction: 419 us without guides,
// 455 with both).  Beside the scattered position writes of list_finish_kernel
// the guides by time cost it 100 us there, as a load after such a store waits for
// it.
template <typename TT>
struct NOrderFix {
    const uint32_t* nbr;
    const TT* time;
    const int32_t* neid;
    const int32_t* tpos;
    const uint32_t* own;
    const int32_t* off;
    const TT* tt;
    u64* nkey;
    int32_t* nxref;
    int32_t* nguide;
    int32_t* tguide;
};

template <typename TT>
__global__ void __launch_bounds__(kBlock)
n_order_fix_kernel(NOrderFix<TT> f0, NOrderFix<TT> f1, int64_t m, int32_t n, int bt, int bn, uint32_t tmul,
                   uint32_t nmul) {
    const int y = blockIdx.y;
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint32_t* nbr = pick_arg(f0.nbr, f1.nbr, y);
    if (q < m) {
        pick_arg(f0.nkey, f1.nkey, y)[q] = ((u64)nbr[q] << bt) | (u64)pick_arg(f0.time, f1.time, y)[q];
        const int32_t e = pick_arg(f0.neid, f1.neid, y)[q];
        pick_arg(f0.nxref, f1.nxref, y)[q] = (uint32_t)e < (uint64_t)m ? pick_arg(f0.tpos, f1.tpos, y)[e] : -1;
    }
    int32_t* nguide = pick_arg(f0.nguide, f1.nguide, y);
    if (!nguide) return;
    const uint32_t* own = pick_arg(f0.own, f1.own, y);
    const int32_t* off = pick_arg(f0.off, f1.off, y);
    const TT* tt = pick_arg(f0.tt, f1.tt, y);
    guide_fill(own, off, m, n, q, [&](int64_t i) { return (u64)nbr[i]; }, bn, nmul, nguide);
    guide_fill(own, off, m, n, q, [&](int64_t i) { return (u64)tt[i]; }, bt, tmul, pick_arg(f0.tguide, f1.tguide, y));
}

// The pair ranks of both lists (see DevGraph) of a finished graph, in one
// launch: thread i < m takes position i of the out-lists' N order, the next m
// those of the in-lists.  Both lists of a vertex are in (neighbour, time) order,
// so consecutive lanes search the other list at nearby keys (their probes fall
// on lines the wave shares); the lookup of the edge's T position in the other
// list and the write to its own, one record inside one line, are the scattered
// part and most of its time (6.8 ms at 1e8 edges; carrying that position through
// the list sorts instead took 4 ms there and 1.3 off the kernel).
__global__ void __launch_bounds__(kBlock)
pair_rank_kernel(DevGraph G, uint4* rank0, uint4* rank1) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t m = G.m;
    if (i >= 2 * m) return;
    const int w = i >= m ? 1 : 0;
    const int64_t q = w ? i - m : i;
    const u64* nk = w ? G.nkey[1] : G.nkey[0];
    const u64* ok = w ? G.nkey[0] : G.nkey[1];
    const int32_t g = (w ? G.lown[1] : G.lown[0])[q];  // (the same sequence in both orders)
    const int32_t* off = w ? G.off[1] : G.off[0];
    const int32_t* ooff = w ? G.off[0] : G.off[1];
    const int32_t a = ooff[g], b = ooff[g + 1];
    const u64 key = nk[q];
    const u64 o = key >> G.bt;
    // two keys of one neighbour differ by their times
    uint32_t sp = kGapNone, sn = kGapNone, rp = kGapNone, rn = kGapNone;
    if (q > 0 && q > off[g] && (nk[q - 1] >> G.bt) == o) sp = gap_code(key - nk[q - 1]);
    if (q + 1 < m && q + 1 < off[g + 1] && (nk[q + 1] >> G.bt) == o) sn = gap_code(nk[q + 1] - key);
    int32_t c = a, n = b - a;
    const int32_t* gd = w ? G.nguide[0] : G.nguide[1];
    if (gd) {
        const int32_t* e = gd + guide_first(g, a) + slice_of(slice_frac(o, G.bn, G.nmul), guide_slices(a, b));
        c = e[0];
        n = e[1] - c;
    }
    while (n > 0) {
        const int32_t h = n >> 1;
        const bool up = ok[c + h] < key;
        c = up ? c + h + 1 : c;
        n = up ? n - h - 1 : h;
    }
    if (c > a && (ok[c - 1] >> G.bt) == o) rp = gap_code(key - ok[c - 1]);
    if (c < b && (ok[c] >> G.bt) == o) rn = gap_code(ok[c] - key + 1);
    const int32_t at = (w ? G.nxref[1] : G.nxref[0])[q], e = (w ? G.neid[1] : G.neid[0])[q];
    (w ? rank1 : rank0)[at] = make_uint4((uint32_t)q, (uint32_t)c, (uint32_t)(w ? G.tpos[0] : G.tpos[1])[e],
                                         sp | (sn << 8) | (rp << 16) | (rn << 24));
}

// List offsets from the owner-sorted keys: off[v] is the first position whose
// owner is >= v.  Position p writes the offsets of the owners in
// (key[p-1], key[p]]; the last position also closes the owners after it.
// (both directions: blockIdx.y)
__global__ void offsets_kernel(const uint32_t* key0, const uint32_t* key1, int64_t m, int32_t n, int32_t* off0,
                               int32_t* off1) {
    const uint32_t* key = pick_arg(key0, key1, blockIdx.y);
    int32_t* off = pick_arg(off0, off1, blockIdx.y);
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int64_t from = 0, to = 0, end = 0;
    if (p < m) {
        // (owners are below n; the clamps keep a broken order from writing
        // outside off)
        const int64_t cur = key[p] < (uint32_t)n ? (int64_t)key[p] : (int64_t)n - 1;
        const int64_t prev = p == 0 ? -1 : (key[p - 1] < (uint32_t)n ? (int64_t)key[p - 1] : (int64_t)n - 1);
        from = prev + 1;
        to = cur + 1;
        if (p == m - 1) end = (int64_t)n + 1;
    }
    wave_fill(off, from, to, (int32_t)p);
    wave_fill(off, to, end, (int32_t)m);
}

// List sorts side by side up to this many edges (a pass of few tiles leaves the
// chip idle: a build of 2^14 edges takes 157 us with pairs and 206 without,
// 2^20 395 and 518, 2^21 649 and 836, 2^22 1255 and 1350).  Larger builds
// gain 3 to 5% (2^24 edges 4.48 and 4.65 ms) and keep the memory of the second
// buffers (28 to 32 B per edge).
constexpr int64_t kPairedSorts = (int64_t)1 << 22;

int bits_for(u64 x) {
    int b = 0;
    while (x) { ++b; x >>= 1; }
    return b;
}

unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

void graph_pair_ranks(tm_graph* g, int launches, u64 need, hipStream_t st) {
    PairRanks& R = g->ranks;
    if (g->m < kRanksFrom || g->m > kRanksTo || R.state.load(std::memory_order_acquire) != PairRanks::kNone ||
        dev_deferring())
        return;
    const bool pays = R.launches.fetch_add(launches) + launches >= kRankAllLaunches ||
                      (launches >= kRankLaunches && g->m >= kRanksAtOnce);
    if (!pays) return;
    int none = PairRanks::kNone;
    if (!R.state.compare_exchange_strong(none, PairRanks::kBusy)) return;  // another thread makes them
    AllocScope scope_(alloc_of(g));
    R.arena.stream = st;
    uint4* rank[2] = {nullptr, nullptr};
    bool ok = g->has_alloc || dev_room() >= need + 2 * (u64)g->m * sizeof(uint4);
    for (uint4*& r : rank) ok = ok && arena_alloc(R.arena, &r, (size_t)g->m) == TM_OK;
    if (ok) {
        hipLaunchKernelGGL(pair_rank_kernel, dim3(grid_for(2 * g->m)), dim3(kBlock), 0, st, g->d, rank[0], rank[1]);
        ok = hipGetLastError() == hipSuccess;
        // (from here on every stream may read them)
        ok = sync_stream(st) == hipSuccess && ok;
    }
    if (!ok) R.arena.release();
    R.arena.stream = g->arena.stream;
    for (int dir = 0; dir < 2; ++dir) R.rank[dir] = ok ? rank[dir] : nullptr;
    R.state.store(ok ? PairRanks::kReady : PairRanks::kGivenUp, std::memory_order_release);
}

DevGraph graph_view(const tm_graph* g) {
    DevGraph D = g->d;
    if (g->ranks.state.load(std::memory_order_acquire) == PairRanks::kReady)
        for (int dir = 0; dir < 2; ++dir) D.nrank[dir] = g->ranks.rank[dir];
    return D;
}

int graph_build(tm_graph* g, const int32_t* src, const int32_t* dst, const int64_t* t, hipStream_t st) {
    const int64_t m = g->m;
    const int32_t n = g->n;
    DevGraph& D = g->d;
    D.m = m;
    D.n = n;
    if (m == 0) {
        // empty graph: empty lists, every offset 0
        g->shift = 0;
        g->T = 0;
        D.T = 0;
        D.bt = 1;
        for (int dir = 0; dir < 2; ++dir) {
            int32_t* off;
            TM_TRY(arena_alloc(g->arena, &off, (size_t)n + 1));
            TM_HIP(hipMemsetAsync(off, 0, ((size_t)n + 1) * sizeof(int32_t), st));
            D.off[dir] = off;
        }
        TM_HIP(sync_stream(st));
        return TM_OK;
    }

    StageTimer timer;
    timer.start(TM_STAGE_GRAPH, st);
    // --- validation: ids, self loops, time span -------------------------
    int* flags = nullptr;
    u64* tbounds = nullptr;
    TM_HIP(dev_alloc((void**)&flags, sizeof(int) * kFlagWords, st));
    TM_HIP(dev_alloc((void**)&tbounds, sizeof(u64) * 3, st));
    TM_HIP(hipMemsetAsync(flags, 0, sizeof(int) * kFlagWords, st));
    {
        const unsigned blocks = (unsigned)std::min<int64_t>(grid_for(m), 1024);
        u64* part = nullptr;
        TM_HIP(dev_alloc((void**)&part, (size_t)blocks * 3 * sizeof(u64), st));
        hipLaunchKernelGGL(validate_kernel, dim3(blocks), dim3(kBlock), 0, st, src, dst, t, m, n, part);
        TM_HIP(hipGetLastError());
        hipLaunchKernelGGL(validate_reduce_kernel, dim3(1), dim3(kBlock), 0, st, (const u64*)part, (int)blocks,
                           t, m, tie_samples(m), flags, tbounds, tbounds + 1, tbounds + 2);
        TM_HIP(hipGetLastError());
        TM_HIP(dev_free(part, st));
    }
    // error exits return the flag words to the cache
    auto bail = [&](int r) {
        (void)dev_free(flags, st);
        (void)dev_free(tbounds, st);
        return r;
    };
    int hflags[kFlagWords];
    u64 hb[3];
    TM_HIP(read_back({{hflags, flags, sizeof hflags}, {hb, tbounds, sizeof hb}}, st));
    if (hflags[kFlags] & kBadRange) return bail(tm_fail(TM_EINVAL, "graph: vertex id outside [0, %d)", n));
    if (hflags[kFlags] & kSelfLoop) return bail(tm_fail(TM_ESELFLOOP, "graph: self loop"));
    const int64_t tmin = (int64_t)(hb[0] ^ 0x8000000000000000ull);
    const int64_t tmax = (int64_t)(hb[1] ^ 0x8000000000000000ull);
    if ((__int128)tmax - (__int128)tmin >= ((__int128)1 << 62))
        return bail(tm_fail(TM_ERANGE, "graph: time span %lld..%lld too large", (long long)tmin, (long long)tmax));
    g->shift = tmin;
    g->T = tmax - tmin;
    D.T = g->T;
    const int bn = bits_for((u64)(n > 0 ? n - 1 : 0));
    D.bt = bits_for((u64)g->T);
    if (D.bt == 0) D.bt = 1;
    D.bn = bn;
    D.tmul = slice_scale((u64)g->T, D.bt);
    D.nmul = slice_scale((u64)(n - 1), bn);
    if (bn + D.bt > 64)
        return bail(tm_fail(TM_ERANGE, "graph: %d vertex-id bits + %d time bits exceed 64", bn, D.bt));

    // --- canonical order (t, u, v) ----------------------------------------
    // Four 64-bit work arrays serve every sort below: the canonical sorts use
    // them whole, the list sorts as halves.
    u64* work[4] = {nullptr, nullptr, nullptr, nullptr};
    uint32_t* nbr_tmp = nullptr;  // N order: the carried neighbours, when work[3] holds the owners
    // Lists keep their times in 32 bits when every shifted time is below
    // 2^32 - 1; t32e: those times by eid, the list sorts' input.
    const bool narrow = g->T < (int64_t)0xFFFFFFFFll;
    uint32_t* t32e = nullptr;
    unsigned char* scr = nullptr;     // the sorts' scratch
    unsigned char* second = nullptr;  // buffers of a second list sort
    uint32_t* nbr32[2] = {nullptr, nullptr};  // 32-bit times: the T orders' neighbours until packed
    auto release = [&]() {
        for (uint32_t*& b : nbr32) {
            if (b) (void)dev_free(b, st);
            b = nullptr;
        }
        for (u64*& w : work) {
            if (w) (void)dev_free(w, st);
            w = nullptr;
        }
        if (nbr_tmp) (void)dev_free(nbr_tmp, st);
        nbr_tmp = nullptr;
        if (scr) (void)dev_free(scr, st);
        scr = nullptr;
        if (second) (void)dev_free(second, st);
        second = nullptr;
        if (t32e) (void)dev_free(t32e, st);
        t32e = nullptr;
    };
    int rc = TM_OK;
    for (u64*& w : work)
        if (rc == TM_OK && dev_alloc((void**)&w, (size_t)m * sizeof(u64), st) != hipSuccess)
            rc = tm_fail(TM_ENOMEM, "graph: work arrays");
    if (rc == TM_OK && narrow && dev_alloc((void**)&t32e, (size_t)m * sizeof(uint32_t), st) != hipSuccess)
        rc = tm_fail(TM_ENOMEM, "graph: work arrays");
    if (rc != TM_OK) {
        release();
        return bail(rc);
    }
    int32_t *esrc = nullptr, *edst = nullptr;
    int64_t* et = nullptr;
    rc = arena_alloc(g->arena, &esrc, m);
    if (rc == TM_OK) rc = arena_alloc(g->arena, &edst, m);
    if (rc == TM_OK) rc = arena_alloc(g->arena, &et, m);
    const bool one_key = 2 * bn + D.bt <= 64;
    if (rc == TM_OK) {
        hipLaunchKernelGGL(canon_keys_kernel, dim3(grid_for(m)), dim3(kBlock), 0, st, src, dst, t, m, tmin, bn,
                           one_key ? 1 : 0, work[0], work[1]);
        if (hipGetLastError() != hipSuccess) rc = tm_fail(TM_EDEVICE, "graph: key launch");
    }
    // One block, cleared by one launch, holds every sort's scratch: the digit
    // counts and tickets of the canonical sorts (0, 1) and of the lists' by
    // source and by destination (2, 3), tickets of the N orders (4, 5; they
    // sort the same owners as the T order of their direction, so its counts
    // serve them), and the status words all of them share.  (At 20,000 edges
    // clearing, counting and starting five sorts one by one was a fifth of the
    // build.)
    constexpr int kHeads = 7;  // (6: the sort by time alone)
    const size_t scr_bytes = kHeads * kSortHeadBytes + (m <= kPairedSorts ? 2 : 1) * sort_status_bytes(m);
    uint32_t tag = 0;
    auto scratch_of = [&](int tickets, int counts) {
        SortScratch x = sort_scratch_at(scr + (size_t)tickets * kSortHeadBytes);
        x.counts = reinterpret_cast<uint32_t*>(scr + (size_t)counts * kSortHeadBytes);
        // (the directions' own when they sort side by side, with equal tags)
        const bool own = m <= kPairedSorts && tickets >= 2 && tickets < 6 && (tickets & 1);
        x.status = reinterpret_cast<u64*>(scr + kHeads * kSortHeadBytes + (own ? sort_status_bytes(m) : 0));
        x.counted = tickets >= 2 && tickets < 6;
        x.tag0 = tag;
        tag += kSortMaxPasses;
        return x;
    };
    if (rc == TM_OK && dev_alloc((void**)&scr, scr_bytes, st) != hipSuccess)
        rc = tm_fail(TM_ENOMEM, "graph: sort scratch");
    if (rc == TM_OK) rc = fill_u32(scr, (int64_t)(scr_bytes / sizeof(uint32_t)), 0u, st);
    // A sort of `count` keys between two buffer sets: the result lands in
    // `spare` after an odd number of passes, else back in `in`.
    auto sort_two = [&](const auto& in, const auto& spare, int64_t count, int lo_bit, int nbits, int which,
                        auto* res) -> int {
        const bool odd = (std::max(1, radix_passes(nbits - lo_bit)) & 1) != 0;
        *res = odd ? spare : in;
        return sort_into(in, odd ? spare : in, odd ? in : spare, count, lo_bit, nbits, 0, flags + kSortErr, st,
                         scratch_of(which, which));
    };
    using S1 = SortSet<u64>;
    using S2 = SortSet<u64, u64>;
    auto set1 = [](u64* k) {
        S1 x;
        x.k = k;
        return x;
    };
    auto set2 = [](u64* k, u64* v) {
        S2 x;
        x.k = k;
        x.v0 = v;
        return x;
    };
    // The canonical order of `count` edges, by every bit of their keys.
    // Packed keys in k0 (k1 the other buffer): *key the result, *uv null.
    // Else (u, v) keys in k0 and times in v0 (k1, v1 the other buffers): by
    // (u, v) with the time carried, then by time with (u, v) carried.
    auto order_all = [&](u64* k0, u64* v0, u64* k1, u64* v1, int64_t count, u64** key, u64** uv) -> int {
        if (one_key) {
            S1 res;
            TM_TRY(sort_two(set1(k0), set1(k1), count, 0, 2 * bn + D.bt, 0, &res));
            *key = res.k;
            *uv = nullptr;
            return TM_OK;
        }
        S2 r1, r2;
        TM_TRY(sort_two(set2(k0, v0), set2(k1, v1), count, 0, 2 * bn, 0, &r1));
        const S2 o1 = r1.k == k0 ? set2(k1, v1) : set2(k0, v0);
        TM_TRY(sort_two(set2(r1.v0, r1.k), set2(o1.k, o1.v0), count, 0, D.bt, 1, &r2));
        *key = r2.k;
        *uv = r2.v0;
        return TM_OK;
    };
    // The error that the flag words, once read, hold.
    auto flags_error = [&]() -> int {
        if (hflags[kFlags] & kDup) return tm_fail(TM_EDUP, "graph: duplicate (u, v, t) tuple");
        if (hflags[kSortErr]) return tm_fail(TM_EDEVICE, "graph: internal sort error (look-back stalled)");
        return TM_OK;
    };
    // Times first: where the average time holds few edges, a sort by the time
    // bits alone (2-4 passes instead of 5-10) leaves short runs of equal times
    // to put in order, and the edges of the few long ones are sorted apart; how
    // many those are costs a round trip to the host.  Builds with the full sort
    // and this way: 2^14 edges 162 and 157 us, 2^18 286 and 240, 2^20 480 and
    // 395, 2^22 1416 and 1255, 2^24 5.46 and 4.65 ms.  (300 edges at one time,
    // for which the full sort started over before there was the list, add 96 us
    // at 2^18 edges and 97 at 4e6; they added 186 and 474.)  It pays while fewer
    // than half of the edges are in long runs (each then costs the full sort's
    // passes on top); past that the full sort starts over.  Where the sampled
    // times say that an edge shares its time with more than kTieMean others on
    // average, it is not tried: each edge reads that many to find its place.
    // Every time held by 16, 24 and 60 edges, the full sort and this way: 4e6
    // edges 1397 and 1378, 1391 and 1425, 1372 and 1636 us; 2e7 7.00 and 6.71,
    // 6.97 and 6.95, 6.88 and 8.02 ms; 1e6 456 and 417, 458 and 432, 453 and 490
    // us.
    auto order_by_time = [&](bool* done) -> int {
        u64 *key, *uv = nullptr;
        u64 *lk, *lv = nullptr, *lk1, *lv1 = nullptr;  // the listed edges' keys and their sort's other buffers
        const int64_t cap = m / 2;
        if (one_key) {
            S1 res;
            TM_TRY(sort_two(set1(work[0]), set1(work[2]), m, 2 * bn, 2 * bn + D.bt, 6, &res));
            key = res.k;
            lk = work[1];
            lk1 = work[3];
        } else {
            S2 res;
            TM_TRY(sort_two(set2(work[1], work[0]), set2(work[2], work[3]), m, 0, D.bt, 6, &res));
            key = res.k;
            uv = res.v0;
            lk = res.k == work[1] ? work[2] : work[1];
            lv = res.k == work[1] ? work[3] : work[0];
            lk1 = lk + cap;
            lv1 = lv + cap;
        }
        hipLaunchKernelGGL(decode_ties_kernel, dim3(grid_for(m)), dim3(kBlock), 0, st, (const u64*)key,
                           (const u64*)uv, m, bn, esrc, edst, et, t32e, flags, lk, lv, cap);
        TM_HIP(hipGetLastError());
        TM_HIP(read_back({{hflags, flags, sizeof hflags}}, st));
        TM_TRY(flags_error());  // (what this refuses, no list is built for)
        const int64_t c = (int64_t)(uint32_t)hflags[kLongEdges];
        *done = c <= cap;
        if (c == 0) return TM_OK;
        if (c > cap) {
            hipLaunchKernelGGL(canon_keys_kernel, dim3(grid_for(m)), dim3(kBlock), 0, st, src, dst, t, m, tmin, bn,
                               one_key ? 1 : 0, work[0], work[1]);
            TM_HIP(hipGetLastError());
            return TM_OK;
        }
        u64 *sk, *suv;
        TM_TRY(one_key ? order_all(lk, nullptr, lk1, nullptr, c, &sk, &suv)
                       : order_all(lv, lk, lv1, lk1, c, &sk, &suv));
        hipLaunchKernelGGL(decode_long_kernel, dim3(grid_for(c)), dim3(kBlock), 0, st, (const u64*)sk,
                           (const u64*)suv, c, (const u64*)key, m, bn, esrc, edst, et, t32e, flags);
        TM_HIP(hipGetLastError());
        return TM_OK;
    };
    bool ordered = false;
    const double pairs = 0.5 * tie_samples(m) * (tie_samples(m) - 1);
    if (rc == TM_OK && m / 8 <= g->T && (double)hb[2] * (double)m <= kTieMean * pairs) rc = order_by_time(&ordered);
    if (rc == TM_OK && !ordered) {
        u64 *key = nullptr, *uv = nullptr;
        rc = order_all(work[0], work[1], work[2], work[3], m, &key, &uv);
        if (rc == TM_OK && one_key)
            hipLaunchKernelGGL(decode_packed_kernel, dim3(grid_for(m)), dim3(kBlock), 0, st, (const u64*)key, m, bn,
                               esrc, edst, et, t32e, flags);
        else if (rc == TM_OK)
            hipLaunchKernelGGL(decode_split_kernel, dim3(grid_for(m)), dim3(kBlock), 0, st, (const u64*)key,
                               (const u64*)uv, m, bn, esrc, edst, et, t32e, flags);
        if (rc == TM_OK && hipGetLastError() != hipSuccess) rc = tm_fail(TM_EDEVICE, "graph: decode launch");
    }
    if (rc != TM_OK) {
        release();
        return bail(rc);
    }
    D.src = esrc;
    D.dst = edst;
    D.t = et;

    // --- per-vertex lists ---------------------------------------------------
    // dir 0: out-lists (owner = source, neighbour = destination)
    // dir 1: in-lists  (owner = destination, neighbour = source)
    // T order: the eids stably sorted by owner, carrying time, eid and
    // neighbour, so that every list array comes out of the sort in place.
    // TT: the lists' time type (uint32_t or int64_t).
    auto build_lists = [&](auto time_tag) -> int {
        using TT = decltype(time_tag);
        using V = typename std::conditional<sizeof(TT) == 4, uint32_t, u64>::type;
        using L = SortSet<uint32_t, V, uint32_t, uint32_t>;
        // What every list needs, then what a build can go on without.
        TT* lt[2] = {nullptr, nullptr};
        int32_t *leid[2], *lnbr[2], *lown[2] = {nullptr, nullptr}, *off[2], *tpos[2], *nxref[2], *neid[2];
        uint2* nt[2] = {nullptr, nullptr};
        u64* nkey[2];
        const bool keep_own = m <= ((int64_t)1 << 28);
        if (!keep_own && dev_alloc((void**)&nbr_tmp, (size_t)m * sizeof(uint32_t), st) != hipSuccess)
            return tm_fail(TM_ENOMEM, "graph: work arrays");
        for (int dir = 0; dir < 2; ++dir) {
            TM_TRY(arena_alloc(g->arena, &lt[dir], (size_t)m));
            TM_TRY(arena_alloc(g->arena, &leid[dir], (size_t)m));
            if constexpr (sizeof(TT) == 4) {
                // the neighbours end up in the (neighbour, time) records
                if (dev_alloc((void**)&nbr32[dir], (size_t)m * sizeof(uint32_t), st) != hipSuccess)
                    return tm_fail(TM_ENOMEM, "graph: work arrays");
                lnbr[dir] = reinterpret_cast<int32_t*>(nbr32[dir]);
                TM_TRY(arena_alloc(g->arena, &nt[dir], (size_t)m));
            } else {
                TM_TRY(arena_alloc(g->arena, &lnbr[dir], (size_t)m));
            }
            if (keep_own) TM_TRY(arena_alloc(g->arena, &lown[dir], (size_t)m));
            TM_TRY(arena_alloc(g->arena, &off[dir], (size_t)n + 1));
            TM_TRY(arena_alloc(g->arena, &tpos[dir], (size_t)m));
            TM_TRY(arena_alloc(g->arena, &nkey[dir], (size_t)m));
            TM_TRY(arena_alloc(g->arena, &nxref[dir], (size_t)m));
            TM_TRY(arena_alloc(g->arena, &neid[dir], (size_t)m));
        }
        // guides pay from lists of a few entries on; with fewer edges than
        // vertices the lists are shorter than that (1e6 edges, 9e5 and 1.1e6
        // vertices: a build 511 and 503 us, a 6-chain estimate 375 and 379)
        // and the guides' entry per vertex would outweigh the edges
        int32_t *tguide[2] = {nullptr, nullptr}, *nguide[2] = {nullptr, nullptr};
        if (n <= m) {
            const size_t len = (size_t)guide_first(n, (int32_t)m) + 1;
            int32_t* block = nullptr;
            if (arena_alloc(g->arena, &block, 4 * len) == TM_OK)
                for (int dir = 0; dir < 2; ++dir) {
                    tguide[dir] = block + (2 * dir) * len;
                    nguide[dir] = block + (2 * dir + 1) * len;
                }
        }
        // Graphs of few sort tiles sort both directions side by side, with
        // buffers of their own (six 4-byte arrays and the values of type V);
        // larger ones in turn, through the same ones.
        bool paired = m <= kPairedSorts;
        if (paired && dev_alloc((void**)&second, (size_t)m * (6 * sizeof(uint32_t) + sizeof(V)), st) != hipSuccess) {
            (void)hipGetLastError();
            paired = false;
        }
        struct Bufs {
            L tmp;           // the other buffer of the list sorts
            uint32_t* nkeys;  // N order: its sorted keys (unused)
            uint32_t* ntime;  // N order: the carried 32-bit times (64-bit ones: the key array itself,
                              // packed in place afterwards)
            uint32_t* nbr;    // N order: the carried neighbours
        } buf[2];
        buf[0].tmp.k = reinterpret_cast<uint32_t*>(work[0]);
        buf[0].tmp.v1 = reinterpret_cast<uint32_t*>(work[0]) + m;
        buf[0].tmp.v0 = reinterpret_cast<V*>(work[1]);
        buf[0].tmp.v2 = reinterpret_cast<uint32_t*>(work[2]);
        buf[0].nkeys = reinterpret_cast<uint32_t*>(work[2]) + m;
        buf[0].ntime = reinterpret_cast<uint32_t*>(work[1]) + m;
        buf[0].nbr = keep_own ? reinterpret_cast<uint32_t*>(work[3]) : nbr_tmp;
        buf[1] = buf[0];
        if (paired) {
            buf[1].tmp.v0 = reinterpret_cast<V*>(second);
            uint32_t* at = reinterpret_cast<uint32_t*>(buf[1].tmp.v0 + m);
            uint32_t** const arrays[6] = {&buf[1].tmp.k, &buf[1].tmp.v1, &buf[1].tmp.v2, &buf[1].nkeys, &buf[1].ntime,
                                          &buf[1].nbr};
            for (uint32_t** x : arrays) {
                *x = at;
                at += m;
            }
        }
        uint32_t* own[2];
        for (int dir = 0; dir < 2; ++dir)
            own[dir] = keep_own ? reinterpret_cast<uint32_t*>(lown[dir])
                                : reinterpret_cast<uint32_t*>(work[3]) + dir * m;
        const SortPlan plan = sort_plan_copy(0, bn);
        // two sorts side by side, or one after the other
        auto sort_lists = [&](auto* jobs, int iota) -> int {
            int res = 0;
            if (paired) return sort_run(jobs, 2, m, plan, iota, flags + kSortErr, st, &res);
            TM_TRY(sort_run(jobs, 1, m, plan, iota, flags + kSortErr, st, &res));
            return sort_run(jobs + 1, 1, m, plan, iota, flags + kSortErr, st, &res);
        };
        TM_TRY(sort_count<uint32_t>(reinterpret_cast<uint32_t*>(esrc), reinterpret_cast<uint32_t*>(edst), 2, m, plan,
                                    scratch_of(2, 2).counts, scratch_of(3, 3).counts, st));
        SortJob<L> tsort[2];
        ListFinish<TT> fin[2];
        for (int dir = 0; dir < 2; ++dir) {
            L in, out;
            in.k = reinterpret_cast<uint32_t*>(dir == 0 ? esrc : edst);
            in.v0 = sizeof(TT) == 4 ? reinterpret_cast<V*>(t32e) : reinterpret_cast<V*>(et);
            in.v2 = reinterpret_cast<uint32_t*>(dir == 0 ? edst : esrc);
            out.k = own[dir];
            out.v0 = reinterpret_cast<V*>(lt[dir]);
            out.v1 = reinterpret_cast<uint32_t*>(leid[dir]);
            out.v2 = reinterpret_cast<uint32_t*>(lnbr[dir]);
            tsort[dir] = sort_job(in, out, buf[dir].tmp, plan.npass, scratch_of(2 + dir, 2 + dir));
            fin[dir] = ListFinish<TT>{leid[dir], reinterpret_cast<uint32_t*>(lnbr[dir]), lt[dir], tpos[dir], nt[dir]};
            D.off[dir] = off[dir];
            D.tpos[dir] = tpos[dir];
            D.tguide[dir] = tguide[dir];
            if constexpr (sizeof(TT) == 4) {
                D.lt32[dir] = reinterpret_cast<const uint32_t*>(lt[dir]);
                D.lt[dir] = nullptr;
                D.lnt[dir] = nt[dir];
                D.lnbr[dir] = nullptr;
            } else {
                D.lt[dir] = reinterpret_cast<const int64_t*>(lt[dir]);
                D.lt32[dir] = nullptr;
                D.lnt[dir] = nullptr;
                D.lnbr[dir] = lnbr[dir];
            }
            D.leid[dir] = leid[dir];
            D.lown[dir] = lown[dir];
        }
        TM_TRY(sort_lists(tsort, 2 /* eids: 0, 1, ... */));
        hipLaunchKernelGGL(offsets_kernel, dim3(grid_for(m), 2), dim3(kBlock), 0, st, (const uint32_t*)own[0],
                           (const uint32_t*)own[1], m, n, off[0], off[1]);
        auto finish = [&](const ListFinish<TT>& f0, const ListFinish<TT>& f1, unsigned dirs) {
            hipLaunchKernelGGL((list_finish_kernel<TT>), dim3(grid_for(m), dirs), dim3(kBlock), 0, st, f0, f1, m);
        };
        if (m <= kFinishTogether) {
            finish(fin[0], fin[1], 2);
        } else {
            for (const ListFinish<TT>& f : fin) {
                ListFinish<TT> pos = f, records = f;
                pos.nt = nullptr;
                records.pos = nullptr;
                finish(pos, pos, 1);
                if (records.nt) finish(records, records, 1);
            }
        }
        if (hipGetLastError() != hipSuccess) return tm_fail(TM_EDEVICE, "graph: list launch");
        // N order of dir d: the T order of the other direction (sorted by this
        // direction's neighbour, then time) stably re-sorted by this
        // direction's owner, carrying time, eid and neighbour.
        SortJob<L> nsort[2];
        NOrderFix<V> fix[2];
        for (int dir = 0; dir < 2; ++dir) {
            const int other = 1 - dir;
            L in, out;
            in.k = reinterpret_cast<uint32_t*>(lnbr[other]);
            in.v0 = reinterpret_cast<V*>(lt[other]);
            in.v1 = reinterpret_cast<uint32_t*>(leid[other]);
            in.v2 = own[other];
            out.k = buf[dir].nkeys;
            out.v0 = sizeof(TT) == 4 ? reinterpret_cast<V*>(buf[dir].ntime) : reinterpret_cast<V*>(nkey[dir]);
            out.v1 = reinterpret_cast<uint32_t*>(neid[dir]);
            out.v2 = buf[dir].nbr;
            nsort[dir] = sort_job(in, out, buf[dir].tmp, plan.npass, scratch_of(4 + dir, 2 + dir));
            fix[dir] = NOrderFix<V>{buf[dir].nbr, out.v0, neid[dir], tpos[dir], own[dir], off[dir],
                                    reinterpret_cast<const V*>(lt[dir]), nkey[dir], nxref[dir], nguide[dir],
                                    tguide[dir]};
            D.nkey[dir] = nkey[dir];
            D.nxref[dir] = nxref[dir];
            D.neid[dir] = neid[dir];
            D.nguide[dir] = nguide[dir];
        }
        auto fix_lists = [&](int first, int count) -> int {
            hipLaunchKernelGGL((n_order_fix_kernel<V>), dim3(grid_for(m), (unsigned)count), dim3(kBlock), 0, st,
                               fix[first], fix[1], m, n, D.bt, bn, D.tmul, D.nmul);
            return hipGetLastError() == hipSuccess ? TM_OK : tm_fail(TM_EDEVICE, "graph: list launch");
        };
        int res = 0;
        if (paired) {
            TM_TRY(sort_run(nsort, 2, m, plan, 0, flags + kSortErr, st, &res));
            return fix_lists(0, 2);
        }
        for (int dir = 0; dir < 2; ++dir) {
            TM_TRY(sort_run(nsort + dir, 1, m, plan, 0, flags + kSortErr, st, &res));
            TM_TRY(fix_lists(dir, 1));
        }
        return TM_OK;
    };
    rc = narrow ? build_lists(uint32_t{}) : build_lists(int64_t{});
    release();
    if (rc != TM_OK) return bail(rc);
    timer.stop();
    TM_HIP(read_back({{hflags, flags, sizeof hflags}}, st));
    TM_HIP(dev_free(flags, st));
    TM_HIP(dev_free(tbounds, st));
    timer.finish();
    return flags_error();
}
