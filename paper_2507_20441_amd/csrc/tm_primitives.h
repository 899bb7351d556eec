// Device-wide primitives of the TIMEST GPU library: exclusive prefix sums and
// a stable LSD radix sort of (key, value) pairs.  Templates, instantiated by
// the translation units that use them.
#pragma once

#include <algorithm>
#include <type_traits>

#include "tm_internal.h"

constexpr int kScanItems = 8;                      // values per lane in a scan tile
constexpr int kScanTile = kBlock * kScanItems;     // 2048
constexpr int kSortBits = 8;                       // sort digits: up to 8 bits, one per lane
constexpr int kSortDigits = 1 << kSortBits;        // 256
// Keys per lane in a sort tile.  A pass over many tiles wants large ones (each
// digit's run of a tile goes out to consecutive addresses; 4096 keys); a pass
// over few tiles is one tile's serial work -- ranking key by key, one array
// after another through LDS -- and is left after a quarter of the keys (1024,
// whose values also fit in registers from the start).  A graph build of 2^14
// edges takes 158 us with the small tiles and 222 with the large, 2^18 edges
// 238 and 275, 2^19 324 and 309, 2^20 509 and 394; sampling 2^16 roots 80 and
// 93 us, 2^18 104 and 111, 2^20 200 and 179.
constexpr int kSortItems = 16;
constexpr int kSortItemsSmall = 4;
constexpr int64_t kSortSmall = (int64_t)1 << 18;
constexpr int sort_items(int64_t n) { return n <= kSortSmall ? kSortItemsSmall : kSortItems; }
constexpr int64_t sort_tiles(int64_t n) { return (n + kBlock * sort_items(n) - 1) / (kBlock * sort_items(n)); }
constexpr int kSortMaxPasses = 8;
static_assert(kSortDigits == kBlock, "one digit per lane of a block");

// Radix passes over nb key bits (digits of at most kSortBits, split as
// evenly as possible).
inline int radix_passes(int nb) { return nb <= 0 ? 0 : (nb + kSortBits - 1) / kSortBits; }

// Clearing device words with a kernel rather than a memset node, so that the
// same code can be captured into a HIP graph.
__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v);
// p[i] = i for i < n.
int fill_iota_u32(uint32_t* p, int64_t n, hipStream_t st);

// Of two kernel arguments, as a select between the two loaded values: an index
// into the kernel's arguments has the compiler copy them to scratch, and so
// does a plain select, which the optimiser may turn back into a select of the
// two addresses.  The empty asm statement pins both in scalar registers first
// (arguments are uniform across the wave).
template <typename P>
__device__ __forceinline__ P pick_arg(P x0, P x1, int i) {
    asm("" : "+s"(x0), "+s"(x1));
    return i ? x1 : x0;
}

// The staged copies (StageList), by the lanes of one block.
__device__ __forceinline__ void stage_copy(const StageList& L) {
#pragma unroll
    for (int i = 0; i < kStageReads; ++i)
        for (uint32_t w = threadIdx.x; w < L.words[i]; w += blockDim.x) L.dst[i][w] = L.src[i][w];
}

// ---------------------------------------------------------------------------
// Wave and block scans of 128-bit values (two 64-bit shuffles per step).
// ---------------------------------------------------------------------------
__device__ __forceinline__ u128 shfl_up_u128(u128 v, int d) {
    u64 lo = __shfl_up((u64)v, d, 64);
    u64 hi = __shfl_up((u64)(v >> 64), d, 64);
    return ((u128)hi << 64) | lo;
}

// Inclusive scan across the 64 lanes of a wave; sets *carry on wrap-around.
__device__ __forceinline__ u128 wave_inclusive(u128 v, int lane, bool* carry) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        u128 o = shfl_up_u128(v, d);
        if (lane >= d) {
            u128 s = v + o;
            if (s < v) *carry = true;
            v = s;
        }
    }
    return v;
}

// Exclusive scan over the block's 256 lanes; returns the lane's exclusive
// prefix and writes the block total.  Uses a small LDS array.
__device__ __forceinline__ u128 block_exclusive(u128 v, u128* total, bool* carry) {
    __shared__ u128 wsum[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u128 inc = wave_inclusive(v, lane, carry);
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    u128 before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        u128 x = wsum[w];
        if (w < wave) before += x;
        u128 s = all + x;
        if (s < all) *carry = true;
        all = s;
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

// ---------------------------------------------------------------------------
// Exclusive scan: out[i] = sum of f(0..i-1) for i = 0..n (out[n] = total).
// Accumulation is exact in 128 bits; out is written in T.  Every output is
// exact when the total fits T; otherwise bit 1 of *ovf is set.  A 128-bit
// wrap sets bit 0.
// Reduce-then-scan: tile sums, a scan of the tile sums, then each tile.
// ---------------------------------------------------------------------------
template <typename F>
__global__ void __launch_bounds__(kBlock) scan_tiles_kernel(F f, int64_t n, u128* part, int* ovf) {
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    u128 s = 0;
    bool carry = false;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + (int64_t)k * kBlock + threadIdx.x;
        if (i < n) {
            u128 x = to_u128(f(i));
            u128 y = s + x;
            if (y < s) carry = true;
            s = y;
        }
    }
    u128 tot;
    block_exclusive(s, &tot, &carry);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
    if (carry) atomicOr(ovf, 1);
}

template <typename T, typename F>
__global__ void __launch_bounds__(kBlock)
scan_apply_kernel(F f, int64_t n, const u128* part_scan, T* out, int* ovf) {
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    // each lane owns kScanItems consecutive values of the tile
    const int64_t first = base + (int64_t)threadIdx.x * kScanItems;
    u128 v[kScanItems];
    u128 s = 0;
    bool carry = false;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = first + k;
        v[k] = i < n ? to_u128(f(i)) : (u128)0;
        u128 y = s + v[k];
        if (y < s) carry = true;
        s = y;
    }
    u128 tot;
    u128 run = part_scan[blockIdx.x] + block_exclusive(s, &tot, &carry);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = first + k;
        if (i < n) out[i] = (T)run;
        u128 y = run + v[k];
        if (y < run) carry = true;
        run = y;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const u128 total = part_scan[gridDim.x];
        out[n] = (T)total;
        if ((u128)(T)total != total) atomicOr(ovf, 2);  // total does not fit T
    }
    if (carry) atomicOr(ovf, 1);
}

struct ArrayReader128 {
    const u128* a;
    __device__ u128 operator()(int64_t i) const { return a[i]; }
};

// Exclusive scan of the tile sums in place: part[0..nb] (part[nb] = total).
int scan_parts(u128* part, int64_t nb, int* ovf, hipStream_t st);

template <typename T, typename F>
int device_exclusive_scan(F f, int64_t n, T* out, int* ovf, hipStream_t st) {
    if (n == 0) {
        static_assert(sizeof(T) % 4 == 0, "scan outputs are whole words");
        return fill_u32(out, sizeof(T) / 4, 0u, st);
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    u128* part = nullptr;
    TM_HIP(dev_alloc((void**)&part, (nb + 1) * sizeof(u128), st));
    hipLaunchKernelGGL((scan_tiles_kernel<F>), dim3((unsigned)nb), dim3(kBlock), 0, st, f, n, part,
                       ovf);
    TM_HIP(hipGetLastError());
    int rc = scan_parts(part, nb, ovf, st);
    if (rc == TM_OK) {
        hipLaunchKernelGGL((scan_apply_kernel<T, F>), dim3((unsigned)nb), dim3(kBlock), 0, st, f,
                           n, (const u128*)part, out, ovf);
        TM_HIP(hipGetLastError());
    }
    TM_HIP(dev_free(part, st));
    return rc;
}

// ---------------------------------------------------------------------------
// Pairs of exclusive scans: a job scans two sequences at once, f(i) giving the
// i-th value of both (a Pair2), so a record holding both is read once; the
// jobs of a call (same length) share their launches.  Sums run in T, whose
// wrapping leaves the low bits of the exact sums; a sum that does not fit T
// sets bit 2 (64-bit) or bit 1 (128-bit) of *ovf.
//
// Two launches up to kScanSelfTiles tiles: the tile sums, then the tiles, each
// block adding up the sums before its own.  (Four launches, with a launch of
// one block per sequence between them, spent more on the gaps than on the
// values: a slot's two scans and its coarse entries at 1e6 edges, 60 us busy in
// ten launches, take 25 us in two.)  Above that, one more launch scans the
// tile sums in groups and a block adds up the groups before its own.
// ---------------------------------------------------------------------------
template <typename V>
struct Pair2 {
    V a, b;
};

constexpr int kScanJobs = 2;
constexpr int64_t kScanSelfTiles = 2048;

template <typename T, typename F>
struct Scan2Job {
    F f;
    T* out0;  // [n + 1] each
    T* out1;
    T* c0;    // every 2^kCoarseBits-th entry of out0 and out1, or null
    T* c1;
};

template <typename T, typename F>
struct Scan2Args {
    Scan2Job<T, F> job[kScanJobs];
    T* part;  // per job and sequence, len entries: the tile sums; unless self,
              // scanned in groups, and after them the groups' sums
    int64_t n, nb, len;
    int self;
    int* ovf;
};

// The block's job (blockIdx.y); F::pick selects between two functors.
template <typename T, typename F>
__device__ __forceinline__ Scan2Job<T, F> scan2_job(const Scan2Args<T, F>& a) {
    static_assert(kScanJobs == 2, "one select");
    const int y = blockIdx.y;
    return {F::pick(a.job[0].f, a.job[1].f, y), pick_arg(a.job[0].out0, a.job[1].out0, y),
            pick_arg(a.job[0].out1, a.job[1].out1, y), pick_arg(a.job[0].c0, a.job[1].c0, y),
            pick_arg(a.job[0].c1, a.job[1].c1, y)};
}

template <typename T>
__device__ __forceinline__ T add_carry(T x, T y, bool& carry) {
    const T s = x + y;
    carry = carry || s < x;
    return s;
}

template <typename T>
__device__ __forceinline__ T shfl_up_word(T v, int d) {
    if constexpr (sizeof(T) == 16) return shfl_up_u128(v, d);
    else return __shfl_up(v, d, 64);
}

// Exclusive scan of v over the lanes of a block of kW waves; *total the sum.
template <typename T, int kW = kWaves>
__device__ __forceinline__ T block_exclusive_t(T v, T* total, bool& carry) {
    __shared__ T wsum[kW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T o = shfl_up_word<T>(inc, d);
        if (lane >= d) inc = add_carry(inc, o, carry);
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
        const T x = wsum[w];
        if (w < wave) before += x;
        all = add_carry(all, x, carry);
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

template <typename T, typename F>
__global__ void __launch_bounds__(kBlock) scan2_tiles_kernel(Scan2Args<T, F> args) {
    const Scan2Job<T, F> job = scan2_job(args);
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    T s0 = 0, s1 = 0;
    bool carry = false;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + (int64_t)k * kBlock + threadIdx.x;
        if (i < args.n) {
            const auto x = job.f(i);
            s0 = add_carry<T>(s0, x.a, carry);
            s1 = add_carry<T>(s1, x.b, carry);
        }
    }
    T tot0, tot1;
    block_exclusive_t<T>(s0, &tot0, carry);
    block_exclusive_t<T>(s1, &tot1, carry);
    if (threadIdx.x == 0) {
        T* part = args.part + 2 * (int64_t)blockIdx.y * args.len;
        part[blockIdx.x] = tot0;
        part[args.len + blockIdx.x] = tot1;
    }
    if (carry) atomicOr(args.ovf, sizeof(T) == 8 ? 2 : 1);
}

// Tile sums in groups of kBlock: each group into exclusive prefixes, in place,
// and its sum after the sequence's tile sums.
template <typename T>
__global__ void __launch_bounds__(kBlock) scan2_parts_kernel(T* parts, int64_t nb, int64_t len, int* ovf) {
    T* part = parts + (int64_t)blockIdx.y * len;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    bool carry = false;
    T total;
    const T at = block_exclusive_t<T>(i < nb ? part[i] : (T)0, &total, carry);
    if (i < nb) part[i] = at;
    if (threadIdx.x == 0) part[nb + blockIdx.x] = total;
    if (carry) atomicOr(ovf, sizeof(T) == 8 ? 2 : 1);
}

template <typename T, typename F>
__global__ void __launch_bounds__(kBlock) scan2_apply_kernel(Scan2Args<T, F> args) {
    const Scan2Job<T, F> job = scan2_job(args);
    // Values come in and results go out in rounds of kBlock consecutive
    // entries (coalesced), through LDS; in between each lane scans a run of
    // kScanItems consecutive entries.  Entry j of the tile sits at LDS
    // position j + j / kScanItems, so that the lanes reading their runs do
    // not all fall on the same banks.
    constexpr int kPad = kScanTile + kScanTile / kScanItems;
    __shared__ __align__(16) unsigned char sbuf[2 * kPad * sizeof(T)];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    const int64_t n = args.n;
    T* l0 = reinterpret_cast<T*>(sbuf);
    T* l1 = l0 + kPad;
    const T* part0 = args.part + 2 * (int64_t)blockIdx.y * args.len;
    const T* part1 = part0 + args.len;
    bool carry = false;
    T before0 = 0, before1 = 0;
    // the sums of the tiles before this one, or of the groups before its own
    const int64_t pfirst = args.self ? 0 : args.nb;
    const int64_t pcount = args.self ? (int64_t)blockIdx.x : (int64_t)blockIdx.x / kBlock;
    for (int64_t i = threadIdx.x; i < pcount; i += kBlock) {
        before0 = add_carry<T>(before0, part0[pfirst + i], carry);
        before1 = add_carry<T>(before1, part1[pfirst + i], carry);
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int j = k * kBlock + (int)threadIdx.x;
        const int64_t i = base + j;
        T a = 0, b = 0;
        if (i < n) {
            const auto x = job.f(i);
            a = x.a;
            b = x.b;
        }
        l0[j + j / kScanItems] = a;
        l1[j + j / kScanItems] = b;
    }
    {
        T t0, t1;
        block_exclusive_t<T>(before0, &t0, carry);
        block_exclusive_t<T>(before1, &t1, carry);
        before0 = t0;
        before1 = t1;
    }
    if (!args.self) {
        before0 = add_carry<T>(before0, part0[blockIdx.x], carry);
        before1 = add_carry<T>(before1, part1[blockIdx.x], carry);
    }
    __syncthreads();
    // (a lane's run stays its own until the last round: the values are read
    // again rather than held, for registers)
    const int lane0 = (int)threadIdx.x * (kScanItems + 1);
    T s0 = 0, s1 = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        s0 += l0[lane0 + k];
        s1 += l1[lane0 + k];
    }
    T tot0, tot1;
    T run0 = before0 + block_exclusive_t<T>(s0, &tot0, carry);
    T run1 = before1 + block_exclusive_t<T>(s1, &tot1, carry);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const T x = l0[lane0 + k], y = l1[lane0 + k];
        l0[lane0 + k] = run0;
        l1[lane0 + k] = run1;
        run0 += x;
        run1 += y;
    }
    __syncthreads();
    constexpr int64_t kCoarse = (int64_t)1 << kCoarseBits;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int j = k * kBlock + (int)threadIdx.x;
        const int64_t i = base + j;
        if (i < n) {
            const T x = l0[j + j / kScanItems], y = l1[j + j / kScanItems];
            job.out0[i] = x;
            job.out1[i] = y;
            if (job.c0 && (i & (kCoarse - 1)) == 0) {
                job.c0[i >> kCoarseBits] = x;
                job.c1[i >> kCoarseBits] = y;
            }
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        // (the tile sums' wraps are flagged where they are added up)
        const T t0 = add_carry<T>(before0, tot0, carry), t1 = add_carry<T>(before1, tot1, carry);
        job.out0[n] = t0;
        job.out1[n] = t1;
        if (job.c0 && (n & (kCoarse - 1)) == 0) {
            job.c0[n >> kCoarseBits] = t0;
            job.c1[n >> kCoarseBits] = t1;
        }
    }
    if (carry) atomicOr(args.ovf, sizeof(T) == 8 ? 2 : 1);
}

template <typename T, typename F>
int device_exclusive_scan2(const Scan2Job<T, F>* jobs, int njobs, int64_t n, int* ovf, hipStream_t st) {
    if (njobs <= 0 || njobs > kScanJobs || n <= 0) return tm_fail(TM_EDEVICE, "scan: %d jobs", njobs);
    Scan2Args<T, F> a;
    for (int j = 0; j < kScanJobs; ++j) a.job[j] = jobs[j < njobs ? j : 0];
    a.n = n;
    a.nb = (n + kScanTile - 1) / kScanTile;
    a.self = a.nb <= kScanSelfTiles ? 1 : 0;
    a.ovf = ovf;
    const int64_t groups = (a.nb + kBlock - 1) / kBlock;
    a.len = a.nb + groups;
    TM_HIP(dev_alloc((void**)&a.part, (size_t)(2 * njobs) * a.len * sizeof(T), st));
    const dim3 grid((unsigned)a.nb, (unsigned)njobs);
    hipLaunchKernelGGL((scan2_tiles_kernel<T, F>), grid, dim3(kBlock), 0, st, a);
    if (!a.self)
        hipLaunchKernelGGL((scan2_parts_kernel<T>), dim3((unsigned)groups, 2 * (unsigned)njobs), dim3(kBlock), 0, st,
                           a.part, a.nb, a.len, ovf);
    hipLaunchKernelGGL((scan2_apply_kernel<T, F>), grid, dim3(kBlock), 0, st, a);
    const hipError_t e = hipGetLastError();
    TM_HIP(dev_free(a.part, st));
    TM_HIP(e);
    return TM_OK;
}

// Exclusive scan of v over the block's 256 threads (thread t holds entry t):
// shuffles inside each wave, then the wave totals through LDS.
__device__ __forceinline__ uint32_t block_excl_scan_256(uint32_t v, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) before += w < wave ? wsum[w] : 0u;
    __syncthreads();
    return before + inc - v;
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort of keys that carry up to three value arrays
// (structure of arrays), one kernel per digit of up to 8 bits:
//  * sort_hist_kernel counts the digits of every pass in one read of the
//    keys (each pass turns its counts into the digits' first positions);
//  * sort_pass_kernel, once per pass: a block takes the next tile by ticket
//    (so a tile only ever waits on tiles that are already running), ranks
//    its keys by digit with wave ballots, publishes its digit counts, and
//    finds where its run of each digit starts by adding up the counts that
//    the tiles before it published, back to a tile that has published its
//    inclusive total (decoupled look-back).  Keys and values then go out
//    through LDS, each digit's run of the tile to consecutive addresses.
// A status word holds a value (bits 0-31), a flag (bits 32-33: 1 the tile's
// own count, 2 the total through the tile) and the pass's tag (bits 40-47).
// The words are cleared once, and sorts that share them use tags of their own,
// so a word left by an earlier pass reads as not yet published.  Waits are bounded: a lane that has polled
// kSortMaxSpins times sets kSortStall in the caller's error word and goes on
// (the order is then wrong, and the caller reports the error).
// ---------------------------------------------------------------------------
struct SortNone {};  // an absent value array
constexpr int kSortStall = 4;
constexpr uint32_t kSortMaxSpins = 1u << 20;
constexpr int kSortLook = 8;  // status words a look-back step reads
constexpr size_t kSortHeadBytes =
    ((size_t)kSortMaxPasses * kSortDigits * sizeof(uint32_t) + kSortMaxPasses * sizeof(uint32_t) + 255) &
    ~(size_t)255;

// Scratch of a sort of up to n keys: per-pass digit counts and tickets, then
// one status word per tile and digit.  (2^18 keys take more tiles than 2^18 + 1,
// whose tiles are larger: the size is that of the count with the most.)
constexpr size_t sort_status_bytes(int64_t n) {
    const int64_t small = n > kSortSmall ? sort_tiles(kSortSmall) : 0;
    const int64_t tiles = n > 0 ? sort_tiles(n) : 0;
    return (size_t)(tiles > small ? tiles : small) * kSortDigits * sizeof(u64);
}
constexpr size_t sort_scratch_bytes(int64_t n) { return kSortHeadBytes + sort_status_bytes(n); }

// Where a sort finds its scratch when the caller cleared it: digit counts
// (made by the sort unless counted) and tickets of its own, and the status
// words, which sorts of one stream may share, each with tags above the others'.
struct SortScratch {
    uint32_t* counts = nullptr;   // [kSortMaxPasses][kSortDigits]
    uint32_t* tickets = nullptr;  // [kSortMaxPasses]
    u64* status = nullptr;
    uint32_t tag0 = 0;
    bool counted = false;
};

// The layout of sort_scratch_bytes.
inline SortScratch sort_scratch_at(void* base) {
    SortScratch s;
    s.counts = static_cast<uint32_t*>(base);
    s.tickets = s.counts + kSortMaxPasses * kSortDigits;
    s.status = reinterpret_cast<u64*>(static_cast<unsigned char*>(base) + kSortHeadBytes);
    return s;
}

struct SortPlan {
    int npass;
    int shift[kSortMaxPasses];
    int bits[kSortMaxPasses];
};

// Digits over bits [lo_bit, nbits), as even as possible; no pass when the
// range is empty.
inline SortPlan sort_plan(int lo_bit, int nbits) {
    SortPlan P{};
    P.npass = radix_passes(nbits - lo_bit);
    int shift = lo_bit;
    for (int p = 0; p < P.npass; ++p) {
        const int b = (nbits - shift + (P.npass - p) - 1) / (P.npass - p);
        P.shift[p] = shift;
        P.bits[p] = b;
        shift += b;
    }
    return P;
}

// The plan with at least one pass: a stable copy when no bit is sorted.
inline SortPlan sort_plan_copy(int lo_bit, int nbits) {
    SortPlan P = sort_plan(lo_bit, nbits);
    if (P.npass == 0) {
        P.npass = 1;
        P.shift[0] = 0;
        P.bits[0] = 0;
    }
    return P;
}

template <typename V>
struct SortSize {
    static constexpr size_t value = sizeof(V);
};
template <>
struct SortSize<SortNone> {
    static constexpr size_t value = 0;
};

struct SortIO {
    const void* in[4];  // keys, then the value arrays
    void* out[4];
    const uint32_t* counts;
    uint32_t* ticket;
    u64* status;
};

// One pass of one sort or of two of the same kind (blockIdx.y).
struct SortPass {
    SortIO io[2];
};

// (two key arrays of one length: blockIdx.y picks)
template <typename K>
__global__ void __launch_bounds__(kBlock)
sort_hist_kernel(const K* keys0, const K* keys1, int64_t n, SortPlan P, uint32_t* ghist0, uint32_t* ghist1) {
    __shared__ uint32_t h[kSortMaxPasses][kSortDigits];
    const K* keys = pick_arg(keys0, keys1, blockIdx.y);
    uint32_t* ghist = pick_arg(ghist0, ghist1, blockIdx.y);
#pragma unroll
    for (int p = 0; p < kSortMaxPasses; ++p) h[p][threadIdx.x] = 0;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        const K k = keys[i];
        for (int p = 0; p < P.npass; ++p)
            atomicAdd(&h[p][(uint32_t)(k >> P.shift[p]) & ((1u << P.bits[p]) - 1u)], 1u);
    }
    __syncthreads();
    for (int p = 0; p < P.npass; ++p) {
        const uint32_t c = h[p][threadIdx.x];
        if (c) atomicAdd(&ghist[p * kSortDigits + threadIdx.x], c);
    }
}

template <typename K>
int sort_count(const K* keys0, const K* keys1, int narrays, int64_t n, const SortPlan& P, uint32_t* counts0,
               uint32_t* counts1, hipStream_t st) {
    if (n <= 0 || P.npass <= 0) return TM_OK;
    const unsigned hb = (unsigned)std::min<int64_t>((n + kBlock * kSortItems - 1) / (kBlock * kSortItems), 1024);
    hipLaunchKernelGGL((sort_hist_kernel<K>), dim3(hb, (unsigned)narrays), dim3(kBlock), 0, st, keys0, keys1, n, P,
                       counts0, counts1);
    TM_HIP(hipGetLastError());
    return TM_OK;
}

// One value array of a tile: its loads (before the ranking where registers
// allow, small tiles: kPre), and its way through LDS to the positions of its
// keys.
template <typename V, int kItems>
__device__ __forceinline__ void sort_load_values(const void* vin, bool iota, int64_t wbase, int lane, int64_t n,
                                                 V (&x)[kItems]) {
    if constexpr (!std::is_same<V, SortNone>::value) {
        const V* in = static_cast<const V*>(vin);
        const int64_t tbase = wbase - (int64_t)(threadIdx.x >> 6) * 64 * kItems;
        if (!iota && tbase + kBlock * kItems <= n) {
            // a whole tile: one base address, the items at fixed offsets
            const V* vp = in + wbase + lane;
#pragma unroll
            for (int k = 0; k < kItems; ++k) x[k] = vp[k * 64];
        } else {
#pragma unroll
            for (int k = 0; k < kItems; ++k) {
                const int64_t i = wbase + (int64_t)k * 64 + lane;
                x[k] = i < n ? (iota ? (V)i : in[i]) : (V)0;
            }
        }
    }
}

template <typename V, int kItems, bool kPre>
__device__ __forceinline__ void sort_move_values(const void* vin, void* vout, bool iota, int64_t wbase, int lane,
                                                 int64_t n, const uint32_t (&lp)[kItems],
                                                 const V (&pre)[kPre ? kItems : 1],
                                                 unsigned char* sbuf, const uint8_t* sdig, const uint32_t* gofs, int tn) {
    if constexpr (!std::is_same<V, SortNone>::value) {
        V* sv = reinterpret_cast<V*>(sbuf);
        V* out = static_cast<V*>(vout);
        V x[kItems];
        if constexpr (kPre) {
#pragma unroll
            for (int k = 0; k < kItems; ++k) x[k] = pre[k];
        } else {
            sort_load_values(vin, iota, wbase, lane, n, x);
        }
        __syncthreads();  // the buffer's previous contents have gone out
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = wbase + (int64_t)k * 64 + lane;
            if (i < n) sv[lp[k]] = x[k];
        }
        __syncthreads();
        for (int p = threadIdx.x; p < tn; p += kBlock) {
            const uint32_t g = gofs[sdig[p]] + (uint32_t)p;
            if ((int64_t)g < n) out[g] = sv[p];
        }
    }
}

template <typename K, typename V0, typename V1, typename V2, int kItems>
__global__ void __launch_bounds__(kBlock)
sort_pass_kernel(SortPass pass, int64_t n, int shift, int bits, uint32_t tag, int iota, int* __restrict__ err) {
    constexpr size_t kElt = std::max(std::max(sizeof(K), SortSize<V0>::value),
                                     std::max(SortSize<V1>::value, SortSize<V2>::value));
    constexpr int kTile = kBlock * kItems;
    constexpr bool kPre = kItems <= kSortItemsSmall;
    __shared__ __align__(16) unsigned char sbuf[kElt * kTile];
    __shared__ uint8_t sdig[kTile];
    // per wave and digit: counts, then tile-local starts, at most kTile
    // (16 bits keep a 64-bit-key pass within four workgroups' LDS per CU)
    __shared__ uint16_t cnt[kWaves][kSortDigits];
    __shared__ uint32_t gofs[kSortDigits];  // per digit: its global position minus its tile-local one
    __shared__ uint32_t wsum[kWaves];
    __shared__ uint32_t s_tile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int which = blockIdx.y;
    SortIO io;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        io.in[x] = pick_arg(pass.io[0].in[x], pass.io[1].in[x], which);
        io.out[x] = pick_arg(pass.io[0].out[x], pass.io[1].out[x], which);
    }
    const uint32_t* __restrict__ counts = pick_arg(pass.io[0].counts, pass.io[1].counts, which);
    uint32_t* __restrict__ ticket = pick_arg(pass.io[0].ticket, pass.io[1].ticket, which);
    u64* __restrict__ status = pick_arg(pass.io[0].status, pass.io[1].status, which);
    if (threadIdx.x == 0) s_tile = atomicAdd(ticket, 1u);
    const uint32_t mask = (1u << bits) - 1u;
    const uint32_t d = threadIdx.x;
    const uint32_t gcount = d <= mask ? counts[d] : 0u;  // the digit over all keys
#pragma unroll
    for (int w = 0; w < kWaves; ++w) cnt[w][threadIdx.x] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    const int64_t tbase = (int64_t)tile * kTile;
    // wave w owns tile positions [w 64 kItems, (w + 1) 64 kItems), in
    // rounds of 64 consecutive keys: the wave ranks its keys in input order
    const int64_t wbase = tbase + (int64_t)wave * 64 * kItems;
    const u64 lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const K* keys = static_cast<const K*>(io.in[0]);
    K key[kItems];
    V0 x0[kPre ? kItems : 1];
    V1 x1[kPre ? kItems : 1];
    V2 x2[kPre ? kItems : 1];
    uint32_t lp[kItems];  // (the digits are recomputed from the keys: fewer registers)
    if (tbase + kTile <= n) {
        // a whole tile: one base address, the items at fixed offsets
        const K* kp = keys + wbase + lane;
#pragma unroll
        for (int k = 0; k < kItems; ++k) key[k] = kp[k * 64];
    } else {
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = wbase + (int64_t)k * 64 + lane;
            key[k] = i < n ? keys[i] : (K)0;
        }
    }
    if constexpr (kPre) {
        sort_load_values(io.in[1], iota & 1, wbase, lane, n, x0);
        sort_load_values(io.in[2], iota & 2, wbase, lane, n, x1);
        sort_load_values(io.in[3], iota & 4, wbase, lane, n, x2);
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t i = wbase + (int64_t)k * 64 + lane;
        const bool ok = i < n;
        const uint32_t dk = ok ? ((uint32_t)(key[k] >> shift) & mask) : 0u;
        u64 peers = __ballot(ok);
        for (int b = 0; b < bits; ++b) {
            const u64 bal = __ballot((dk >> b) & 1u);
            peers &= ((dk >> b) & 1u) ? bal : ~bal;
        }
        const uint32_t before = cnt[wave][dk];
        lp[k] = before + (uint32_t)__popcll(peers & lt_mask);
        // the lowest lane of each digit group advances the wave's counter
        if (ok && (peers & lt_mask) == 0) cnt[wave][dk] = (uint16_t)(before + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // lane d: the tile's count of digit d, published at once (the first tile
    // publishes it as its inclusive total)
    uint32_t tcount = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) tcount += cnt[w][d];
    u64* my = status + (size_t)tile * kSortDigits + d;
    const u64 tagw = (u64)tag << 40;
    if (d <= mask)
        __hip_atomic_store(my, tagw | ((u64)(tile == 0 ? 2 : 1) << 32) | tcount, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    // tile-local starts: of each digit, and of each wave's keys inside it
    const uint32_t dstart = block_excl_scan_256(tcount, wsum);
    const uint32_t start = block_excl_scan_256(gcount, wsum);  // the digit's first position
    {
        uint32_t run = dstart;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = cnt[w][d];
            cnt[w][d] = (uint16_t)run;
            run += c;
        }
    }
    __syncthreads();
    K* skey = reinterpret_cast<K*>(sbuf);
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t i = wbase + (int64_t)k * 64 + lane;
        if (i < n) {
            const uint32_t dk = (uint32_t)(key[k] >> shift) & mask;  // the digit again
            const uint32_t p = cnt[wave][dk] + lp[k];
            lp[k] = p;
            skey[p] = key[k];
            sdig[p] = (uint8_t)dk;
        }
    }
    // look-back: the digit's count over all earlier tiles, kSortLook status
    // words per step (their loads in flight together), back to a tile that
    // has published its inclusive total
    if (d <= mask) {
        uint32_t excl = 0;
        if (tile > 0) {
            int64_t j = (int64_t)tile - 1;  // the nearest tile not yet added
            uint32_t spins = 0;
            while (true) {
                u64 sw[kSortLook];
#pragma unroll
                for (int i = 0; i < kSortLook; ++i) {
                    const int64_t x = j - i;
                    // before tile 0: an inclusive total of 0
                    sw[i] = x >= 0 ? __hip_atomic_load(status + (size_t)x * kSortDigits + d, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT)
                                   : tagw | ((u64)2 << 32);
                }
                int used = 0;
                bool done = false;
#pragma unroll
                for (int i = 0; i < kSortLook; ++i) {
                    if (done || used < i) continue;  // stopped before i
                    const uint32_t f = (uint32_t)(sw[i] >> 32) & 3u;
                    if ((uint32_t)(sw[i] >> 40) != tag || f == 0) continue;  // not published yet: poll again
                    excl += (uint32_t)sw[i];
                    used = i + 1;
                    done = f == 2;
                }
                if (done) break;
                j -= used;
                if (used == 0) {
                    if (++spins >= kSortMaxSpins) {
                        atomicOr(err, kSortStall);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __hip_atomic_store(my, tagw | ((u64)2 << 32) | (u64)(excl + tcount), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        gofs[d] = start + excl - dstart;
    }
    __syncthreads();
    const int tn = (int)(n - tbase < kTile ? n - tbase : kTile);
    K* okeys = static_cast<K*>(io.out[0]);
    // (positions are below n whenever the digit counts hold; the test keeps
    // a broken invariant from writing outside the output)
    for (int p = threadIdx.x; p < tn; p += kBlock) {
        const uint32_t g = gofs[sdig[p]] + (uint32_t)p;
        if ((int64_t)g < n) okeys[g] = skey[p];
    }
    sort_move_values<V0, kItems, kPre>(io.in[1], io.out[1], iota & 1, wbase, lane, n, lp, x0, sbuf, sdig, gofs,
                                       tn);
    sort_move_values<V1, kItems, kPre>(io.in[2], io.out[2], iota & 2, wbase, lane, n, lp, x1, sbuf, sdig, gofs,
                                       tn);
    sort_move_values<V2, kItems, kPre>(io.in[3], io.out[3], iota & 4, wbase, lane, n, lp, x2, sbuf, sdig, gofs,
                                       tn);
}

// A key array and up to three value arrays (null where a value is absent).
template <typename K, typename V0 = SortNone, typename V1 = SortNone, typename V2 = SortNone>
struct SortSet {
    K* k = nullptr;
    V0* v0 = nullptr;
    V1* v1 = nullptr;
    V2* v2 = nullptr;
};

// Where a sort's passes read and write: pass p reads `in` (p = 0) or the
// previous pass's output, and writes bufs[p & 1]; bufs[0] must not be `in`
// (bufs[1] may be: the first pass has consumed it before the second writes).
// scratch: cleared by the caller, or with null counts allocated and cleared by
// the sort.
template <typename S>
struct SortJob {
    S in;
    S bufs[2];
    SortScratch scratch;
};

// Runs the plan's passes of one sort, or of two of n keys each with the same
// plan side by side (their scratch must be the caller's): a pass of few tiles
// leaves the chip idle, and two fill it better for the time of one.  Sets
// *result to the index of the buffer that holds the result.  iota: bit j set,
// value array j holds nothing yet and stands for 0, 1, ..., n - 1.
template <typename K, typename V0, typename V1, typename V2>
int sort_run(const SortJob<SortSet<K, V0, V1, V2>>* jobs, int njobs, int64_t n, const SortPlan& P, int iota,
             int* err, hipStream_t st, int* result) {
    using S = SortSet<K, V0, V1, V2>;
    *result = (P.npass - 1) & 1;
    if (n <= 0 || P.npass <= 0) return TM_OK;
    SortScratch scratch[2];
    unsigned char* own = nullptr;
    int rc = TM_OK;
    for (int j = 0; j < njobs; ++j) {
        scratch[j] = jobs[j].scratch;
        if (jobs[j].bufs[0].k == jobs[j].in.k)
            return tm_fail(TM_EDEVICE, "sort: the first pass would overwrite its input");
        if (!scratch[j].counts && (njobs > 1 || j > 0)) return tm_fail(TM_EDEVICE, "sort: no scratch");
    }
    if (!scratch[0].counts) {
        const size_t bytes = sort_scratch_bytes(n);
        TM_HIP(dev_alloc((void**)&own, bytes, st));
        scratch[0] = sort_scratch_at(own);
        rc = fill_u32(own, (int64_t)(bytes / sizeof(uint32_t)), 0u, st);
    }
    for (int j = 0; j < njobs && rc == TM_OK; ++j)
        if (!scratch[j].counted)
            rc = sort_count<K>(jobs[j].in.k, jobs[j].in.k, 1, n, P, scratch[j].counts, scratch[j].counts, st);
    const int items = sort_items(n);
    const dim3 grid((unsigned)sort_tiles(n), (unsigned)njobs);
    for (int p = 0; p < P.npass && rc == TM_OK; ++p) {
        SortPass pass;
        for (int j = 0; j < 2; ++j) {
            const int y = j < njobs ? j : 0;
            const S& src = p == 0 ? jobs[y].in : jobs[y].bufs[(p - 1) & 1];
            const S& dst = jobs[y].bufs[p & 1];
            pass.io[j] = SortIO{{src.k, src.v0, src.v1, src.v2},
                                {dst.k, dst.v0, dst.v1, dst.v2},
                                scratch[y].counts + p * kSortDigits,
                                scratch[y].tickets + p,
                                scratch[y].status};
        }
        const uint32_t tag = scratch[0].tag0 + (uint32_t)p + 1;
        if (items == kSortItems)
            hipLaunchKernelGGL((sort_pass_kernel<K, V0, V1, V2, kSortItems>), grid, dim3(kBlock), 0, st, pass, n,
                               P.shift[p], P.bits[p], tag, p == 0 ? iota : 0, err);
        else
            hipLaunchKernelGGL((sort_pass_kernel<K, V0, V1, V2, kSortItemsSmall>), grid, dim3(kBlock), 0, st, pass, n,
                               P.shift[p], P.bits[p], tag, p == 0 ? iota : 0, err);
        if (hipGetLastError() != hipSuccess) rc = tm_fail(TM_EDEVICE, "sort: pass launch");
    }
    if (own) {
        const hipError_t e = dev_free(own, st);
        if (rc == TM_OK && e != hipSuccess) rc = tm_fail(TM_EDEVICE, "sort: free");
    }
    return rc;
}

// The job that sorts `in` into `out` in npass passes, with `tmp` as the other
// buffer (`in` is left as it was unless tmp is `in`, which is allowed only
// when an odd number of passes runs).
template <typename S>
SortJob<S> sort_job(const S& in, const S& out, const S& tmp, int npass, const SortScratch& scratch) {
    return SortJob<S>{in, {(npass & 1) ? out : tmp, (npass & 1) ? tmp : out}, scratch};
}

// Sorts `in` by bits [lo_bit, nbits) of its keys into `out`, stably (see
// sort_job).  At least one pass runs: a stable copy when no bit is sorted.
template <typename S>
int sort_into(const S& in, const S& out, const S& tmp, int64_t n, int lo_bit, int nbits, int iota, int* err,
              hipStream_t st, const SortScratch& scratch = {}) {
    const SortPlan P = sort_plan_copy(lo_bit, nbits);
    const SortJob<S> job = sort_job(in, out, tmp, P.npass, scratch);
    int res = 0;
    return sort_run(&job, 1, n, P, iota, err, st, &res);
}

// Sorts (keys, vals) by bits [lo_bit, nbits) of the key, stably.  Buffers
// ping-pong between (keys, vals) and (tkeys, tvals); on return *k_out /
// *v_out point to whichever pair holds the result (the tkeys pair after an
// odd number of passes).  iota_vals: vals holds nothing yet and stands for
// 0 .. n-1.  scratch: as for sort_run.  err: bit kSortStall is set if a
// look-back wait ran out.
template <typename K>
int radix_sort_pairs(K* keys, uint32_t* vals, K* tkeys, uint32_t* tvals, int64_t n, int lo_bit, int nbits,
                     K** k_out, uint32_t** v_out, int* err, hipStream_t st, bool iota_vals = false,
                     const SortScratch& scratch = {}) {
    *k_out = keys;
    *v_out = vals;
    if (n > 1 && nbits > lo_bit) {
        using S = SortSet<K, uint32_t>;
        S in, b0, b1;
        in.k = keys;
        in.v0 = vals;
        b0.k = tkeys;
        b0.v0 = tvals;
        b1 = in;
        const SortJob<S> job{in, {b0, b1}, scratch};
        const SortPlan P = sort_plan(lo_bit, nbits);
        int res = 0;
        TM_TRY(sort_run(&job, 1, n, P, iota_vals ? 1 : 0, err, st, &res));
        *k_out = job.bufs[res].k;
        *v_out = job.bufs[res].v0;
    } else if (iota_vals) {
        TM_TRY(fill_iota_u32(vals, n, st));  // no pass ran
    }
    return TM_OK;
}
