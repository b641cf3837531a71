// xred_batched.hpp -- many independent reductions in one launch: kernels and
// launch templates, instantiated per group of element types by
// xred_batched_{float,fp8,int}.hip so the groups compile in parallel.
//
// Small messages are dominated by per-call overhead (the T_c term of the
// LogP model in Section 6.2), so a batch of K reductions is run as one
// kernel.  Work is cut into tiles of 16-byte vectors of one item, in the
// global order item 0's tiles, then item 1's, ...  Five kernels:
//   table        (host descriptors, the usual case): the host stages the
//                item of every tile and one workgroup runs each tile, so the
//                hardware dispatches tiles in order, as for the fused kernel;
//   queue        (device descriptors of more than 64 items, eager): a persistent
//                grid takes tiles in order from a counter in device memory;
//   runs         (other device descriptors: up to 64 items, under graph
//                capture, or past the queue's limits): runs of up to 64
//                consecutive items, each dealt tile by tile to its own set of
//                workgroups, whose waves plan their tiles from the descriptors
//                in registers (metadata by reference, Section 6.1); no state
//                between calls;
//   round-robin  (host batches past the table's size): a persistent grid,
//                tile g on workgroup g mod G, the tile-start prefix staged;
//   range        (host batches past the round-robin plan's items): contiguous
//                tile ranges per workgroup, planned on the host.

#pragma once

#include <type_traits>

#include "xred_dispatch.hpp"
#include "xred_internal.hpp"
#include "xred_kernels.hpp"

namespace xred {
namespace {

constexpr int kU = 1;     // vectors per thread in one pass over a sub-tile
constexpr int kB = 512;
// Sub-tiles of kB*kU vectors per tile: two halve the per-tile descriptor
// work (measured +5-6 % on batches of large or equal items, neutral on the
// log-uniform 4096-item batch); four were no better.
constexpr int kSub = 2;

template <class T>
constexpr uint64_t tile_vecs() { return (uint64_t)kB * kU * kSub; }
template <class T>
constexpr uint64_t tile_elems() { return tile_vecs<T>() * T::kVec; }
constexpr uint32_t kSubBytes = (uint32_t)kB * kU * 16u;

__device__ __forceinline__ bool item_runnable(const xred_item &it)
{
    return it.nsrc >= 1 && it.nsrc <= XRED_MAX_SRC && it.reserved == 0 && it.srcs != nullptr &&
           it.dst != nullptr;
}

// Tiles of an item (0: nothing to run, or a descriptor that cannot be run).
template <class T>
__device__ __forceinline__ uint64_t item_tiles(const xred_item &it)
{
    return item_runnable(it) ? (it.count + tile_elems<T>() - 1) / tile_elems<T>() : 0;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// v plus the value a DPP move brings from a lower lane (0 where none does).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_add(uint64_t v)
{
    const uint32_t lo =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, false);
    return v + (((uint64_t)hi << 32) | lo);
}

// Inclusive prefix sum over the wavefront: within rows of 16 lanes by
// row_shr:1, 2, 4, 8, then row_bcast:15 into rows 1 and 3 and row_bcast:31
// into rows 2 and 3.  All in the vector ALU (64-bit shuffles through LDS
// took 0.4 us a scan, on the critical path of every small batch).
__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t v)
{
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    return dpp_add<0x143, 0xc>(v);
}

// Exclusive prefix sum of v over the workgroup (kB threads); *total gets the
// sum, *wsum the sum of w.  s_wave: 2 * kB / 64 words of LDS.
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t w, uint64_t *s_wave,
                                                         uint64_t *total, uint64_t *wsum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t incl = wave_inclusive_scan(v);
    w = wave_inclusive_scan(w);
    if (lane == 63) {
        s_wave[2 * wave] = incl;
        s_wave[2 * wave + 1] = w;
    }
    __syncthreads();
    uint64_t before = 0, sum = 0, ws = 0;
#pragma unroll
    for (int i = 0; i < kB / 64; ++i) {
        const uint64_t x = s_wave[2 * i];
        before += i < wave ? x : 0;
        sum += x;
        ws += s_wave[2 * i + 1];
    }
    *total = sum;
    *wsum = ws;
    return before + incl - v;
}

// Lane l's value of v (l uniform).
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// One tile of one item, resolved: what its workgroup needs to run it.
// Uniform over the wavefront.
enum TilePath : int {
    kGrid,       // sources at one offset within 16 bytes
    kOffset,     // sources at different offsets
    kElems,      // too short for a vector: element by element
    kNothing,    // a NULL source: the item is skipped
};
struct TileDesc {
    const char *p[8];         // sources 0..7 (valid below nsrc)
    const char *const *srcs;  // the item's source array
    char *dst;
    uint64_t count;
    uint64_t lt;              // tile within the item
    int nsrc;
    uint32_t lead;
    TilePath path;
};

// The rest of a descriptor whose srcs, dst, count, nsrc and lt are set: the
// source pointers, and how the item is cut (vec_plan).
template <class T>
__device__ __forceinline__ void fetch_sources(TileDesc &d)
{
    uintptr_t sdiff = 0;   // bits in which some source's address differs from the first's
    bool null_src = false;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        d.p[q] = q < d.nsrc ? sload(d.srcs + q) : nullptr;
        sdiff |= q < d.nsrc ? (uintptr_t)d.p[q] ^ (uintptr_t)d.p[0] : 0;
        null_src |= q < d.nsrc && d.p[q] == nullptr;
    }
    for (int q = 8; q < d.nsrc; ++q) {
        const uintptr_t x = (uintptr_t)sload(d.srcs + q);
        sdiff |= x ^ (uintptr_t)d.p[0];
        null_src |= x == 0;
    }
    const VecPlan vp = vec_plan<T>((uintptr_t)d.p[0], sdiff, (uintptr_t)d.dst, d.count);
    d.lead = vp.lead;
    d.path = null_src ? kNothing : !vp.any ? kElems : vp.grid ? kGrid : kOffset;
}

// Tile lt of item `it` (a descriptor in device memory).
template <class T>
__device__ __forceinline__ void fetch_desc(TileDesc &d, const xred_item *it, uint64_t lt)
{
    d.lt = lt;
    d.srcs = (const char *const *)sload(&it->srcs);
    d.dst = (char *)sload(&it->dst);
    d.count = sload(&it->count);
    d.nsrc = (int)sload(&it->nsrc);
    fetch_sources<T>(d);
}

// Runs one tile of SUB sub-tiles of kB vectors.  mid() is called once, on the
// grid path while loads are in flight (the next tile is claimed and resolved
// there).  EARLY: the loads of the item's ends join the tile's, on its last
// wavefront, which shortens the chain of a workgroup that runs few tiles
// (captured batches of 4096 log-uniform items 1375 against 1450 us); a
// workgroup that runs many folds them after the tile, on its first (queue
// kernel, 4096 / 619 items: 1250 / 204.4 against 1257 / 206.3 us).
template <class T, class Op, int SUB, bool EARLY, class Mid>
__device__ __forceinline__ void run_tile(const TileDesc &d, Mid &&mid)
{
    constexpr uint32_t kBytes = (uint32_t)kB * SUB * 16u;
    const GlobalSrc src{d.srcs};
    const size_t lb = (size_t)d.lead * T::kSize;   // bytes before the first vector
    const uint64_t nvec = (d.count - d.lead) / T::kVec;
    const size_t vbytes = nvec * 16, toff = d.lt * kBytes;
    // the item's first tile also takes the elements before its first vector,
    // its last tile those after its last full vector
    auto ends = [&] {
        reduce_ends<T, Op>(src, d.nsrc, d.dst, d.lt == 0 ? d.lead : 0u,
                           (d.lt + 1) * kB * SUB * T::kVec >= d.count
                               ? (uint32_t)((d.count - d.lead) % T::kVec)
                               : 0u,
                           d.lead + nvec * T::kVec, EARLY ? threadIdx.x - (kB - 64) : threadIdx.x);
    };
    if (d.path == kGrid) {
        // Groups of 8 sources.  A source the item does not have is not read: a
        // load of an empty range still takes its turn in the address units (P=1:
        // range kernel 2070 us a 10.2 GB batch, 2310 with them; 100 items of 4 MiB
        // captured 201 / 281 us, with P=2 231 / 294; 1000 log-uniform eager 115 /
        // 166; P=9 159 / 170).  A whole first group has no test per source, which
        // gains over one body with them (captured P=8 4096 items 904 / 935 us).
        const uint32_t nrec = toff < vbytes ? tile_nrec(vbytes, toff, kBytes) : 0u;
        u32x4 in[8][SUB];
        typename T::Acc acc[SUB][T::kVec];
        auto load = [&](int q, const char *p) {
            const rsrc_t r = make_rsrc(p + lb + toff, nrec);
#pragma unroll
            for (int h = 0; h < SUB; ++h)
                in[q][h] = bload<kLoadStream>(r, (uint32_t)(h * kB + threadIdx.x) * 16u);
        };
        auto first = [&](auto whole) {
            constexpr bool kWhole = decltype(whole)::value;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (kWhole || q < d.nsrc) load(q, d.p[q]);
            mid();
            if (EARLY) ends();
#pragma unroll
            for (int h = 0; h < SUB; ++h) {
                up_vec<T>(in[0][h], acc[h]);
#pragma unroll
                for (int q = 1; q < 8; ++q)
                    if (kWhole || q < d.nsrc) fold_vec<T, Op>(acc[h], in[q][h]);
            }
        };
        if (d.nsrc >= 8) first(std::true_type{});
        else first(std::false_type{});
        for (int p0 = 8; p0 < d.nsrc; p0 += 8) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (p0 + q < d.nsrc) load(q, sload(d.srcs + p0 + q));
#pragma unroll
            for (int h = 0; h < SUB; ++h)
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (p0 + q < d.nsrc) fold_vec<T, Op>(acc[h], in[q][h]);
        }
#pragma unroll
        for (int h = 0; h < SUB; ++h) {
            if constexpr (__is_same(Op, OpAvg)) {
#pragma unroll
                for (int e = 0; e < T::kVec; ++e)
                    acc[h][e] = avg_scale<T, Op>(acc[h][e], d.nsrc);
            }
            char *base = d.dst + lb + toff;
            const uint32_t o = (uint32_t)(h * kB + threadIdx.x) * 16u;
            const u32x4 v = down_vec<T, Op>(acc[h]);
            if (((uintptr_t)base & 15u) == 0) store_out<false>(v, base, nrec, o);
            else store_out<true>(v, base, nrec, o);
        }
        if (!EARLY) ends();
        return;
    }
    // one sub-tile at a time
    auto sub = [&](int h) {
        const size_t off = toff + (size_t)h * kSubBytes;
        if (d.path == kElems) {
            const uint64_t e0 = off / T::kSize;
            const uint64_t left = d.count > e0 ? d.count - e0 : 0;
            const uint64_t n = left < kSubBytes / T::kSize ? left : kSubBytes / T::kSize;
            for (uint64_t i = threadIdx.x; i < n; i += kB)
                reduce_elem<T, Op>(src, d.nsrc, d.dst, e0 + i);
        } else if (d.path != kNothing && off < vbytes) {
            offset_tile<T, Op>(src, d.nsrc, d.dst, lb, off, tile_nrec(vbytes, off, kSubBytes));
        }
    };
    for (int h = 0; h < SUB; ++h) sub(h);
    if (d.path == kOffset) ends();
    mid();
}

template <class T, class Op>
__global__ __launch_bounds__(kB) void batched_kernel(const xred_item *items, int nitems,
                                                     const WgStart *wg)
{
    const WgStart *w = wg + blockIdx.x;
    uint64_t k = sload(&w->item);
    uint64_t lt = sload(&w->local_tile);
    uint64_t left = sload(&w->ntiles);
    k = uniform64(k);
    lt = uniform64(lt);
    left = uniform64(left);
    while (left > 0 && k < (uint64_t)nitems) {
        k = uniform64(k);
        const uint64_t nt = (sload(&items[k].count) + tile_elems<T>() - 1) / tile_elems<T>();
        if (lt >= nt) {
            ++k;
            lt = 0;
            continue;
        }
        TileDesc d;
        fetch_desc<T>(d, items + k, lt);
        run_tile<T, Op, kSub, false>(d, [] {});
        ++lt;
        --left;
    }
}

// ------------------------------------------------------ round-robin variant --
// Host batches too large for the tile table: global tile g is processed by
// workgroup g mod G (G = the workgroups that fit on the chip at once), so the
// tiles in flight form one moving window over the batch, as in the fused
// kernel, instead of G scattered ranges.  Each workgroup copies the batch's
// tile-start prefix to LDS, finds the (item, tile) of each of its tiles by
// binary search in parallel, and while one tile's loads are in flight fetches
// the next tile's descriptor and source pointers with scalar loads.
constexpr int kListMax = 1024;     // tiles a workgroup plans per pass
constexpr int kRrMaxItems = 8192;  // items whose prefix fits the LDS budget

template <class T, class Op>
__global__ __launch_bounds__(kB) void batched_rr_kernel(const xred_item *items, int nitems,
                                                        const uint32_t *tile_start)
{
    extern __shared__ uint2 s_dyn[];
    uint2 *s_list = s_dyn;                             // kListMax entries
    uint32_t *s_pre = (uint32_t *)(s_dyn + kListMax);  // nitems + 1 entries
    for (int i = threadIdx.x; i <= nitems; i += kB) s_pre[i] = tile_start[i];
    __syncthreads();
    const uint64_t total = s_pre[nitems];
    const uint64_t G = gridDim.x;
    for (uint64_t g0 = blockIdx.x; g0 < total; g0 += (uint64_t)kListMax * G) {
        const uint64_t left = (total - g0 + G - 1) / G;
        const int n = left < (uint64_t)kListMax ? (int)left : kListMax;
        for (int j = threadIdx.x; j < n; j += kB) {
            const uint64_t g = g0 + (uint64_t)j * G;
            int lo = 0, hi = nitems;   // s_pre[lo] <= g < s_pre[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_pre[mid] <= g) lo = mid;
                else hi = mid;
            }
            s_list[j] = uint2{(uint32_t)lo, (uint32_t)(g - s_pre[lo])};
        }
        __syncthreads();
        auto fetch = [&](TileDesc &d, int j) {
            fetch_desc<T>(d, items + __builtin_amdgcn_readfirstlane(s_list[j].x),
                          __builtin_amdgcn_readfirstlane(s_list[j].y));
        };
        TileDesc cur, nxt;
        fetch(cur, 0);
        for (int j = 0; j < n; ++j) {
            run_tile<T, Op, kSub, false>(cur, [&] {
                if (j + 1 < n) fetch(nxt, j + 1);
            });
            cur = nxt;
            // the waves start every tile together (8 items of 32M bf16 per
            // source: 5.18 against 4.99 TB/s; 64 items of 4M: 4.90 against 4.98)
            __syncthreads();
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------ queue variant --
// Device descriptors (the host never sees the sizes): a persistent grid takes
// the batch's tiles in order, so the tiles in flight stay one compact window
// over the batch, as when the hardware dispatches one workgroup per tile of a
// host-built table, and no workgroup keeps a fixed share of the batch.  Each
// workgroup scans the tile counts of all items into an LDS tile-start prefix;
// its first unit of tiles is its own index, later ones come from a counter in
// device memory.  While a tile's loads are in flight, the next unit's claim
// is handed to all waves through LDS and every wave finds the next tile's item
// (a 64-ary search of the prefix) and fetches its descriptor and source
// pointers, so the next tile's loads follow this tile's stores at once.
//
// The counter answers one claim in about 14 ns.  A unit is therefore as many
// tiles as it takes to move kClaimBytes (most tiles of a batch of small items
// are far from full), and a batch of at most one unit per workgroup claims
// nothing.  With one claim per tile, the first included, P=4 bf16 items of
// 8-16 KiB took 17.6 us for 563 (16.8 now), 66 of 8-128 KiB 10.4 us (6.5).
//
// What was measured on the 4096-item log-uniform batch (MI355X, same box):
// one workgroup of 512 threads per CU and tiles of two 512-vector sub-tiles
// (16 KiB per source) 1237-1240 us, against 1267 us with the next tile's
// descriptor fetched after this tile's stores.  With the fetch overlapped:
// 8 KiB tiles 1611 us (one or two workgroups per CU: the one counter then
// answers twice as many claims), 24 KiB 1281 us, 32 KiB 1322 us, two
// workgroups per CU 1393 us; the loads issued sub-tile by sub-tile instead
// of source by source 1248 us; the first sub-tile folded and stored before
// the claim is handed over 1314 us.  Before it: claiming two tiles ahead 1445 us
// and double-buffered loads 1262 us (a tile claimed or loaded ahead widens
// the window of tiles being read, which costs more than the latency it
// hides); eight interleaved counters 1339 us.
//
// The counter: *next is zero when the launch starts.  clear (if set) is
// another counter the launch zeroes for the next launch on the stream;
// finished (if set) counts workgroups out, and the last one returns *next and
// *finished to zero, so the counters are zero again when the launch ends.
struct QueueCtl {
    uint64_t *next;
    uint64_t *clear;
    uint64_t *finished;
};
constexpr int kQMaxItems = 16384;   // items whose 32-bit tile-start prefix fits in LDS
constexpr float kClaimBytes = 96 << 10;   // 14 ns at 6.9 TB/s
constexpr uint32_t kClaimMost = 8;        // tiles per unit

// The item k < n holding tile g: the last k with pre[k] <= g (pre[0] = 0 <= g,
// pre non-decreasing).  Each level reads one prefix entry per lane and keeps
// the run of lanes at or below g: 64^levels entries in `levels` LDS reads.
__device__ __forceinline__ int find_item(const uint32_t *pre, int n, uint32_t g)
{
    const int lane = (int)(threadIdx.x & 63);
    int step = 1;
    while (step * 64 < n) step *= 64;
    int lo = 0;
    for (;;) {
        const int i = lo + lane * step;
        const bool ok = i < n && pre[i] <= g;
        lo += (__popcll(__ballot(ok)) - 1) * step;
        if (step == 1) break;
        step /= 64;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// A workgroup barrier that orders LDS only: __syncthreads() also waits for
// every outstanding global store and atomic of the wave (its release fence
// covers global memory), which would drain each tile's stores before the
// next tile's loads could be issued.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <class T, class Op>
__global__ __launch_bounds__(kB) void batched_queue_kernel(const xred_item *items, int nitems,
                                                           QueueCtl q)
{
    auto claim = [&q]() -> uint64_t {
        return __hip_atomic_fetch_add(q.next, (uint64_t)1, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    };
    extern __shared__ uint32_t s_pre[];   // nitems + 1 tile starts, in the occupancy reservation
    __shared__ uint64_t s_wave[2 * kB / 64];
    // The claim made during a tile is written to s_claim[b % 2], b counting
    // the claims, and read after the tile's barrier; the slot's previous claim
    // was read before the barrier that precedes the write.
    __shared__ uint64_t s_claim[2];
    if (q.clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(q.clear, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // tile counts of this thread's consecutive items (four descriptor loads
    // in flight at a time), kept in the prefix's place; then the
    // workgroup's exclusive scan turns them into tile starts
    const int per = (nitems + kB - 1) / kB;
    const int i0 = min(nitems, (int)threadIdx.x * per), i1 = min(nitems, i0 + per);
    uint64_t mine = 0, bytes = 0;
    for (int j = i0; j < i1; j += 4) {
        xred_item it[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j + u < i1) it[u] = items[j + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (j + u < i1) {
                const uint64_t t = item_tiles<T>(it[u]);
                mine += t;
                if (t != 0) bytes += it[u].count * T::kSize * (it[u].nsrc + 1);
                s_pre[j + u] = t < 0xFFFFFFFFull ? (uint32_t)t : 0xFFFFFFFFu;
            }
        }
    }
    uint64_t total = 0;
    uint64_t run = block_exclusive_scan(mine, bytes, s_wave, &total, &bytes);
    for (int i = i0; i < i1; ++i) {
        const uint32_t t = s_pre[i];
        s_pre[i] = (uint32_t)run;
        run += t;
    }
    total = uniform64(total);
    if (total > 0xFFFFFFFFull) total = 0;   // more tiles than the prefix indexes: run nothing
    if (threadIdx.x == 0) s_pre[nitems] = (uint32_t)total;
    __syncthreads();
    // tiles per unit, the same in every workgroup; one while there are fewer
    // than eight per workgroup (units of two end 563 one-tile items a round later)
    const uint32_t G = gridDim.x;
    const float want = __builtin_ceilf((float)total * kClaimBytes / (float)bytes);
    uint32_t unit = want < (float)kClaimMost ? (uint32_t)want : kClaimMost;
    unit = min(unit, (uint32_t)total / (4 * G));
    unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)max(unit, 1u));
    const bool dynamic = total > (uint64_t)unit * G;
    uint64_t g = (uint64_t)blockIdx.x * unit;   // the tile being run
    uint32_t left = unit;                       // tiles of its unit, itself included
    TileDesc cur{};
    auto fetch = [&](TileDesc &d, uint64_t t) {
        const int k = find_item(s_pre, nitems, (uint32_t)t);
        fetch_desc<T>(d, items + k, uniform64(t - s_pre[k]));
    };
    if (g < total) fetch(cur, g);
    for (uint32_t b = 0; g < total;) {
        const bool refill = dynamic && left == 1;
        uint64_t c = 0;
        if (refill && threadIdx.x == 0) c = claim();   // answered while this tile streams
        uint64_t gn = left == 1 ? total : g + 1;
        TileDesc nxt{};
        run_tile<T, Op, kSub, false>(cur, [&] {
            if (refill && threadIdx.x == 0) s_claim[b & 1] = c;
            lds_barrier();   // also keeps the waves on one tile
            if (refill) gn = (G + uniform64(s_claim[b & 1])) * unit;
            if (gn < total) fetch(nxt, gn);
        });
        b += refill;
        left = left == 1 ? unit : left - 1;
        cur = nxt;
        g = gn;
    }
    // every claim of this workgroup has been answered (each was read back
    // above), so the last workgroup's reset is the counter's last write
    if (q.finished != nullptr && dynamic && threadIdx.x == 0) {
        const uint64_t n = __hip_atomic_fetch_add(q.finished, (uint64_t)1, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        if (n + 1 == gridDim.x) {
            __hip_atomic_store(q.next, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(q.finished, (uint64_t)0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ------------------------------------------------------- tile-table variant --
// Host descriptors: the host lists the item of every tile, and stages each
// item with the index of its first tile in the descriptor's reserved field;
// workgroup w takes tile w.  One workgroup per tile, dispatched in
// order, keeps the tiles in flight one compact window over the batch, as in
// the fused kernel; persistent workgroups each walking their own tiles drift
// apart and spread the loads in flight over the batch (c4: 5.3 against
// 6.9 TB/s for the same data).  Tiles are one 16-byte vector per thread and
// source, two workgroups per CU (16 waves: 6.9 TB/s against 5.9 uncapped).
// Other shapes on the 4096-item log-uniform batch (same box): 512 threads and
// 8 KiB per source, two per CU, 1199 us; one or three per CU 1462 / 1472 us;
// 16 KiB tiles one / two per CU 1321 / 1488 us; 1024 threads one per CU
// 1314 us; 256 threads four per CU, 4 / 8 KiB tiles 1367 / 1489 us.  The
// three dependent scalar loads before a tile's loads (table entry, then the
// descriptor, then the source pointers) also pace the workgroups: staging
// eight pointer slots per item so that the descriptor and the pointers load
// together made c4 slower (1241-1254 against 1204 us), like more resident
// workgroups per CU.
// Under a CU budget the grid is smaller and each workgroup strides over the
// table.
constexpr int kTB = kB;
constexpr int kTableSub = 1;          // 16-byte vectors per thread and source
constexpr int kTableWgsPerCu = 2;

template <class T>
constexpr uint64_t table_tile_elems() { return (uint64_t)kTB * kTableSub * T::kVec; }

// NARROW: the table holds 16-bit item indices (batches of at most 65536
// items), two per 32-bit word, little-endian; the word is loaded whole (the
// table is padded to 8 bytes) so every scalar load stays dword-aligned.
template <class T, class Op, bool NARROW>
__global__ __launch_bounds__(kTB, kTableWgsPerCu * kTB / 256) void batched_table_kernel(const xred_item *items,
                                                            const uint32_t *table,
                                                            uint64_t ntiles)
{
    extern __shared__ char occupancy_reservation[];
    (void)occupancy_reservation;
    for (uint64_t g = blockIdx.x; g < ntiles; g += gridDim.x) {
        uint32_t k;
        if constexpr (NARROW) {
            const uint32_t pair = sload(&table[g >> 1]);
            k = (g & 1) ? pair >> 16 : pair & 0xFFFFu;
        } else {
            k = sload(&table[g]);
        }
        TileDesc d;
        fetch_desc<T>(d, items + k, g - sload(&items[k].reserved));
        run_tile<T, Op, kTableSub, true>(d, [] {});
    }
}

template <class T, class Op>
hipError_t go_table(const xred_item *d_items, const uint32_t *d_table, bool narrow,
                    uint64_t ntiles, hipStream_t s)
{
    const size_t lds = (size_t)(lds_per_cu() / kTableWgsPerCu) / 512 * 512 - 512;
    if (narrow)
        return launch_kernel(batched_table_kernel<T, Op, true>, dim3(grid_for(ntiles)), dim3(kTB),
                             lds, s, d_items, d_table, ntiles);
    return launch_kernel(batched_table_kernel<T, Op, false>, dim3(grid_for(ntiles)), dim3(kTB),
                         lds, s, d_items, d_table, ntiles);
}

// Tile-table launcher for the element types Ts.
template <class... Ts>
hipError_t batched_table_group(xred_dtype dtype, xred_op op, const xred_item *d_items,
                               const uint32_t *d_table, bool narrow, uint64_t ntiles,
                               hipStream_t s)
{
    return with_dtype_among<Ts...>(dtype, [&](auto t) {
        using T = decltype(t);
        return with_op<T, true>(op, [&](auto o) {
            return go_table<T, decltype(o)>(d_items, d_table, narrow, ntiles, s);
        });
    });
}

// ------------------------------------------------------------- runs variant --
// Device descriptors without state between calls, so that the launch can be
// captured in a graph: the batch is cut into runs of up to 64 consecutive
// items, run r gets its own m workgroups (blockIdx m*r .. m*r+m-1), and tile j
// of the run goes to the run's workgroup j mod m.  The m workgroups of a run
// walk its tiles side by side, so the tiles in flight stay one compact
// window; and since the workgroups of later runs are dispatched in order as
// earlier ones retire, no workgroup keeps a fixed share of the whole batch.
// Every wave holds the run's descriptors, one item per lane, and finds its
// tiles with a scan, a ballot and readlanes: one memory latency and no LDS
// before the first source pointers are fetched.  (Against scanning into LDS
// and listing tiles by binary search, bf16 sum: P=8 items of 8 KiB-1 MiB, 4096 /
// 619 of them 1652 / 273 -> 1366 / 220 us; 563 items of 8-16 KiB 53 -> 17; P=16
// 3000 items 774 -> 444; and against one persistent grid of the same tiles for
// up to 64 items: 12 items 6.5 -> 5.0 us, 64 of 8 MiB 860 -> 855.)  Two
// workgroups per CU of 8 KiB tiles are within 2 % on large batches and lose
// 15 % on 64 large items.  With fewer workgroups than m * nruns (a CU budget),
// each set of m workgroups strides over the runs.
constexpr int kRunItems = 64;      // one per lane
constexpr int kRunsWgsPerCu = 1;

template <class T, class Op>
__global__ __launch_bounds__(kB) void batched_runs_kernel(const xred_item *items, int nitems,
                                                          uint32_t nruns, uint32_t m)
{
    extern __shared__ char occupancy_reservation[];
    (void)occupancy_reservation;
    const int lane = (int)(threadIdx.x & 63);
    const uint32_t w = blockIdx.x % m;
    const uint32_t sets = gridDim.x / m;
    for (uint32_t r = blockIdx.x / m; r < nruns; r += sets) {
        const int i0 = (int)r * kRunItems;
        const int n = min(kRunItems, nitems - i0);
        const xred_item it = items[i0 + min(lane, n - 1)];
        const uint64_t tiles = lane < n ? item_tiles<T>(it) : 0;
        const uint64_t upto = wave_inclusive_scan(tiles);
        const uint64_t total = readlane64(upto, 63);
        for (uint64_t g = w; g < total; g += m) {
            const int k = __popcll(__ballot(upto <= g));   // the first item past tile g
            TileDesc d;
            d.lt = g - readlane64(upto - tiles, k);
            d.srcs = (const char *const *)readlane64((uint64_t)it.srcs, k);
            d.dst = (char *)readlane64((uint64_t)it.dst, k);
            d.count = readlane64(it.count, k);
            d.nsrc = __builtin_amdgcn_readlane((int)it.nsrc, k);
            fetch_sources<T>(d);
            run_tile<T, Op, kSub, true>(d, [] {});
            __builtin_amdgcn_s_barrier();   // the waves start every tile together
        }
    }
}

template <class T, class Op>
hipError_t go_runs(const xred_item *d_items, int nitems, uint32_t nruns, uint32_t m, unsigned grid,
                   hipStream_t s)
{
    const size_t lds = (size_t)(lds_per_cu() / kRunsWgsPerCu) / 512 * 512 - 512;
    return launch_kernel(batched_runs_kernel<T, Op>, dim3(grid), dim3(kB), lds, s, d_items, nitems,
                         nruns, m);
}

// Runs launcher for the element types Ts.
template <class... Ts>
hipError_t batched_runs_group(xred_dtype dtype, xred_op op, const xred_item *d_items, int nitems,
                              uint32_t nruns, uint32_t m, unsigned grid, hipStream_t s)
{
    return with_dtype_among<Ts...>(dtype, [&](auto t) {
        using T = decltype(t);
        return with_op<T, true>(op, [&](auto o) {
            return go_runs<T, decltype(o)>(d_items, nitems, nruns, m, grid, s);
        });
    });
}

template <class T, class Op>
hipError_t go_queue(const xred_item *d_items, int nitems, QueueCtl q, unsigned grid,
                    int wgs_per_cu, hipStream_t s)
{
    size_t lds = (size_t)(lds_per_cu() / wgs_per_cu) / 512 * 512 - 512;
    const size_t need = sizeof(uint32_t) * ((size_t)nitems + 1);
    if (lds < need) lds = need;
    return launch_kernel(batched_queue_kernel<T, Op>, dim3(grid), dim3(kB), lds, s,
                         d_items, nitems, q);
}

// Queue launcher for the element types Ts.
template <class... Ts>
hipError_t batched_queue_group(xred_dtype dtype, xred_op op, const xred_item *d_items,
                               int nitems, QueueCtl q, unsigned grid, int wgs_per_cu,
                               hipStream_t s)
{
    return with_dtype_among<Ts...>(dtype, [&](auto t) {
        using T = decltype(t);
        return with_op<T, true>(op, [&](auto o) {
            return go_queue<T, decltype(o)>(d_items, nitems, q, grid, wgs_per_cu, s);
        });
    });
}

constexpr size_t rr_lds_bytes(int nitems)
{
    return sizeof(uint2) * kListMax + sizeof(uint32_t) * ((size_t)nitems + 1);
}

// The round-robin kernel's LDS is rounded up to whole kRrLdsStep blocks, so
// its occupancy is known per block count and cached per device.
constexpr size_t kRrLdsStep = 4096;
constexpr int kRrLdsSteps = (int)((rr_lds_bytes(kRrMaxItems) + kRrLdsStep - 1) / kRrLdsStep);

template <class T, class Op>
int rr_per_cu(int steps)
{
    static int cache[kMaxDevicesCached][kRrLdsSteps + 1];
    const int dev = current_device_index();
    int v = __atomic_load_n(&cache[dev][steps], __ATOMIC_RELAXED);
    if (v <= 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &v, (const void *)batched_rr_kernel<T, Op>, kB, (size_t)steps * kRrLdsStep) !=
                hipSuccess ||
            v <= 0)
            v = 1;
        __atomic_store_n(&cache[dev][steps], v, __ATOMIC_RELAXED);
    }
    return v;
}

template <class T, class Op>
hipError_t go_rr(const xred_item *d_items, int nitems, const uint32_t *d_tile_start, hipStream_t s)
{
    const int steps = (int)((rr_lds_bytes(nitems) + kRrLdsStep - 1) / kRrLdsStep);
    const unsigned grid = batched_rr_grid(rr_per_cu<T, Op>(steps));
    return launch_kernel(batched_rr_kernel<T, Op>, dim3(grid), dim3(kB),
                         (size_t)steps * kRrLdsStep, s, d_items, nitems, d_tile_start);
}

template <class T, class Op>
hipError_t go(const xred_item *d_items, int nitems, const WgStart *d_wg, unsigned grid,
              hipStream_t s)
{
    return launch_kernel(batched_kernel<T, Op>, dim3(grid), dim3(kB), 0, s, d_items, nitems, d_wg);
}

// Range-walking launcher for the element types Ts.
template <class... Ts>
hipError_t batched_group(xred_dtype dtype, xred_op op, const xred_item *d_items, int nitems,
                         const WgStart *d_wg, unsigned grid, hipStream_t s)
{
    return with_dtype_among<Ts...>(dtype, [&](auto t) {
        using T = decltype(t);
        return with_op<T, true>(op, [&](auto o) {
            return go<T, decltype(o)>(d_items, nitems, d_wg, grid, s);
        });
    });
}

// Round-robin launcher for the element types Ts.
template <class... Ts>
hipError_t batched_rr_group(xred_dtype dtype, xred_op op, const xred_item *d_items, int nitems,
                            const uint32_t *d_tile_start, hipStream_t s)
{
    return with_dtype_among<Ts...>(dtype, [&](auto t) {
        using T = decltype(t);
        return with_op<T, true>(op, [&](auto o) {
            return go_rr<T, decltype(o)>(d_items, nitems, d_tile_start, s);
        });
    });
}

}  // namespace
}  // namespace xred
