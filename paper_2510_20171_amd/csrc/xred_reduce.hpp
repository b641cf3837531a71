// xred_reduce.hpp -- launch templates of the fused P-source reduce
// (xred_allreduce_local and xred_reduce_scatter_local), instantiated per
// group of element types by xred_reduce_{float,fp8,int}.hip so the groups
// compile in parallel.
#pragma once

#include <stdlib.h>

#include <algorithm>

#include "xred_dispatch.hpp"
#include "xred_internal.hpp"
#include "xred_kernels.hpp"

namespace xred {
namespace {

// Three tile shapes, one 16-byte vector of every source per thread but for the
// second's up to 8 sources:
//
// * Up to 8 sources, launches of at most four 512-thread workgroups per CU (up
//   to 8 MiB per source) are latency-bound: 512-thread workgroups, uncapped, so
//   the whole message is in flight after the fewest workgroup dispatches (P=8
//   bf16 4 MiB per source 6.8 us against 7.0-7.4 with 128 threads; equal at 7
//   MiB; e4m3 8 MiB 11.2 / 12.3).  All four are resident at once where a kernel
//   takes at most 64 VGPRs, as most do.  More sources spread over the chip in
//   128-thread workgroups (P=32 bf16 1 / 4 / 7 MiB: 6.4 / 22.2 / 38.2 us against
//   8.1 / 23.6 / 41.6; P=16 512 KiB 3.1 against 4.3), except in the next case.
//   Counts without a kernel of their own keep the next group of 8 sources in
//   flight up to 1 MiB a source, where few waves hide the loads (bf16, rotating
//   buffers, with / without: P=9, 24, 48 512 KiB 3.6 / 3.8, 4.7 / 5.2, 7.2 / 8.3
//   us; P=9 32 MiB 54.6 / 51.2).
// * A call of at most 128 MiB of sources and output (half the MALL) mostly finds
//   the last step's buffers there, and is then bound by dispatches and by what
//   the wave cap keeps out rather than by HBM.  Up to the same number of
//   workgroups, up to 8 sources take 512-thread ones of two vectors a thread
//   while the call has at most 108 MiB, and more sources past 1 MiB each those
//   of one, uncapped (bf16, this / 128-thread tiles: P=2 12 MiB 4.3 / 6.8 us,
//   P=4 9 / 16 MiB 7.3 / 8.2, 11.2 / 12.1, P=8 12 MiB 15.3 / 16.9, e4m3 16.5 /
//   17.5; P=9 4 MiB 5.6 / 7.7, P=12 2 / 4 MiB 4.5 / 4.6, 7.8 / 8.5, P=16 2 / 4
//   MiB 5.2 / 5.4, 9.6 / 11.2, e4m3 P=16 4 MiB 10.9 / 12.1).  108 MiB is 12 MiB
//   of 8 sources: there two vectors a thread make three whole workgroups per CU;
//   at 13 to 15 MiB, a broken fourth, the 128-thread tiles win warm and from HBM
//   (two vectors / 128 threads, back to back and rotating buffers: 13 MiB 18.4 /
//   17.3, 21.6 / 20.0 us; 14 MiB 19.9 / 19.2, 22.9 / 21.3; e4m3 13 MiB 19.4 /
//   18.1, 22.5 / 20.6).  At 16 MiB it depends on the buffers' addresses: 16 MiB
//   apart 22.3 / 23.6, 25.1 / 24.3; with 4 KiB, 1 MiB or 2 MiB more between them
//   21.8 / 22.6, 22.4 / 21.0 and 22.3 / 22.3 back to back, 24.4 / 24.6, 25.2 /
//   24.0 and 25.0 / 23.9 rotating.  Outputs off the sources' grid keep two
//   vectors to 128 MiB (P=8 14 MiB 20.8 / 21.5 back to back; P=7 16 MiB 20.6 /
//   22.3).
// * Larger launches are bandwidth-bound: 128-thread workgroups with a
//   bounded number of waves per CU.  HBM3E on MI355X delivers the most when
//   a CU keeps a moderate number of loads in flight; more waves than that
//   lower the rate (P=8 bf16, 2^26 elements per source: 168.6 us against
//   190.7 us with uncapped 512-thread workgroups).  Waves per CU -> TB/s on
//   32 MiB per source: P=4 is flat from 16 waves up; P=8 is flat between 8
//   and 16 and falls at full occupancy; P=12 (runtime source count) wants
//   ~16; P=16 ~10; P=32 ~6; P=64 ~4.  The cap is applied by giving each
//   workgroup an LDS reservation it never touches, sized so that only the
//   wanted number of workgroups fit on a CU.
// * Five to eight sources want more loads in flight when each holds several
//   hundred MiB, and when a launch is only a few rounds long (12 / 16 / 20 / 24
//   waves, back to back: P=5 bf16 17 MiB 16.7 / 15.3 / 15.1 / 15.1 us, 24 MiB
//   24.1 / 23.2 / 23.1 / 23.0; P=6 24 MiB 27.9 / 26.7 / 26.8 / 26.8; P=7 24 MiB
//   29.5 / 28.2 / 28.2 / 28.7; P=8 17 MiB 22.9 / 22.5 / 22.7 / 23.1, 24 MiB 33.3
//   / 33.5 / 33.6 / 33.9; P=8 e4m3 17 MiB 25.0 / 23.7 / 23.4 / 23.8, int8 24 MiB
//   35.3 / 32.2 / 32.9 / 33.1, fp32 within 1 % of bf16); P=8 32 MiB and 128 MiB
//   12; 256 MiB 16, 360 us against 374 us; 512 MiB 24, 830 us against 963 us;
//   768 MiB 20-24, 1232 us against 1346 us).  16 and 32 sources keep their caps
//   up to 4.4 GB.
//
// Tile order of the 128-thread shape.  In address order, with one 2 KiB tile
// per workgroup, XCD x reads the 2 KiB blocks x mod 8 of every stream.  That is
// as good as any order only while all streams' blocks coincide: the buffers'
// bases on 2 KiB boundaries and equal modulo 16 KiB.  Runs of 32 tiles per XCD
// (64 KiB) do not depend on it, and let an XCD's L2 serve the lines that tiles
// off line boundaries share (P=8 bf16, bases at multiples of 512 B / 128 B /
// odd multiples of 4 KiB: 64 MiB 91.3 / 95.1 / 107.6 -> 89.2 / 89.4 / 90.3 us,
// 128 MiB 189.9 / 195.0 / 217.5 -> 191.4 / 190.4 / 194.6; 16 MiB 25.2 -> 24.1 and, on
// equal bases, 25.2 us with two vectors per 512-thread workgroup -> 23.5).
// With equal bases address order wins from about 512 MiB of sources up (P=8
// 64 MiB 87.4 against 86.9 in runs, 128 MiB 179.9 / 183.7; P=4 64 MiB 49.3 /
// 48.8, 128 MiB 104.7 / 106.2; P=32 16 MiB 86.6 / 86.8, 32 MiB 169.3 / 173.4; int8
// P=32 48 MiB 252 / 258, bf16 P=64 24 MiB 246 / 255).  Below it runs win in every
// count and type (address order / runs, rotating buffers: P=2 24 / 64 MiB 13.9 /
// 12.6, 31.5 / 29.3 us, P=3 24 MiB 17.9 / 15.8, P=6 64 MiB 72.3 / 68.4, P=12 24 MiB
// 58.1 / 50.7, P=16 24 MiB 71.7 / 66.1, P=64 8 MiB 99.8 / 88.6; P=8 24 MiB fp32 40.3 /
// 34.9, e4m3 40.0 / 35.6; int8 P=32 8 MiB 59.3 / 45.1).
constexpr int kB = 128;        // threads per workgroup, bandwidth-bound launches
constexpr int kBWide = 512;    // threads per workgroup, one-round launches
constexpr int kWideWgsPerCu = 4;   // most 512-thread workgroups per CU of one-round launches
constexpr size_t kAheadBytes = (size_t)1 << 20;      // a source of a latency-bound call
constexpr size_t kCachedBytes = (size_t)128 << 20;   // sources and output of a MALL-sized call
template <bool OFF>
constexpr size_t kTwoVecBytes = (size_t)(OFF ? 128 : 108) << 20;   // the same, two vectors a thread

// One source stays in address order: a copy that fits the L2s is served from
// them when an XCD meets its last call's lines (20 MiB 5.2 us, in runs 7.1).
bool run_order(const char *const *srcs, int nsrc, const char *dst, size_t bytes)
{
    if (nsrc == 1) return false;
    if ((size_t)nsrc * bytes <= ((size_t)512 << 20)) return true;
    uintptr_t any = (uintptr_t)dst, diff = 0;
    for (int p = 0; p < nsrc; ++p) {
        any |= (uintptr_t)srcs[p];
        diff |= (uintptr_t)srcs[p] ^ (uintptr_t)dst;
    }
    return (any & 2047u) != 0 || (diff & 16383u) != 0;
}

// Waves per CU for a compile-time source count (NP = 0, a runtime count: see
// waves_for); 0 = no cap.
// Five and six sources stream best with more waves than seven or eight (bf16
// at 128 MiB per source on two boxes, 12 / 16 / 20 waves: P=5 6.39-6.61 /
// 6.85-7.10 / 6.92-7.08 TB/s, P=6 6.69-6.82 / 6.91-6.98 / 6.90-6.91); two to
// four sources are within noise of uncapped at 16-28 waves.
template <int NP>
constexpr int waves_per_cu()
{
    return NP == 0 ? 12 : NP <= 4 ? 0 : NP == 5 ? 20 : NP == 6 ? 16 : NP <= 8 ? 12
         : NP <= 16 ? 10 : NP <= 32 ? 6 : 4;
}

// The cap of a bandwidth-bound launch with `bytes` per source.  A runtime
// source count takes fewer waves the more sources each thread reads (bf16 at
// 32 MiB per source, 8 / 10 / 12 / 16 waves: 9 sources 6.23-6.26 / 6.22-6.26 /
// 6.37-6.44 / 6.28-6.30 TB/s, 24 sources 6.28-6.29 / 6.29 / 6.26-6.30 /
// 6.06, 48 sources 6.52-6.54 / 6.54 / 6.38-6.40 / 6.10-6.12).
// Eight-bit integers (sixteen 32-bit accumulators per vector) want 16 waves
// for 5-8 sources (P=8 at 128 MiB per source, 12 / 16 waves: uint8 max 6.64-6.66
// / 6.84 TB/s, int8 sum 6.80-6.86 / 6.90-6.91; the other types are best at 12).
template <class T, int NP>
int waves_for(size_t bytes, int nsrc)
{
    if (NP == 0) return nsrc <= 12 ? 12 : nsrc <= 48 ? 10 : 6;
    constexpr bool kByteInt = !T::kFloat && T::kSize == 1;
    if (kByteInt && NP >= 5 && NP <= 8 && bytes > ((size_t)24 << 20) &&
        bytes <= ((size_t)192 << 20))
        return waves_per_cu<NP>() > 16 ? waves_per_cu<NP>() : 16;
    if (NP >= 5 && NP <= 8) {
        if (bytes > ((size_t)384 << 20)) return 24;
        if (bytes > ((size_t)192 << 20)) return waves_per_cu<NP>() > 16 ? waves_per_cu<NP>() : 16;
        if (bytes <= ((size_t)24 << 20)) return waves_per_cu<NP>() > 16 ? waves_per_cu<NP>() : 16;
    }
    return waves_per_cu<NP>();
}

// Dynamic LDS that leaves room for `waves` wavefronts per CU (0: no cap).
size_t lds_for_waves(int waves)
{
    static const long force = [] {
        const char *e = getenv("XRED_FUSED_WAVES_PER_CU");
        return e && *e ? strtol(e, nullptr, 10) : 0L;
    }();
    if (force > 0) waves = (int)force;
    if (waves <= 0) return 0;
    const int wgs = waves / (kB / 64);
    if (wgs <= 0 || wgs >= 16) return 0;     // at or beyond the natural occupancy
    return (size_t)(lds_per_cu() / wgs) / 512 * 512;
}

// ------------------------------------------------- sources at offsets --
// Sources at different offsets within 16 bytes (views into flat buffers laid
// out differently): the output grid is dst's after `lead` elements, and every
// source is read in vectors where it lies (offset_tile).
//
// Tiles go in runs per XCD whatever the size (mixed offsets, 12 waves per CU,
// in address order against runs: 19 MiB per source 29.9 / 28.3 us, 128 MiB
// 190.8 / 185.8 us).
template <class T, class Op, int B>
__global__ __launch_bounds__(B) void reduce_offset_kernel(KernargSrc<XRED_MAX_SRC> src, int nsrc,
                                                          char *dst, size_t nvec, uint32_t tail,
                                                          uint32_t lead)
{
    constexpr uint32_t kTileBytes = (uint32_t)B * 16u;
    const size_t vbytes = nvec * 16;
    const size_t lb = (size_t)lead * T::kSize;
    const uint32_t ntiles = (uint32_t)((vbytes + kTileBytes - 1) / kTileBytes);
    for (uint32_t i = blockIdx.x; i < ntiles; i += gridDim.x) {
        const size_t off = (size_t)xcd_run_tile(i, xcd_run_end(ntiles)) * kTileBytes;
        offset_tile<T, Op>(src, nsrc, dst, lb, off, tile_nrec(vbytes, off, kTileBytes));
    }
    if ((tail | lead) != 0 && blockIdx.x == ntiles % gridDim.x)
        reduce_ends<T, Op>(src, nsrc, dst, lead, tail, lead + nvec * T::kVec);
}

// waves_for with the compile-time counts the vector path would pick.
template <class T>
int waves_split(size_t bytes, int nsrc)
{
    switch (nsrc) {
    case 1: return waves_for<T, 1>(bytes, nsrc);
    case 2: return waves_for<T, 2>(bytes, nsrc);
    case 3: return waves_for<T, 3>(bytes, nsrc);
    case 4: return waves_for<T, 4>(bytes, nsrc);
    case 5: return waves_for<T, 5>(bytes, nsrc);
    case 6: return waves_for<T, 6>(bytes, nsrc);
    case 7: return waves_for<T, 7>(bytes, nsrc);
    case 8: return waves_for<T, 8>(bytes, nsrc);
    case 16: return waves_for<T, 16>(bytes, nsrc);
    case 32: return waves_for<T, 32>(bytes, nsrc);
    case 64: return waves_for<T, 64>(bytes, nsrc);
    default: return waves_for<T, 0>(bytes, nsrc);
    }
}

template <class T, class Op>
hipError_t go_offset(const char *const *srcs, int nsrc, char *dst, size_t count, const VecPlan &vp,
                     hipStream_t s)
{
    KernargSrc<XRED_MAX_SRC> ks;
    for (int p = 0; p < nsrc; ++p) ks.p[p] = srcs[p];
    for (int p = nsrc; p < XRED_MAX_SRC; ++p) ks.p[p] = nullptr;
    const size_t bytes = count * T::kSize, nvec = vp.nvec;
    const uint32_t tail = (uint32_t)(count - vp.lead - nvec * T::kVec);
    const dim3 grid(grid_for((nvec + kB - 1) / kB + ((tail | vp.lead) ? 1 : 0)));
    // 5 and 6 sources want 16 waves up to 192 MiB, 7 and 8 want 12, in every type,
    // also where the vector path takes others (mixed offsets, 12 / 16 / 20 waves:
    // bf16 P=5 19 / 64 / 128 MiB 22.1 / 19.4 / 19.6, 66.5 / 59.6 / 60.3, 131.3 / 119.7 /
    // 121.2 us, P=6 64 MiB 72.9 / 68.9 / 70.1, int8 P=5 128 MiB 137.5 / 129.1 / -; P=7
    // 64 MiB 80.5 / 82.9 / 84.9, P=8 19 / 128 MiB 28.2 / 29.1 / 29.9, 181.4 / 190.0 /
    // 194.2, f16 avg, fp32, e4m3 and int8 alike)
    const int waves = nsrc >= 5 && nsrc <= 8 && bytes <= ((size_t)192 << 20)
                          ? (nsrc <= 6 ? 16 : 12) : waves_split<T>(bytes, nsrc);
    return launch_kernel(reduce_offset_kernel<T, Op, kB>, grid, dim3(kB), lds_for_waves(waves), s,
                         ks, nsrc, dst, nvec, tail, vp.lead);
}

// OFF: dst off the grid of the sources' vectors.
template <class T, class Op, int NP, int MAXP, bool OFF>
hipError_t go_shape(const char *const *srcs, int nsrc, char *dst, size_t count, uint32_t lead,
                    hipStream_t s)
{
    KernargSrc<MAXP> ks;
    for (int p = 0; p < nsrc; ++p) ks.p[p] = srcs[p];
    for (int p = nsrc; p < MAXP; ++p) ks.p[p] = nullptr;
    const size_t nvec = (count - lead) / T::kVec;
    const uint32_t tail = (uint32_t)((count - lead) % T::kVec);
    // a short first tile up to the first source's next 128-byte line
    const size_t mis = ((uintptr_t)srcs[0] + (size_t)lead * T::kSize) & 127u;
    const uint32_t head = (uint32_t)(mis == 0 ? 0 : std::min<size_t>(128 - mis, nvec * 16));
    const size_t hv = head / 16, first = head != 0 ? 1 : 0;
    const uint64_t extra = (tail | lead) ? 1 : 0;
    const size_t bytes = count * T::kSize;
    const bool cached = bytes <= kCachedBytes / ((size_t)nsrc + 1);
    constexpr bool kFew = NP >= 1 && NP <= 8;
    const uint64_t one_round = (uint64_t)device_cus() * kWideWgsPerCu;
    const uint64_t tiles_wide = first + (nvec - hv + kBWide - 1) / kBWide + extra;
    if (tiles_wide <= one_round && (kFew || (cached && bytes > kAheadBytes)))
        return launch_kernel(reduce_vec_kernel<T, Op, NP, MAXP, 1, kBWide, OFF>,
                             dim3(grid_for(tiles_wide)), dim3(kBWide), 0, s, ks, nsrc, dst, nvec,
                             tail, head, lead, 0u);
    if constexpr (kFew) {
        const uint64_t tiles_wide2 = first + (nvec - hv + 2 * kBWide - 1) / (2 * kBWide) + extra;
        if (tiles_wide2 <= one_round && bytes <= kTwoVecBytes<OFF> / ((size_t)nsrc + 1))
            return launch_kernel(reduce_vec_kernel<T, Op, NP, MAXP, 2, kBWide, OFF>,
                                 dim3(grid_for(tiles_wide2)), dim3(kBWide), 0, s, ks, nsrc, dst,
                                 nvec, tail, head, lead, 0u);
    }
    const uint64_t tiles = first + (nvec - hv + kB - 1) / kB + extra;
    const uint32_t run_end =
        run_order(srcs, nsrc, dst, bytes) ? xcd_run_end((uint32_t)(tiles - extra)) : 0u;
    auto narrow = [&](auto kernel) {
        return launch_kernel(kernel, dim3(grid_for(tiles)), dim3(kB),
                             lds_for_waves(waves_for<T, NP>(bytes, nsrc)), s, ks, nsrc, dst, nvec,
                             tail, head, lead, run_end);
    };
    if constexpr (NP == kAnyCount)
        if (bytes <= kAheadBytes)
            return narrow(reduce_vec_kernel<T, Op, kAnyCountAhead, MAXP, 1, kB, OFF>);
    return narrow(reduce_vec_kernel<T, Op, NP, MAXP, 1, kB, OFF>);
}

template <class T, class Op, int NP, int MAXP>
hipError_t go_vec(const char *const *srcs, int nsrc, char *dst, size_t count, uint32_t lead,
                  hipStream_t s)
{
    if ((((uintptr_t)dst + (size_t)lead * T::kSize) & 15u) == 0)
        return go_shape<T, Op, NP, MAXP, false>(srcs, nsrc, dst, count, lead, s);
    return go_shape<T, Op, NP, MAXP, true>(srcs, nsrc, dst, count, lead, s);
}

template <class T, class Op>
hipError_t go(const char *const *srcs, int nsrc, char *dst, size_t count, hipStream_t s)
{
    // Sources at one offset within 16 bytes (views at one element offset, a
    // reduce-scatter shard) take the vector path, whatever dst's; others read
    // vectors where they lie (go_offset) unless the call is too short, which
    // is scalar.
    uintptr_t sdiff = 0;
    for (int p = 1; p < nsrc; ++p) sdiff |= (uintptr_t)srcs[p] ^ (uintptr_t)srcs[0];
    const VecPlan vp = vec_plan<T>((uintptr_t)srcs[0], sdiff, (uintptr_t)dst, count);
    if (!vp.any) {
        KernargSrc<XRED_MAX_SRC> ks;
        for (int p = 0; p < nsrc; ++p) ks.p[p] = srcs[p];
        for (int p = nsrc; p < XRED_MAX_SRC; ++p) ks.p[p] = nullptr;
        return launch_kernel(reduce_scalar_kernel<T, Op, kB>,
                             dim3(grid_for((count + kB - 1) / kB)), dim3(kB), 0, s, ks, nsrc, dst,
                             count);
    }
    if (!vp.grid) return go_offset<T, Op>(srcs, nsrc, dst, count, vp, s);
    const uint32_t lead = vp.lead;
    constexpr bool kWide = is_core_type<T>() && !__is_same(Op, OpAvg);
    switch (nsrc) {
    case 1: return go_vec<T, Op, 1, 8>(srcs, nsrc, dst, count, lead, s);
    case 2: return go_vec<T, Op, 2, 8>(srcs, nsrc, dst, count, lead, s);
    case 3: return go_vec<T, Op, 3, 8>(srcs, nsrc, dst, count, lead, s);
    case 4: return go_vec<T, Op, 4, 8>(srcs, nsrc, dst, count, lead, s);
    case 5: return go_vec<T, Op, 5, 8>(srcs, nsrc, dst, count, lead, s);
    case 6: return go_vec<T, Op, 6, 8>(srcs, nsrc, dst, count, lead, s);
    case 7: return go_vec<T, Op, 7, 8>(srcs, nsrc, dst, count, lead, s);
    case 8: return go_vec<T, Op, 8, 8>(srcs, nsrc, dst, count, lead, s);
    case 16:
        if constexpr (kWide) return go_vec<T, Op, 16, 16>(srcs, nsrc, dst, count, lead, s);
        break;
    case 32:
        if constexpr (kWide) return go_vec<T, Op, 32, 32>(srcs, nsrc, dst, count, lead, s);
        break;
    case 64:
        if constexpr (kWide) return go_vec<T, Op, 64, 64>(srcs, nsrc, dst, count, lead, s);
        break;
    default: break;
    }
    return go_vec<T, Op, kAnyCount, XRED_MAX_SRC>(srcs, nsrc, dst, count, lead, s);
}


// The fused launcher for the element types Ts (one translation unit each).
template <class... Ts>
hipError_t reduce_group(xred_dtype dtype, xred_op op, const char *const *srcs, int nsrc,
                        char *dst, size_t count, hipStream_t stream)
{
    return with_dtype_among<Ts...>(dtype, [&](auto t) {
        using T = decltype(t);
        return with_op<T, true>(op, [&](auto o) {
            return go<T, decltype(o)>(srcs, nsrc, dst, count, stream);
        });
    });
}

}  // namespace
}  // namespace xred
