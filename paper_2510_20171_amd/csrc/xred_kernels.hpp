// xred_kernels.hpp -- reduce-step kernels for gfx950.
//
// All kernels stream 16-byte vectors: one wavefront covers 64 lanes x 16 B =
// 1 KiB of every source per vector step, and each thread keeps U vectors of
// every source, or of a group of 8, in flight before folding (the fold order over
// sources is the fixed left fold 0..P-1 whatever the load order).
//
// Memory on the 16-byte grid is accessed through buffer resource descriptors
// built per tile (base = stream + tile offset, num_records = bytes of the tile
// that exist).  The hardware range check then replaces per-lane bounds tests: loads past
// num_records return 0 and stores past it are dropped, so the ragged last
// tile runs the same straight-line code as every other tile.  Buffer
// instructions also always address global memory, wherever the pointer came
// from, and carry the cache policy.  (Vectors off the grid, and the parts of
// narrow types' steps, take global accesses the hardware realigns.)  The policy:
// sources are read nontemporally (each byte is used once); outputs are
// written with device-scope (sc1) stores, which measured 2-5 % faster on
// MI355X for this 8:1 read/write mix than ordinary write-back stores and
// faster still than nontemporal stores; the step-wise accumulator uses
// ordinary loads and stores, which may leave it in the MALL between
// launches (not in L2: a launch starts with its L2 lines invalidated).
//
// Work is split into tiles of B*U vectors.  Work item i is processed by
// workgroup i mod gridDim.x, so with a fixed grid it always lands on the same XCD
// (workgroups are dispatched to the 8 XCDs round-robin); it is tile i, or with
// runs per XCD another tile of its block (xcd_run_tile).
#pragma once

#include "xred_device.hpp"
#include "../../include/xred.h"

namespace xred {

// Fourth dword of a raw (stride 0) buffer descriptor on gfx9-family parts:
// 32-bit data format, no swizzle.
constexpr int kRsrcWord3 = 0x00020000;
// Cache-policy bits of buffer instructions (gfx940 family): sc0 = 1, nt = 2, sc1 = 16.
constexpr int kLoadStream = 2;   // nontemporal
constexpr int kLoadKeep = 0;     // ordinary
constexpr int kStoreOut = 16;    // sc1: device scope
constexpr int kStoreKeep = 0;    // ordinary write-back

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// Global accesses at any byte alignment (the hardware realigns them).
typedef u32x4 __attribute__((aligned(1))) u32x4_any;
typedef u32x2 __attribute__((aligned(1))) u32x2_any;
typedef uint32_t __attribute__((aligned(1))) u32_any;
typedef const __attribute__((address_space(1))) char *global_bytes;

__device__ __forceinline__ rsrc_t make_rsrc(const char *base, uint32_t nbytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, (int)nbytes, kRsrcWord3);
}

template <int POL>
__device__ __forceinline__ u32x4 bload(rsrc_t r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, POL);
}

template <int POL>
__device__ __forceinline__ void bstore(u32x4 v, rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, POL);
}

// One result vector, `o` bytes into a tile at `base` of which nrec bytes (whole
// vectors) exist.  OFF: off the 16-byte grid, where the vector is one unaligned
// nontemporal store: the output is one stream of P + 1, and from HBM its
// misalignment costs little (P=8 bf16, output off the sources' grid, 4 / 16 / 128
// MiB per source: 7.0 / 25.0 / 186 us against 6.8 / 25.1 / 192 us on it;
// realigning the results across lanes, with narrow stores at each wavefront's
// ends, took 7.4 / 25.7 / 195; of calls that stay in the MALL only those around 4
// MiB were faster realigned, P=6 and 7 3.6 and 3.9 us against 4.0 and 4.5).
template <bool OFF>
__device__ __forceinline__ void store_out(u32x4 v, char *base, uint32_t nrec, uint32_t o)
{
    if constexpr (!OFF) {
        bstore<kStoreOut>(v, make_rsrc(base, nrec), o);
    } else {
        // the vector stays above the test: sunk below it with its fold, it would
        // keep every source's loads in registers (P=64 bf16: 254 VGPRs)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t w = v[i];
            __asm__ volatile("" : "+v"(w));
            v[i] = w;
        }
        // a global store also where the address came from another lane's registers
        if (o < nrec)
            __builtin_nontemporal_store(
                v, (__attribute__((address_space(1))) u32x4_any *)(base + o));
    }
}

// Bytes of a tile that exist: min(tile, total - off).
__device__ __forceinline__ uint32_t tile_nrec(size_t total, size_t off, uint32_t tile)
{
    const size_t left = total - off;
    return left < tile ? (uint32_t)left : tile;
}

// Source pointers passed by value in the kernel arguments (<= MAXP sources).
template <int MAXP>
struct KernargSrc {
    const char *p[MAXP];
    __device__ __forceinline__ const char *operator()(int i) const { return p[i]; }
};

// Scalar load of a value every lane of the wavefront reads at the same
// address: going through the constant address space makes the compiler use
// s_load into SGPRs, so buffer descriptors built from the value are uniform
// (a vector load would force a readfirstlane loop around every buffer access).
template <class V>
__device__ __forceinline__ V sload(const V *p)
{
    return *(const __attribute__((address_space(4))) V *)p;
}

// Source pointers read from a device array (batched descriptors).
struct GlobalSrc {
    const char *const *p;
    __device__ __forceinline__ const char *operator()(int i) const { return sload(p + i); }
};

// Geometry of one tile of one 16-byte-vector stream: the byte offset of the
// tile and how many of its bytes exist.
struct Tile {
    size_t off;     // byte offset of the tile in every stream
    uint32_t nrec;  // bytes of the tile inside the streams' vector part
};

// Fold G consecutive sources starting at p0 into acc (G known at compile time).
// FIRST: the first source initialises the accumulator instead of being folded.
template <class T, class Op, int G, int U, int B, bool FIRST, class Src>
__device__ __forceinline__ void fold_group(typename T::Acc (&acc)[U][T::kVec], const Src &src,
                                           int p0, Tile tl)
{
    u32x4 in[G][U];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const rsrc_t r = make_rsrc(src(p0 + g) + tl.off, tl.nrec);
#pragma unroll
        for (int u = 0; u < U; ++u)
            in[g][u] = bload<kLoadStream>(r, (uint32_t)(u * B + threadIdx.x) * 16u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (FIRST && g == 0) up_vec<T>(in[0][u], acc[u]);
            else fold_vec<T, Op>(acc[u], in[g][u]);
        }
    }
}

// NG full groups of 8 sources (compile time), software pipelined: the loads of
// group g+1 are issued before group g is folded, so a wave always has the next
// group's bytes in flight while it folds.  Fold order is still 0..8*NG-1.
template <class T, class Op, int NG, int U, int B, class Src>
__device__ __forceinline__ void fold_groups_pipelined(typename T::Acc (&acc)[U][T::kVec],
                                                      const Src &src, Tile tl)
{
    u32x4 buf[2][8][U];
#pragma unroll
    for (int g = 0; g <= NG; ++g) {
        if (g < NG) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const rsrc_t r = make_rsrc(src(8 * g + j) + tl.off, tl.nrec);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    buf[g & 1][j][u] =
                        bload<kLoadStream>(r, (uint32_t)(u * B + threadIdx.x) * 16u);
            }
        }
        if (g > 0) {
            const int h = (g - 1) & 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (g == 1 && j == 0) up_vec<T>(buf[h][0][u], acc[u]);
                    else fold_vec<T, Op>(acc[u], buf[h][j][u]);
                }
            }
        }
    }
}

// Any number of sources above 8, one group of loads at a time: groups of 8 and
// an exact remainder.  One group in registers leaves room for 8 waves per SIMD,
// which is what hides the loads in launches without a wave cap.
template <class T, class Op, int U, int B, class Src>
__device__ __forceinline__ void fold_groups(typename T::Acc (&acc)[U][T::kVec], const Src &src,
                                            int nsrc, Tile tl)
{
    fold_group<T, Op, 8, U, B, true>(acc, src, 0, tl);
    int p = 8;
    for (; p + 8 <= nsrc; p += 8) fold_group<T, Op, 8, U, B, false>(acc, src, p, tl);
    switch (nsrc - p) {
    case 1: fold_group<T, Op, 1, U, B, false>(acc, src, p, tl); break;
    case 2: fold_group<T, Op, 2, U, B, false>(acc, src, p, tl); break;
    case 3: fold_group<T, Op, 3, U, B, false>(acc, src, p, tl); break;
    case 4: fold_group<T, Op, 4, U, B, false>(acc, src, p, tl); break;
    case 5: fold_group<T, Op, 5, U, B, false>(acc, src, p, tl); break;
    case 6: fold_group<T, Op, 6, U, B, false>(acc, src, p, tl); break;
    case 7: fold_group<T, Op, 7, U, B, false>(acc, src, p, tl); break;
    default: break;
    }
}

// This thread's vectors of 8 consecutive sources.
struct Group8 {
    u32x4 v[8];
};

// Fold sources [p0, min(nsrc, p0 + 8)) into acc, in order; source 0 starts it.
template <class T, class Op, bool FULL>
__device__ __forceinline__ void fold8(typename T::Acc (&acc)[T::kVec], const Group8 &g, int nsrc,
                                      int p0)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (FULL || p0 + j < nsrc) {
            if (j == 0 && p0 == 0) up_vec<T>(g.v[0], acc);
            else fold_vec<T, Op>(acc, g.v[j]);
        }
    }
}

// Issue the loads of sources [p0, p0 + 8) of one tile.  Sources past nsrc get
// an empty range, so the number of loads in flight is known at compile time.
template <class Src>
__device__ __forceinline__ void fetch8(Group8 &g, const Src &src, int nsrc, int p0, Tile tl)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool on = p0 + j < nsrc;
        g.v[j] = bload<kLoadStream>(make_rsrc(src(on ? p0 + j : 0) + tl.off, on ? tl.nrec : 0u),
                                    (uint32_t)threadIdx.x * 16u);
    }
}

// Any number of sources above 8, one vector per thread: the next group's loads
// in flight while one is folded (fold order 0..nsrc-1).  Twice the registers of
// fold_groups (bf16 sum 94 VGPRs against 58, e4m3 125 against 79), so for
// launches with few waves, whose time is one chain of loads.
template <class T, class Op, class Src>
__device__ __forceinline__ void fold_groups_ahead(typename T::Acc (&acc)[T::kVec], const Src &src,
                                                  int nsrc, Tile tl)
{
    Group8 a, b;
    fetch8(a, src, nsrc, 0, tl);
#pragma nounroll
    for (int p0 = 0;; p0 += 16) {
        fetch8(b, src, nsrc, p0 + 8, tl);
        fold8<T, Op, true>(acc, a, nsrc, p0);
        if (p0 + 16 >= nsrc) {
            fold8<T, Op, false>(acc, b, nsrc, p0 + 8);
            return;
        }
        fetch8(a, src, nsrc, p0 + 16, tl);
        fold8<T, Op, true>(acc, b, nsrc, p0 + 8);
        if (p0 + 24 >= nsrc) {
            fold8<T, Op, false>(acc, a, nsrc, p0 + 16);
            return;
        }
    }
}

// Source counts known at launch only.
constexpr int kAnyCount = 0, kAnyCountAhead = -1;

// One tile: U vectors per thread at tile-relative vector u*B + threadIdx.x.
// 0 < NP <= 8: exactly NP sources, all loads issued before folding;
// NP = 16, 32, 64: whole groups of 8, software pipelined;
// NP == kAnyCount: any nsrc above 8, in groups of 8 (fold_groups);
// NP == kAnyCountAhead: the same, the next group in flight (fold_groups_ahead).
// Every variant folds in source order 0..P-1.  OFF: dst + tl.off sits off the
// 16-byte grid.
template <class T, class Op, int NP, int U, int B, bool OFF = false, class Src>
__device__ __forceinline__ void reduce_tile(const Src &src, int nsrc, char *dst, Tile tl)
{
    typename T::Acc acc[U][T::kVec];
    if constexpr (NP == kAnyCountAhead) {
        static_assert(U == 1, "one vector per thread");
        fold_groups_ahead<T, Op>(acc[0], src, nsrc, tl);
    } else if constexpr (NP == kAnyCount) {
        fold_groups<T, Op, U, B>(acc, src, nsrc, tl);
    } else if constexpr (NP > 8) {
        static_assert(NP % 8 == 0, "compile-time source counts above 8 are whole groups");
        fold_groups_pipelined<T, Op, NP / 8, U, B>(acc, src, tl);
    } else {
        fold_group<T, Op, NP, U, B, true>(acc, src, 0, tl);
    }
    if constexpr (__is_same(Op, OpAvg)) {
        const int n = NP > 0 ? NP : nsrc;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < T::kVec; ++j) acc[u][j] = avg_scale<T, Op>(acc[u][j], n);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        store_out<OFF>(down_vec<T, Op>(acc[u]), dst + tl.off, tl.nrec,
                       (uint32_t)(u * B + threadIdx.x) * 16u);
}

// Element i (scalar path): leads and tails shorter than a vector, and calls
// without a whole vector.  The loads of up to 8 sources are issued before they
// are folded, in source order.
template <class T, class Op, class Src>
__device__ __forceinline__ void reduce_elem(const Src &src, int nsrc, char *dst, size_t i)
{
    typename T::Acc a{};
    for (int p = 0; p < nsrc; p += 8) {
        typename T::Acc x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (p + q < nsrc) x[q] = up1<T>(src(p + q), i);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (p + q < nsrc) a = p + q == 0 ? x[q] : combine<T, Op>(a, x[q]);
    }
    down1<T, Op>(dst, i, avg_scale<T, Op>(a, nsrc));
}

// The elements of one reduction outside its vectors: the first nl (its lead,
// or 0) and the nt from element tail_at on (its tail, or 0), one per thread t
// of one wavefront, so both are folded by one chain of loads.
template <class T, class Op, class Src>
__device__ __forceinline__ void reduce_ends(const Src &src, int nsrc, char *dst, uint32_t nl,
                                            uint32_t nt, size_t tail_at, uint32_t t = threadIdx.x)
{
    if (t < nl + nt) reduce_elem<T, Op>(src, nsrc, dst, t < nl ? (size_t)t : tail_at + (t - nl));
}

// Bytes [s, s+16) of the 32 bytes lo:hi (lo at the lower address), 0 < s < 16.
__device__ __forceinline__ u32x4 bytes_from(u32x4 lo, u32x4 hi, uint32_t s)
{
    const uint32_t w[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    const uint32_t b = s & 3u;
    u32x4 o;
    switch (s >> 2) {
    case 0:
        for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_alignbyte(w[i + 1], w[i], b);
        break;
    case 1:
        for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_alignbyte(w[i + 2], w[i + 1], b);
        break;
    case 2:
        for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_alignbyte(w[i + 3], w[i + 2], b);
        break;
    default:
        for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_alignbyte(w[i + 4], w[i + 3], b);
        break;
    }
    return o;
}

// The 16-byte results of B lanes, lane q's for output bytes [16q, 16q + 16)
// of `base`, where base sits c bytes past a 16-byte boundary (0 < c < 16, a
// multiple of the element size) and `nrec` of the B*16 bytes exist.  Output
// bytes [16q - c, 16q + 16 - c) are lane q-1's last c result bytes and lane
// q's first 16 - c, so every lane but the first of its wavefront takes its
// neighbour's result (a lane shuffle) and stores one aligned 16-byte vector.
// The two chunks cut by a wavefront's ends (16 - c bytes at its first lane,
// c at its last lane with a vector) go out in aligned pieces of the largest
// power of two dividing c, 16 bytes in all, from up to 16 lanes in one store
// instruction.  Every lane of the workgroup must be active.
__device__ __forceinline__ void split_store(u32x4 mine, char *base, uint32_t nrec, uint32_t c)
{
    const uint32_t q = threadIdx.x, l = q & 63u;
    u32x4 prev;
#pragma unroll
    for (int i = 0; i < 4; ++i) prev[i] = __shfl_up(mine[i], 1u, 64);
    if (l != 0)
        bstore<kStoreOut>(bytes_from(prev, mine, 16u - c), make_rsrc(base - c, nrec), 16u * q);
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(q >> 6)) * 64u;
    const uint32_t nl = nrec / 16u;   // lanes with a vector
    if (w0 >= nl) return;
    const uint32_t last = nl - 1u - w0 < 63u ? nl - 1u - w0 : 63u;
    u32x4 r0, rl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        r0[i] = (uint32_t)__builtin_amdgcn_readlane((int)mine[i], 0);
        rl[i] = (uint32_t)__builtin_amdgcn_readlane((int)mine[i], (int)last);
    }
    const uint32_t piece = c & (~c + 1u);
    const uint32_t hp = (16u - c) / piece;
    if (l >= 16u / piece) return;
    const bool head = l < hp;
    const uint32_t o = head ? l * piece : 16u - c + (l - hp) * piece;   // byte of the vector
    const uint32_t at = 16u * (w0 + (head ? 0u : last)) + o;             // byte of `base`
    const u32x4 v = head ? r0 : rl;
    const uint32_t d = o >> 2;
    const uint32_t x = d == 0 ? v[0] : d == 1 ? v[1] : d == 2 ? v[2] : v[3];
    const rsrc_t w = make_rsrc(base, nrec);
    switch (piece) {
    case 8: {
        const u32x2 x2 = {x, d == 0 ? v[1] : v[3]};
        __builtin_amdgcn_raw_buffer_store_b64(x2, w, at, 0, kStoreOut);
        break;
    }
    case 4: __builtin_amdgcn_raw_buffer_store_b32(x, w, at, 0, kStoreOut); break;
    case 2:
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(x >> (8u * (o & 3u))), w, at, 0,
                                              kStoreOut);
        break;
    default:
        __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(x >> (8u * (o & 3u))), w, at, 0,
                                             kStoreOut);
        break;
    }
}

// Sources at different offsets within 16 bytes: each vector is one unaligned
// global load of exactly its bytes.  On whole dwords that costs no more than an
// aligned load, off them about a fifth more (P=8 bf16, 19 MiB / 128 MiB per
// source: aligned 28.2 / 185 us; offsets of which half are whole dwords 28.3 /
// 186, every source 6 bytes off 34 / 222; reading aligned vectors and joining
// neighbours' across lanes took 32.3 / 218.7 at any offsets, and the dword
// below each vector with a lane shift of one dword 30 / 200; int8 at mixed byte
// offsets 64 / 128 MiB 98 / 200 here and 97 / 187 joined across lanes, e4m3 98 / 200
// and 118 / 230).
template <int G, class Src>
__device__ __forceinline__ void fetch_any(u32x4 (&v)[G], const Src &src, int p0, size_t at,
                                          uint32_t o)
{
    // both opaque, so that each load takes a scalar base and a 32-bit lane
    // offset (64-bit lane addresses took 186 VGPRs, too many for 12 waves per CU)
    __asm__("" : "+v"(o));
#pragma unroll
    for (int j = 0; j < G; ++j) {
        global_bytes base = (global_bytes)(src(p0 + j) + at);
        __asm__("" : "+s"(base));
        v[j] = __builtin_nontemporal_load(
            (const __attribute__((address_space(1))) u32x4_any *)(base + o));
    }
}

template <class T, class Op, int G, bool FIRST, class Src>
__device__ __forceinline__ void fold_rest(typename T::Acc (&acc)[T::kVec], const Src &src, int p0,
                                          size_t at, uint32_t o)
{
    u32x4 v[G];
    fetch_any(v, src, p0, at, o);
#pragma unroll
    for (int j = 0; j < G; ++j) {
        if (FIRST && j == 0) up_vec<T>(v[0], acc);
        else fold_vec<T, Op>(acc, v[j]);
    }
}

// The last n < 8 sources, from p0 on.
template <class T, class Op, bool FIRST, class Src>
__device__ __forceinline__ void fold_last(typename T::Acc (&acc)[T::kVec], const Src &src, int p0,
                                          int n, size_t at, uint32_t o)
{
    switch (n) {
    case 1: fold_rest<T, Op, 1, FIRST>(acc, src, p0, at, o); break;
    case 2: fold_rest<T, Op, 2, FIRST>(acc, src, p0, at, o); break;
    case 3: fold_rest<T, Op, 3, FIRST>(acc, src, p0, at, o); break;
    case 4: fold_rest<T, Op, 4, FIRST>(acc, src, p0, at, o); break;
    case 5: fold_rest<T, Op, 5, FIRST>(acc, src, p0, at, o); break;
    case 6: fold_rest<T, Op, 6, FIRST>(acc, src, p0, at, o); break;
    case 7: fold_rest<T, Op, 7, FIRST>(acc, src, p0, at, o); break;
    default: break;
    }
}

// One tile of output vectors, one per thread: byte lb + off of dst is on a
// 16-byte boundary, nrec > 0 bytes of the tile exist, the sources lie anywhere.
// Groups of 8 sources, all loads of a group in flight.
template <class T, class Op, class Src>
__device__ __forceinline__ void offset_tile(const Src &src, int nsrc, char *dst, size_t lb,
                                            size_t off, uint32_t nrec)
{
    typename T::Acc acc[T::kVec];
    const size_t at = lb + off;
    // lanes past the tile's end read its first vector; their store is dropped
    const uint32_t o = threadIdx.x * 16u < nrec ? threadIdx.x * 16u : 0u;
    if (nsrc < 8) {
        fold_last<T, Op, true>(acc, src, 0, nsrc, at, o);
    } else {
        fold_rest<T, Op, 8, true>(acc, src, 0, at, o);
        int p = 8;
        for (; p + 8 <= nsrc; p += 8) fold_rest<T, Op, 8, false>(acc, src, p, at, o);
        fold_last<T, Op, false>(acc, src, p, nsrc - p, at, o);
    }
    if constexpr (__is_same(Op, OpAvg)) {
#pragma unroll
        for (int e = 0; e < T::kVec; ++e) acc[e] = avg_scale<T, Op>(acc[e], nsrc);
    }
    bstore<kStoreOut>(down_vec<T, Op>(acc), make_rsrc(dst + at, nrec), threadIdx.x * 16u);
}

// How a reduction's elements are cut: `lead` of them one by one, nvec vectors,
// the rest one by one.  Sources at one offset within 16 bytes (grid): their
// lead ends on their next 16-byte boundary, wherever the output then lies.
// Otherwise the output's grid rules (offset_tile).  !any: not one whole
// vector then, or an output off its element size.
struct VecPlan {
    uint64_t nvec;
    uint32_t lead;
    bool any, grid;
};

// s0: the first source; sdiff: bits in which some source differs from it.
template <class T>
__host__ __device__ __forceinline__ VecPlan vec_plan(uintptr_t s0, uintptr_t sdiff, uintptr_t dst,
                                                     uint64_t count)
{
    const bool grid = (sdiff & 15u) == 0 && (s0 & 15u) % T::kSize == 0;
    const uint64_t to = ((0 - (grid ? s0 : dst)) & 15u) / T::kSize;
    const uint32_t lead = (uint32_t)(to < count ? to : count);
    const uint64_t nvec = (count - lead) / T::kVec;
    return VecPlan{nvec, lead, grid || (nvec != 0 && dst % T::kSize == 0), grid};
}

// Work item i's tile when runs of kXcdRun consecutive tiles go to one XCD
// (workgroup i runs on XCD i mod 8): within each block of 8 runs, XCD x takes
// run x.  Work items from `end` on (xcd_run_end: the last, partial block) keep
// their order.
constexpr uint32_t kXcdRun = 32;
constexpr int kRunsB = 128;   // largest workgroup whose tiles may go in runs
__host__ __device__ __forceinline__ uint32_t xcd_run_end(uint32_t ntiles)
{
    return ntiles & ~(8 * kXcdRun - 1);
}
__device__ __forceinline__ uint32_t xcd_run_tile(uint32_t i, uint32_t end)
{
    if (i >= end) return i;
    return (i & ~(8 * kXcdRun - 1)) + (i & 7) * kXcdRun + ((i >> 3) & (kXcdRun - 1));
}

// ------------------------------------------------------ fused P-source --
// Waves per SIMD the compiler must leave room for (1: its own choice).  Two
// vectors of 16 values each from 7 or 8 sources took 129-139 VGPRs, one
// 512-thread workgroup per CU; under 128 two fit (e4m3 sum, P=8 12 MiB per
// source: 18.3 -> 16.5 us; int8 max 17.0 -> 15.4).
template <class T, int NP, int U, bool OFF>
constexpr int reduce_min_waves()
{
    return U != 2 || T::kVec != 16 || OFF ? 1 : NP == 7 ? 5 : NP == 8 ? 4 : 1;
}

// dst[i] = fold_p src_p[i] for lead + nvec*kVec + tail elements, every source
// at the same offset within 16 bytes, dst too or (OFF) at another: the first
// `lead` elements (fewer than a vector) bring the sources to a 16-byte boundary
// and, like the last `tail` ones, are done by one workgroup, scalar; the nvec
// vectors between go in tiles of B * U vectors (the last one ragged, cut by the buffer
// range check).  `head` (a multiple of 16 below 128, at most nvec*16) is the
// byte length of a first, short tile that ends where the first source
// reaches a 128-byte line: the other tiles then start on line boundaries, so
// no line is split between two tiles (whose workgroups, on different XCDs,
// would each fetch it).
//
// The first run_end tiles go in runs per XCD (xcd_run_tile; 0: all in address
// order, as always in the larger workgroups).  A kernel argument and 32-bit
// indices keep the loop's scalar registers few (int8 prod at P=8: 88 VGPRs with
// 64-bit indices and the end computed per tile, 57 so).
// OFF is a template parameter because both store forms in one kernel cost the
// aligned one registers (int8 prod at P=8 61 -> 87 VGPRs, fp32 at P=64 36 bytes
// of scratch).
template <class T, class Op, int NP, int MAXP, int U, int B, bool OFF>
__global__ __launch_bounds__(B, (reduce_min_waves<T, NP, U, OFF>())) void reduce_vec_kernel(
    KernargSrc<MAXP> src, int nsrc, char *dst, size_t nvec, uint32_t tail, uint32_t head,
    uint32_t lead, uint32_t run_end)
{
    constexpr uint32_t kTileBytes = (uint32_t)B * U * 16u;
    const size_t vbytes = nvec * 16;
    const size_t lb = (size_t)lead * T::kSize;   // bytes before the first vector
    const uint32_t first = head != 0 ? 1u : 0u;
    const uint32_t ntiles = first + (uint32_t)((vbytes - head + kTileBytes - 1) / kTileBytes);
    for (uint32_t i = blockIdx.x; i < ntiles; i += gridDim.x) {
        const uint32_t t = B <= kRunsB ? xcd_run_tile(i, run_end) : i;
        const bool h = t < first;
        const size_t off = h ? 0 : head + (size_t)(t - first) * kTileBytes;
        reduce_tile<T, Op, NP, U, B, OFF>(
            src, nsrc, dst, Tile{lb + off, h ? head : tile_nrec(vbytes, off, kTileBytes)});
    }
    if ((tail | lead) != 0 && blockIdx.x == ntiles % gridDim.x)
        reduce_ends<T, Op>(src, nsrc, dst, lead, tail, lead + nvec * T::kVec);
}

// Any alignment: one element per thread per step.
template <class T, class Op, int B>
__global__ __launch_bounds__(B) void reduce_scalar_kernel(KernargSrc<XRED_MAX_SRC> src, int nsrc,
                                                          char *dst, size_t count)
{
    const size_t stride = (size_t)gridDim.x * B;
    for (size_t i = (size_t)blockIdx.x * B + threadIdx.x; i < count; i += stride)
        reduce_elem<T, Op>(src, nsrc, dst, i);
}

// ------------------------------------------------------------ step-wise --
// A thread owns whole 16-byte accumulator vectors (PV = acc_per_vec values),
// vector u*B + threadIdx.x of its tile, and reads the PV * kSize input bytes
// (4, 8 or 16) that belong to each: a wavefront's accumulator accesses are 1 KiB
// contiguous for every type.  (With a 16-byte input vector per thread the
// lanes of a narrow type stepped 32 or 64 bytes through the accumulator,
// four fifths of a step's bytes and more: bf16 4M elements 7.05 us a step
// against 6.0 now, e4m3 9.3 against 5.4, both 6.7 TB/s now.)
//
// Input and output parts may sit at any element offset.  Buffer accesses need
// only 4-byte alignment, which every accumulator and every part of a 4- or
// 8-byte type has; narrower types' input goes through global loads the hardware
// realigns, their output through device-scope buffer stores where it is 4-byte
// aligned and ordinary global stores elsewhere.  (4M elements, global accesses
// under per-lane tests throughout: fp32 plain step / FINAL / cast 7.6 / 7.5 / 5.1 us,
// 7.1 / 6.85 / 3.85 so, fp64 16.0 / 16.4 / 12.8 and 15.9 / 15.6 / 10.0; bf16 16M
// FINAL / cast 20.5 / 17.9 and 19.7 / 14.6.  bf16 chunks cut at odd lengths, 4M: 11
// us element by element, 6.3 now.)

// Input or output bytes of one accumulator vector.
template <class T>
constexpr int part_bytes() { return acc_per_vec<T>() * T::kSize; }

// Input part q of a tile at `base` that holds n > 0 of them, in the low words of
// a vector, the others 0.  Parts of types of 4 and 8 bytes are 4-byte aligned,
// which is all a buffer load needs, and past the end read 0; narrower types'
// parts lie anywhere, and lanes past the end read part 0.
template <class T>
__device__ __forceinline__ u32x4 load_part(const char *base, uint32_t n, uint32_t q)
{
    constexpr int BYTES = part_bytes<T>();
    static_assert(BYTES == 4 || BYTES == 8 || BYTES == 16, "whole accumulator vectors");
    if constexpr (T::kSize >= 4) {
        return bload<kLoadStream>(make_rsrc(base, n * 16u), q * 16u);
    } else {
        const char *p = base + (size_t)(q < n ? q : 0u) * BYTES;
        if constexpr (BYTES == 8) {
            const u32x2 x = __builtin_nontemporal_load((const u32x2_any *)p);
            return u32x4{x[0], x[1], 0u, 0u};
        } else {
            return u32x4{__builtin_nontemporal_load((const u32_any *)p), 0u, 0u, 0u};
        }
    }
}

// Output part q of such a tile; parts past the end are not stored.
template <class T>
__device__ __forceinline__ void store_part(u32x4 v, char *base, uint32_t n, uint32_t q)
{
    constexpr int BYTES = part_bytes<T>();
    if constexpr (T::kSize >= 4) {
        bstore<kStoreOut>(v, make_rsrc(base, n * 16u), q * 16u);
    } else if (((uintptr_t)base & 3u) == 0) {
        const rsrc_t r = make_rsrc(base, n * BYTES);
        if constexpr (BYTES == 8)
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, r, q * 8u, 0, kStoreOut);
        else
            __builtin_amdgcn_raw_buffer_store_b32(v[0], r, q * 4u, 0, kStoreOut);
    } else if (q < n) {
        char *p = base + (size_t)q * BYTES;
        if constexpr (BYTES == 8) *(u32x2_any *)p = u32x2{v[0], v[1]};
        else *(u32_any *)p = v[0];
    }
}

// The first PV values of a vector's up(), and down() of PV values into its
// low words (the other lanes are constants the compiler drops).
template <class T>
__device__ __forceinline__ void up_part(u32x4 v, typename T::Acc (&a)[acc_per_vec<T>()])
{
    typename T::Acc w[T::kVec];
    up_vec<T>(v, w);
#pragma unroll
    for (int j = 0; j < acc_per_vec<T>(); ++j) a[j] = w[j];
}

template <class T, class Op>
__device__ __forceinline__ u32x4 down_part(const typename T::Acc (&a)[acc_per_vec<T>()])
{
    typename T::Acc w[T::kVec];
#pragma unroll
    for (int j = 0; j < T::kVec; ++j) w[j] = j < acc_per_vec<T>() ? a[j] : typename T::Acc(0);
    return down_vec<T, Op>(w);
}

// Accumulator vectors [t*B*U, ...) of nv.
template <class T, class Op, unsigned FLAGS, int U, int B>
__device__ __forceinline__ void step_tile(const char *in, char *acc, char *dst, size_t t,
                                          size_t nv)
{
    constexpr bool kInit = (FLAGS & XRED_STEP_INIT) != 0, kFinal = (FLAGS & XRED_STEP_FINAL) != 0;
    constexpr int PV = acc_per_vec<T>();           // accumulator values per vector
    constexpr int PB = part_bytes<T>();
    constexpr uint32_t kTile = (uint32_t)B * U;
    const size_t v0 = t * kTile;
    const uint32_t n = nv - v0 < kTile ? (uint32_t)(nv - v0) : kTile;
    const rsrc_t racc = make_rsrc(acc + v0 * 16, n * 16u);
    u32x4 x[U];
    typename T::Acc a[U][PV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t q = (uint32_t)u * B + threadIdx.x;
        x[u] = load_part<T>(in + v0 * PB, n, q);
    }
    if constexpr (!kInit) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            unpack_acc<T>(bload<kLoadKeep>(racc, ((uint32_t)u * B + threadIdx.x) * 16u), a[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t q = (uint32_t)u * B + threadIdx.x;
        typename T::Acc b[PV];
        up_part<T>(x[u], b);
#pragma unroll
        for (int j = 0; j < PV; ++j) a[u][j] = kInit ? b[j] : combine<T, Op>(a[u][j], b[j]);
        if constexpr (kFinal) {
            store_part<T>(down_part<T, Op>(a[u]), dst + v0 * PB, n, q);
        } else {
#pragma unroll
            for (int j = 0; j < PV; ++j) a[u][j] = finalize<T, Op>(a[u][j]);
            bstore<kStoreKeep>(pack_acc<T>(a[u]), racc, q * 16u);
        }
    }
}

template <class T, class Op, unsigned FLAGS>
__device__ __forceinline__ void step_elem(const char *in, char *acc, char *dst, size_t i)
{
    constexpr bool kInit = (FLAGS & XRED_STEP_INIT) != 0, kFinal = (FLAGS & XRED_STEP_FINAL) != 0;
    typename T::Acc x = up1<T>(in, i);
    typename T::Acc a;
    if constexpr (kInit) {
        a = x;
    } else {
        a = combine<T, Op>(((const typename T::Acc *)acc)[i], x);
    }
    if constexpr (kFinal)
        down1<T, Op>(dst, i, a);
    else
        ((typename T::Acc *)acc)[i] = finalize<T, Op>(a);
}

// One ReduceCopy step over nv accumulator vectors and the `tail` elements
// after them (fewer than a vector, by one workgroup).
template <class T, class Op, unsigned FLAGS, int U, int B>
__global__ __launch_bounds__(B) void step_kernel(const char *in, char *acc, char *dst, size_t nv,
                                                 uint32_t tail)
{
    constexpr size_t kTile = (size_t)B * U;
    const size_t ntiles = (nv + kTile - 1) / kTile;
    for (size_t t = blockIdx.x; t < ntiles; t += gridDim.x)
        step_tile<T, Op, FLAGS, U, B>(in, acc, dst, t, nv);
    if (tail != 0 && blockIdx.x == ntiles % gridDim.x && threadIdx.x < tail)
        step_elem<T, Op, FLAGS>(in, acc, dst, nv * acc_per_vec<T>() + threadIdx.x);
}

// dst = down(acc): the closing cast of a step-wise sequence, by the same
// split (one accumulator vector per thread and access).
template <class T, int U, int B>
__global__ __launch_bounds__(B) void acc_cast_kernel(const char *acc, char *dst, size_t nv,
                                                     uint32_t tail)
{
    constexpr int PV = acc_per_vec<T>();
    constexpr int PB = part_bytes<T>();
    constexpr uint32_t kTile = (uint32_t)B * U;
    const size_t ntiles = (nv + kTile - 1) / kTile;
    for (size_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const size_t v0 = t * kTile;
        const uint32_t n = nv - v0 < kTile ? (uint32_t)(nv - v0) : kTile;
        const rsrc_t racc = make_rsrc(acc + v0 * 16, n * 16u);
        typename T::Acc a[U][PV];
#pragma unroll
        for (int u = 0; u < U; ++u)
            unpack_acc<T>(bload<kLoadStream>(racc, ((uint32_t)u * B + threadIdx.x) * 16u), a[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t q = (uint32_t)u * B + threadIdx.x;
            store_part<T>(down_part<T, OpSum>(a[u]), dst + v0 * PB, n, q);
        }
    }
    if (tail != 0 && blockIdx.x == ntiles % gridDim.x && threadIdx.x < tail) {
        const size_t i = nv * PV + threadIdx.x;
        down1<T, OpSum>(dst, i, ((const typename T::Acc *)acc)[i]);
    }
}

}  // namespace xred
