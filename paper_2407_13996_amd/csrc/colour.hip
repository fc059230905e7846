// Batched XOR-hash colouring and the ordered page-table build.
//
// Colour bit k of an address is the parity of (address & M_k).  The
// classify kernel hands out tiles to single wavefronts.  A wavefront
// streams its tile's 8-byte addresses through buffer loads, each
// instruction reading 1 KiB of consecutive addresses and each lane keeping
// 8 such loads (16 addresses) in flight, colours them by table lookups
// (the hash is linear over GF(2)), and writes one colour byte per address:
// it passes its tile's 1024 colour bytes through its own 1 KiB of LDS so
// that each lane stores 16 consecutive colours per 16-byte store.  Tiles
// cover the largest multiple of 16 addresses, through buffer ranges that end
// there (so the tile body has no branch around its memory accesses); the
// last n mod 16 addresses are coloured by the grid's last workgroup, or, in a
// static launch without a histogram, by the first worker.
//
// The page-table build is an ordered stream compaction over the pool's page
// addresses.  For most XOR hashes the rank of a run of pages is a product,
// and one launch places every page; other hashes and colour tables take a
// counting and an emitting pass.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "host_common.hpp"

namespace sgdrc {

struct HashArgs {
    uint32_t lo[SGDRC_MAX_MASKS];  // mask bits 0..31
    uint32_t hi[SGDRC_MAX_MASKS];  // mask bits 32..47
};

struct SetArgs {
    uint32_t w[8];  // 256-bit colour set
};

template <int K>
__device__ __forceinline__ uint32_t colour_of(uint32_t lo, uint32_t hi, const HashArgs &h)
{
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint32_t ones = __builtin_popcount(lo & h.lo[k]) + __builtin_popcount(hi & h.hi[k]);
        c |= (ones & 1u) << k;
    }
    return c;
}

// The hash is linear over GF(2): colour(a ^ b) = colour(a) ^ colour(b).  So
// the colour of an address is the XOR of the colours of its six bytes in
// place, colour(byte_t << 8t), each read from a 256-entry table.  A table
// is 64 LDS dwords, so a wavefront's lookups into one table conflict at most
// two ways on a bank (none with 64 banks), without replicated copies.  Six
// lookups and about ten integer ops replace the popcount form's 6 K.
constexpr int kLutBytes = 6;  // address bits 0..47

__device__ __forceinline__ uint32_t colour_lut(const uint8_t (*lut)[256], uint32_t lo, uint32_t hi)
{
    return (uint32_t)lut[0][lo & 0xffu] ^ (uint32_t)lut[1][(lo >> 8) & 0xffu] ^
           (uint32_t)lut[2][(lo >> 16) & 0xffu] ^ (uint32_t)lut[3][lo >> 24] ^
           (uint32_t)lut[4][hi & 0xffu] ^ (uint32_t)lut[5][(hi >> 8) & 0xffu];
}

// The table form of the hash (paper section 5.3): one colour byte per
// 2^shift-byte partition from ``origin``; 255 = no colour (also outside).
struct TableArgs {
    const uint8_t *lut;
    uint64_t origin;
    uint64_t entries;
    uint32_t shift;
};

// (An address outside the table reads entry 0 and ignores it, so that no
// branch separates a lane's gathers and all of them are in flight at once;
// the host gives an empty table one readable byte.)
__device__ __forceinline__ uint32_t table_colour(const TableArgs &t, uint64_t a)
{
    const uint64_t i = (a - t.origin) >> t.shift;
    const bool in = a >= t.origin && i < t.entries;
    const uint32_t c = t.lut[in ? i : 0u];
    return in ? c : 255u;
}

constexpr int kClsThreads = 256;
constexpr int kClsLoads = 8;                             // 16-byte loads per lane per tile
// addresses per wavefront tile: 1024 (4096 with kPhasedLoads)
constexpr uint32_t cls_wave_tile(int loads) { return 64u * 2u * (uint32_t)loads; }
constexpr uint32_t kClsWaves = kClsThreads / 64;
// Each wavefront takes its own tiles of addresses; under a mask
// of whole XCDs by the static schedule, otherwise through work queues of 8
// CUs (one device-wide counter serialises its atomics at about 12 ns each).
constexpr int kClsGroupCus = 8;
// Two workgroups per CU with eight loads per lane: 2^26 addresses in
// 95-96 us (static) or 100 us (queues) on MI355X, against 105-125 us for one
// workgroup with 16 or 32 loads, or three with 8.
constexpr int kClsWgsPerCu = 2;
constexpr int kClsHistWgsPerCu = 2;
// Colour tables: six workgroups per CU, whose gathers hide each other's
// round trips when the table sits in the caches (2^24 addresses, 1024
// entries: 30 us against 35 with two); above that the gathers' cache lines
// bound the kernel and the number makes no difference.
constexpr int kClsTableWgsPerCu = 6;

// Colour tables larger than an XCD's 4 MiB L2: the gathers of a plain pass
// miss it, and every miss moves a 128-byte line for one byte (2^24 addresses
// in a 16 MiB table: 13.7 M lines, 7.5 TB/s, 235 us however many wavefronts
// are in flight).  So each wavefront holds 4096 addresses as table indices in
// registers and gathers them one 2 MiB slice of the table after the other:
// the wavefronts of an XCD start together and keep step (one that runs ahead
// waits for the misses that those behind it then hit), so a slice's lines
// are fetched about once per XCD while all of them use it.  2^24 addresses on
// MI355X, plain / by slices: 8 MiB table 164 / 99 us, 16 MiB 232 / 119, 64
// MiB 307 / 200; with 1024 addresses per wavefront 182 us for 16 MiB, with
// 1 MiB slices 127 us; a 4 MiB table 91 / 94 us.  Two workgroups per CU: three,
// which fit without a histogram, keep step less well (16 MiB 125 us, 32 MiB 166
// against 154).
//
// That is for addresses in any order.  Where neighbouring ones lie in one line of
// the table (ascending addresses, runs of a page's lines), there is little to
// miss and a pass over the slices only costs time, so a wavefront looks at two
// of its lanes' indices and then gathers all of them plainly.  2^24 addresses in
// steps of one partition, plain kernel / every slice / now: 8 MiB table 34.6 /
// 39.9 / 29.0 us, 16 MiB 39.8 / 51.1 / 30.1, 64 MiB 39.5 / 114 / 29.9.
constexpr int kPhasedLoads = 32;
constexpr uint32_t kPhasedGroup = 16;  // gathers in flight per lane
constexpr uint32_t kSliceShift = 21;
constexpr int kPhasedWgsPerCu = 2;

// Histogram bins are replicated 16 times in LDS (copy = lane mod 16,
// bin-major), so that lanes of a wavefront seldom add to one address.  More
// copies cost more to clear and to sum than they save: 16 / 64 copies (one per
// lane) on MI355X, 65536 addresses, K = 4 6.6 / 7.2 us, K = 6 7.0 / 8.0, K = 8
// 7.7 / 12.5; 2^26 addresses, K = 4 102.4 / 103.7 us, K = 6 102.9 / 102.4, K = 8
// 101.5 / 112.1, a 64 KiB colour table (2^24 addresses) 59 / 65.
constexpr int kHistCopies = 16;

// hist_out[b] = the sum of bin b over the kHistAccCopies accumulator copies,
// which are cleared for the next launch (every thread of one workgroup).
template <uint32_t kBins>
__device__ __forceinline__ void publish_histogram(uint64_t *hist_acc, uint64_t *hist_out)
{
    for (uint32_t b = threadIdx.x; b < kBins; b += blockDim.x) {
        uint64_t v = 0;
#pragma unroll
        for (int r = 0; r < kHistAccCopies; ++r) {
            v += __hip_atomic_load(&hist_acc[r * kHistBins + b], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&hist_acc[r * kHistBins + b], (uint64_t)0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        hist_out[b] = v;
    }
}

// The table's colours of a tile's addresses, slice by slice (kSliceShift);
// ``c`` in: table indices, or 0xFFFFFFFF for an address outside the table;
// out: colours.  A lane whose index lies in another slice takes an offset past
// the buffer resource, for which the hardware makes no access.  A finished
// index is replaced by its colour with the upper bits set, which no slice
// matches (the host keeps tables below 2^31 entries here).  Only the slices from
// the wavefront's lowest index to its highest are gathered.
template <int N>
__device__ __forceinline__ void gather_slices(const TableArgs &t, uint32_t (&c)[N])
{
    const Rsrc r = make_rsrc(t.lut, (uint32_t)t.entries);
    // (as a signed number 0xFFFFFFFF is below every index)
    uint32_t first = c[0];
    int32_t last = (int32_t)c[0];
#pragma unroll
    for (int j = 1; j < N; ++j) {
        first = min(first, c[j]);
        last = max(last, (int32_t)c[j]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        first = min(first, (uint32_t)__shfl_xor((int)first, off, 64));
        last = max(last, __shfl_xor(last, off, 64));
    }
    const uint32_t q0 = (uint32_t)__builtin_amdgcn_readfirstlane(first) >> kSliceShift;
    const int32_t q1 = __builtin_amdgcn_readfirstlane(last) >> kSliceShift;
    for (uint32_t q = q0; (int32_t)q <= q1; ++q) {  // (no index: 2047 and -1)
#pragma unroll
        for (int g = 0; g < N; g += (int)kPhasedGroup) {
            uint32_t v[kPhasedGroup];
#pragma unroll
            for (int j = 0; j < (int)kPhasedGroup; ++j)
                v[j] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(
                    r, (c[g + j] >> kSliceShift) == q ? c[g + j] : 0xFFFFFFFFu, 0, 0);
#pragma unroll
            for (int j = 0; j < (int)kPhasedGroup; ++j)
                c[g + j] = (c[g + j] >> kSliceShift) == q ? 0xFFFFFF00u | v[j] : c[g + j];
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
        c[j] &= 0xFFu;
}

// The same in one pass.
template <int N>
__device__ __forceinline__ void gather_plain(const TableArgs &t, uint32_t (&c)[N])
{
    const Rsrc r = make_rsrc(t.lut, (uint32_t)t.entries);
#pragma unroll
    for (int g = 0; g < N; g += (int)kPhasedGroup) {
        uint32_t v[kPhasedGroup];
#pragma unroll
        for (int j = 0; j < (int)kPhasedGroup; ++j)
            v[j] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, c[g + j], 0, 0);
#pragma unroll
        for (int j = 0; j < (int)kPhasedGroup; ++j)
            c[g + j] = c[g + j] == 0xFFFFFFFFu ? 255u : v[j];
    }
}

// Whether neighbouring lanes' indices mostly lie in one 128-byte line, by two of
// the lane's indices: a plain gather then fetches few lines, however large the
// table.
__device__ __forceinline__ bool gathers_share_lines(uint32_t c0, uint32_t c1)
{
    const uint32_t p0 = __shfl_xor(c0, 1, 64), p1 = __shfl_xor(c1, 1, 64);
    return __popcll(__ballot(c0 >> 7 == p0 >> 7)) + __popcll(__ballot(c1 >> 7 == p1 >> 7)) >= 64;
}

// Where colours come from: the XOR hash, or a colour table in device memory
// (one gathered byte per address; K is then 8, 256 bins), gathered at once
// or slice by slice.
enum class ClsFrom { Hash, Table, Slices };

template <int K, bool HIST, ClsFrom FROM, int LOADS>
__device__ __forceinline__ void classify(const uint64_t *__restrict__ addrs, uint64_t n,
                                         uint8_t *__restrict__ colours, const HashArgs &h,
                                         const TableArgs &tab, uint64_t *hist_acc,
                                         uint64_t *hist_out, uint32_t n_tiles, const Gate &g)
{
    constexpr bool TAB = FROM != ClsFrom::Hash;
    constexpr uint32_t kBins = 1u << K;
    constexpr uint32_t kTile = cls_wave_tile(LOADS);
    constexpr int kCopies = kHistCopies;
    __shared__ uint32_t s_hist[HIST ? kBins * kCopies : 1];
    // per wavefront: the colour bytes of one tile, 2 per lane and load
    __shared__ __attribute__((aligned(16))) uint16_t s_col[kClsThreads / 64][kTile / 2];
    __shared__ __attribute__((aligned(16))) uint8_t s_lut[kLutBytes][256];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t copy = lane % kCopies;
    const uint64_t n16 = n & ~15ull;
    if (HIST) {
        for (uint32_t i = threadIdx.x; i < kBins * kCopies; i += kClsThreads)
            s_hist[i] = 0;
        __syncthreads();
    }
    auto body = [&](uint32_t t, uint32_t, uint32_t &, auto &&claim) {
        // a tile is one wavefront's: its first address, and how many of its
        // addresses lie below n16 (a multiple of 16, possibly 0)
        const uint64_t base = (uint64_t)t * kTile;
        const uint32_t valid = n16 > base ? (uint32_t)(n16 - base < kTile ? n16 - base : kTile) : 0u;
        const Rsrc ra = make_rsrc(addrs + base, valid * 8u);
        u32x4 v[LOADS];
#pragma unroll
        for (int j = 0; j < LOADS; ++j)
            v[j] = buf_load_nt(ra, (j * 64u + lane) * 16u);
        claim();
        auto addr = [&](int j) __attribute__((always_inline)) {
            const u32x4 &w = v[j / 2];
            return j & 1 ? ((uint64_t)w.w << 32) | w.z : ((uint64_t)w.y << 32) | w.x;
        };
        // the 1024 addresses of loads 8 q .. 8 q + 7, address j of a lane with
        // colour(j), to LDS and the histogram
        auto put = [&](int q, auto &&colour) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t c0 = colour(2 * j);
                const uint32_t c1 = colour(2 * j + 1);
                const uint32_t at = (uint32_t)(8 * q + j) * 64u + lane;
                s_col[wave][at] = (uint16_t)(c0 | (c1 << 8));
                // both addresses of the load are valid or neither (valid is even);
                // invalid ones (read as address 0, a bin in range) add 0, so
                // that no branch splits the lanes around the atomics (with one,
                // the histogram cost several microseconds more)
                if (HIST) {
                    const uint32_t inc = 2u * at < valid ? 1u : 0u;
                    atomicAdd(&s_hist[c0 * kCopies + copy], inc);
                    atomicAdd(&s_hist[c1 * kCopies + copy], inc);
                }
            }
        };
        // and the colours of N such groups to memory
        auto store = [&](auto count) __attribute__((always_inline)) {
            constexpr int N = decltype(count)::value;
            // LDS accesses of one wavefront complete in order; the wave
            // barriers only keep the compiler from moving these accesses
            __builtin_amdgcn_wave_barrier();
            u32x4 out[N];
#pragma unroll
            for (int i = 0; i < N; ++i)
                out[i] = *reinterpret_cast<const u32x4 *>(&s_col[wave][i * 512u + lane * 8u]);
            __builtin_amdgcn_wave_barrier();
            const Rsrc rc = make_rsrc(colours + base, valid);
#pragma unroll
            for (int i = 0; i < N; ++i)
                buf_store_sc1(rc, i * 1024u + lane * 16u, out[i]);
        };
        using One = std::integral_constant<int, 1>;
        if constexpr (FROM == ClsFrom::Hash) {
            put(0, [&](int j) __attribute__((always_inline)) {
                return j & 1 ? colour_lut(s_lut, v[j / 2].z, v[j / 2].w) : colour_lut(s_lut, v[j / 2].x, v[j / 2].y);
            });
            store(One());
        } else if constexpr (FROM == ClsFrom::Table) {
            uint32_t c[16];
#pragma unroll
            for (int j = 0; j < 16; ++j)
                c[j] = table_colour(tab, addr(j));
            put(0, [&](int j) __attribute__((always_inline)) { return c[j]; });
            store(One());
        } else {
            uint32_t c[2 * LOADS];
#pragma unroll
            for (int j = 0; j < 2 * LOADS; ++j) {
                const uint64_t a = addr(j), i = (a - tab.origin) >> tab.shift;
                c[j] = a >= tab.origin && i < tab.entries ? (uint32_t)i : 0xFFFFFFFFu;
            }
            if (gathers_share_lines(c[0], c[9]))
                gather_plain<2 * LOADS>(tab, c);
            else
                gather_slices<2 * LOADS>(tab, c);
#pragma unroll
            for (int q = 0; q < LOADS / 8; ++q)
                put(q, [&](int j) __attribute__((always_inline)) { return c[16 * q + j]; });
            store(std::integral_constant<int, LOADS / 8>());
        }
    };
    auto flush = [&]() {
        if (HIST) {
            uint32_t xcc;
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
            uint64_t *acc = hist_acc + (xcc % (uint32_t)kHistAccCopies) * kHistBins;
            __syncthreads();
            for (uint32_t b = threadIdx.x; b < kBins; b += kClsThreads) {
                uint32_t v = 0;
#pragma unroll
                for (int r = 0; r < kCopies; ++r) {
                    v += s_hist[b * kCopies + r];
                    s_hist[b * kCopies + r] = 0;
                }
                if (v)
                    __hip_atomic_fetch_add(&acc[b], (uint64_t)v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    };
    // colour the last n mod 16 addresses, then, in the last workgroup with
    // every other workgroup's histogram in hist_acc, publish the counts
    auto epilogue = [&]() {
        const uint64_t i = n16 + threadIdx.x;
        if (i < n) {
            const uint64_t a = addrs[i];
            const uint32_t c = TAB ? table_colour(tab, a)
                                   : colour_of<K>((uint32_t)a, (uint32_t)(a >> 32), h);
            colours[i] = (uint8_t)c;
            if (HIST)
                __hip_atomic_fetch_add(&hist_acc[c], (uint64_t)1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        if (HIST) {
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            publish_histogram<kBins>(hist_acc, hist_out);
        }
    };
    // the byte tables, visible to the whole workgroup after the loop's
    // opening barrier
    auto prologue = [&]() {
        if (TAB)
            return;
#pragma unroll
        for (int r = 0; r < kLutBytes * 256 / kClsThreads; ++r) {
            const uint32_t i = (uint32_t)r * kClsThreads + threadIdx.x;
            const uint32_t t = i >> 8, e = i & 0xffu;
            const uint64_t a = (uint64_t)e << (8u * t);
            s_lut[t][e] = (uint8_t)colour_of<K>((uint32_t)a, (uint32_t)(a >> 32), h);
        }
    };
    if (g.statics)
        static_wave_loop<HIST>(g, n_tiles, prologue, body, flush, epilogue);
    else
        gated_wave_loop(g, n_tiles, prologue, body, flush, epilogue);
}

template <int K, bool HIST, bool TAB>
__global__ __launch_bounds__(kClsThreads) void k_classify(const uint64_t *__restrict__ addrs,
                                                          uint64_t n, uint8_t *__restrict__ colours,
                                                          HashArgs h, TableArgs tab,
                                                          uint64_t *hist_acc, uint64_t *hist_out,
                                                          uint32_t n_tiles, Gate g)
{
    classify<K, HIST, TAB ? ClsFrom::Table : ClsFrom::Hash, kClsLoads>(addrs, n, colours, h, tab,
                                                                       hist_acc, hist_out, n_tiles, g);
}

// (without a histogram the compiler is told of the two wavefronts per SIMD: it
// then keeps all of a slice's gathers in flight, 2^24 addresses in order through a
// 16 MiB table 30.1 against 33.4 us; with one the default is better, at random
// 119.9 against 122.6 us)
template <bool HIST>
__global__ __launch_bounds__(kClsThreads, HIST ? 0 : 2) void k_classify_slices(const uint64_t *__restrict__ addrs,
                                                                 uint64_t n,
                                                                 uint8_t *__restrict__ colours,
                                                                 HashArgs h, TableArgs tab,
                                                                 uint64_t *hist_acc,
                                                                 uint64_t *hist_out,
                                                                 uint32_t n_tiles, Gate g)
{
    classify<8, HIST, ClsFrom::Slices, kPhasedLoads>(addrs, n, colours, h, tab, hist_acc, hist_out,
                                                     n_tiles, g);
}

// ------------------------------------------------- page-table build
//
// Both builds below place each qualifying page by its rank: the number of
// qualifying pages before its workgroup's pages, plus its rank inside the
// workgroup from wavefront ballots and masked bit counts, so the table comes
// out in ascending page order whatever the scheduling.
constexpr int kPtThreads = 256;
constexpr uint32_t kPtWaves = kPtThreads / 64;

// The rank of this thread's first qualifying page among the workgroup's
// pages, for threads whose ``V`` consecutive pages qualify by the bits of
// ``m``; ``sum`` becomes the workgroup's count.  One barrier; s_wave is free
// again after the caller's next one.
template <int V>
__device__ __forceinline__ uint32_t pt_rank(uint32_t m, uint32_t *s_wave, uint32_t &sum)
{
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    uint32_t below = 0u, mine = 0u;
    if (V <= 4) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const uint64_t bal = __ballot((m >> k) & 1u);
            below = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)bal, below));
            mine += (uint32_t)__popcll(bal);
        }
    } else {
        // the counts (at most 16) by their bits
        const uint32_t c = (uint32_t)__popc(m);
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const uint64_t bal = __ballot((c >> k) & 1u);
            below += __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                               __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u)) << k;
            mine += (uint32_t)__popcll(bal) << k;
        }
    }
    if (lane == 0)
        s_wave[wave] = mine;
    __syncthreads();
    uint32_t before = 0u;
    sum = 0u;
#pragma unroll
    for (uint32_t w = 0; w < kPtWaves; ++w) {
        const uint32_t cw = s_wave[w];
        before += w < wave ? cw : 0u;
        sum += cw;
    }
    return before + below;
}

// XOR hashes, one launch.  The colour of page number q (address >> shift) is
// linear over GF(2) in q, so when every aligned run of 2^m pages holds the
// same number ``per_run`` of qualifying pages (the host checks it, see
// plan_runs), the rank of a run's first page is a product and no counting
// pass is needed.  Workgroup w takes run w of 2^m = 1024 R pages counted
// from the run that holds the pool's first page ``q0``; ``skip`` is the
// number of qualifying pages of that first run before q0, and ``total`` the
// qualifying pages of the pool (both from the host).  Each thread takes four
// consecutive pages of an aligned group, whose colours differ from the first
// one's by the constants v0 and v1.
//
// Bound by the launch and one chain of dependent steps (no data is read).
// 409600 pages, 8 of 64 colours, 49152 entries, on MI355X: 3.2 us, and 20.0
// us for the synchronous call, against 6.1 + 4.6 + 7.6 us for a counting, a
// scanning and an emitting launch, and 35.3 us with them and a copy of the
// count.  2^26 pages, 2^22 entries: call 44 against 247 us.
template <int K>
__global__ __launch_bounds__(kPtThreads) void k_pt_runs(HashArgs h, uint64_t q0, uint32_t shift,
                                                        uint64_t pool_pages, SetArgs set, uint32_t R,
                                                        uint32_t per_run, uint32_t skip,
                                                        uint32_t v0, uint32_t v1, uint32_t *pt,
                                                        uint64_t n_needed, uint64_t total,
                                                        uint64_t *d_total)
{
    __shared__ uint32_t s_set[8];
    __shared__ uint32_t s_wave[kPtWaves];
    if (d_total && blockIdx.x == 0 && threadIdx.x == 0)
        *d_total = total;
    if (n_needed == 0)
        return;
    if (threadIdx.x < 8)
        s_set[threadIdx.x] = set.w[threadIdx.x];
    __syncthreads();
    const uint64_t run = 1024ull * R;
    const uint64_t first = (q0 / run + blockIdx.x) * run;
    uint64_t running = (uint64_t)blockIdx.x * per_run;
    for (uint32_t r = 0; r < R; ++r) {
        const uint64_t q = first + r * 1024u + threadIdx.x * 4u;
        const uint64_t a = q << shift;
        const uint32_t c = colour_of<K>((uint32_t)a, (uint32_t)(a >> 32), h);
        uint32_t m = 0u;
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t ck = c ^ (k & 1u ? v0 : 0u) ^ (k & 2u ? v1 : 0u);
            m |= ((s_set[ck >> 5] >> (ck & 31u)) & 1u) << k;
        }
        uint32_t sum;
        uint64_t rank = running + pt_rank<4>(m, s_wave, sum);
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            if ((m >> k) & 1u) {
                // pages before q0 (only in the first run) and past the pool
                // are counted in the ranks and not written
                const uint64_t page = q + k - q0;
                if (page < pool_pages && rank - skip < n_needed)
                    pt[rank - skip] = (uint32_t)page;
                ++rank;
            }
        }
        running += sum;
        __syncthreads();
    }
}

// Any other page test, two launches: the counting pass writes the number of
// qualifying pages of each workgroup's chunk, the emitting pass sums the
// counts before its own and places its pages.  At most kPtMaxChunks
// workgroups, so that the sum is a few loads per thread and needs no scan
// launch between the two.  Each thread tests up to Q::kPages consecutive pages
// at a time; the emitting pass collects a round's entries in LDS and stores them in
// order, and ends once the table is full.
//
// 2^24 1 KiB pages tested through a colour table of as many partitions, a
// quarter of them qualifying, 2^20 entries, on MI355X: 5.8 + 6.7 us, against
// 29.6 + 9.0 + 30.0 us with one byte load per page and 16 barriers per
// workgroup and a scan in between.  2^25 pages of two partitions: call 62
// against 200 us; 2^20 pages of 64 partitions 46 against 381 us.  2048
// chunks keep every wavefront slot of the chip filled (1024: 2^26 pages 68
// against 55 us).
constexpr uint32_t kPtMaxChunks = 2048;

// QXor: the colour of the page's base address is in the set given to the
// kernel, which the host has narrowed to the colours whose whole page lies in
// the caller's set (see page_colour_set).
template <int K>
struct QXor {
    static constexpr int kPages = 4;
    HashArgs h;
    __device__ uint32_t pages() const { return kPages; }
    __device__ uint32_t operator()(uint64_t a, uint32_t page_shift, uint64_t, const uint32_t *s_set) const
    {
        uint32_t m = 0u;
#pragma unroll
        for (int k = 0; k < kPages; ++k) {
            const uint64_t ak = a + ((uint64_t)k << page_shift);
            const uint32_t c = colour_of<K>((uint32_t)ak, (uint32_t)(ak >> 32), h);
            m |= ((s_set[c >> 5] >> (c & 31u)) & 1u) << k;
        }
        return m;
    }
};

// QTable: every partition that the page touches is in the table and has a
// colour in the set.  ALIGNED: a page is 2^log_parts <= 16 whole partitions,
// so that a thread reads the colours of 16 partitions with one load (any
// alignment) where all of them lie in the table; otherwise a thread tests one
// page at a time.
template <bool ALIGNED>
struct QTable {
    static constexpr int kPages = ALIGNED ? 16 : 1;
    TableArgs t;
    uint32_t log_parts;
    __device__ uint32_t pages() const { return ALIGNED ? 16u >> log_parts : 1u; }
    // bits of the 16 partitions from j on whose colours are in the set
    // (255 is never in it)
    __device__ __forceinline__ uint32_t has16(uint64_t j, const uint32_t *s_set) const
    {
        u32x4 v;
        __builtin_memcpy(&v, t.lut + j, sizeof v);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t m = 0u;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t c = (w[k >> 2] >> (8 * (k & 3))) & 0xffu;
            m |= ((s_set[c >> 5] >> (c & 31u)) & 1u) << k;
        }
        return m;
    }
    __device__ bool one(uint64_t a, uint32_t page_shift, const uint32_t *s_set) const
    {
        if (a < t.origin)
            return false;
        uint64_t j = (a - t.origin) >> t.shift;
        const uint64_t j1 = (a + (1ull << page_shift) - 1u - t.origin) >> t.shift;
        if (j1 >= t.entries)
            return false;
        bool ok = true;
        for (; ok && j1 - j >= 15u && j <= j1; j += 16u)
            ok = has16(j, s_set) == 0xffffu;
        for (; ok && j <= j1; ++j) {
            const uint32_t c = t.lut[j];
            ok = ((s_set[c >> 5] >> (c & 31u)) & 1u) != 0u;
        }
        return ok;
    }
    // the first ``n`` (at most pages()) of the pages from address a on
    __device__ uint32_t operator()(uint64_t a, uint32_t page_shift, uint64_t n, const uint32_t *s_set) const
    {
        const uint64_t j = (a - t.origin) >> t.shift;
        if (ALIGNED && a >= t.origin && t.entries >= 16u && j <= t.entries - 16u) {
            uint32_t m = has16(j, s_set);
            if (log_parts == 0u)
                return m;
            for (uint32_t d = 1u; d < 1u << log_parts; d <<= 1)
                m &= m >> d;
            uint32_t out = 0u;
            for (uint32_t k = 0; k < 16u >> log_parts; ++k)
                out |= ((m >> (k << log_parts)) & 1u) << k;
            return out;
        }
        uint32_t m = 0u;
        for (uint32_t k = 0; k < pages() && k < n; ++k)
            m |= (one(a + ((uint64_t)k << page_shift), page_shift, s_set) ? 1u : 0u) << k;
        return m;
    }
};

// Bits of the qualifying ones of this thread's pages [page, page + qual.pages()).
template <class Q>
__device__ __forceinline__ uint32_t pt_test(const Q &qual, uint64_t origin, uint32_t shift,
                                            uint64_t page, uint64_t end, const uint32_t *s_set)
{
    if (page >= end)
        return 0u;
    const uint64_t n = end - page;
    const uint32_t m = qual(origin + (page << shift), shift, n, s_set);
    return n < (uint64_t)qual.pages() ? m & ((1u << n) - 1u) : m;
}

template <class Q>
__global__ __launch_bounds__(kPtThreads) void k_pt_count(Q qual, uint64_t origin, uint32_t shift,
                                                         uint64_t pool_pages, uint64_t chunk,
                                                         SetArgs set, uint32_t *counts)
{
    __shared__ uint32_t s_set[8];
    __shared__ uint32_t s_count[kPtWaves];
    if (threadIdx.x < 8)
        s_set[threadIdx.x] = set.w[threadIdx.x];
    __syncthreads();
    const uint64_t lo = (uint64_t)blockIdx.x * chunk;
    const uint64_t end = pool_pages - lo < chunk ? pool_pages : lo + chunk;
    uint32_t c = 0u;
    const uint32_t each = qual.pages();
    for (uint64_t p = lo + threadIdx.x * each; p < end; p += kPtThreads * each)
        c += (uint32_t)__popc(pt_test(qual, origin, shift, p, end, s_set));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        c += __shfl_xor(c, off, 64);
    if ((threadIdx.x & 63u) == 0u)
        s_count[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t v = 0u;
#pragma unroll
        for (uint32_t w = 0; w < kPtWaves; ++w)
            v += s_count[w];
        counts[blockIdx.x] = v;
    }
}

// ``total`` (device or pinned host memory) receives the pool's count.
template <class Q>
__global__ __launch_bounds__(kPtThreads) void k_pt_emit(Q qual, uint64_t origin, uint32_t shift,
                                                        uint64_t pool_pages, uint64_t chunk,
                                                        SetArgs set, const uint32_t *counts,
                                                        uint32_t n_chunks, uint32_t *pt,
                                                        uint64_t n_needed, uint64_t *total)
{
    __shared__ uint32_t s_set[8];
    __shared__ uint32_t s_wave[kPtWaves];
    __shared__ uint64_t s_sum[2][kPtWaves];
    __shared__ uint32_t s_out[kPtThreads * Q::kPages];
    if (threadIdx.x < 8)
        s_set[threadIdx.x] = set.w[threadIdx.x];
    uint64_t before = 0u, all = 0u;
#pragma unroll
    for (uint32_t r = 0; r < kPtMaxChunks / kPtThreads; ++r) {
        const uint32_t i = r * kPtThreads + threadIdx.x;
        const uint32_t v = i < n_chunks ? counts[i] : 0u;
        before += i < blockIdx.x ? v : 0u;
        all += v;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        before += __shfl_xor(before, off, 64);
        all += __shfl_xor(all, off, 64);
    }
    if ((threadIdx.x & 63u) == 0u) {
        s_sum[0][threadIdx.x >> 6] = before;
        s_sum[1][threadIdx.x >> 6] = all;
    }
    __syncthreads();
    uint64_t running = 0u;
    all = 0u;
#pragma unroll
    for (uint32_t w = 0; w < kPtWaves; ++w) {
        running += s_sum[0][w];
        all += s_sum[1][w];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *total = all;
    const uint64_t lo = (uint64_t)blockIdx.x * chunk;
    const uint64_t end = pool_pages - lo < chunk ? pool_pages : lo + chunk;
    const uint32_t each = qual.pages();
    for (uint64_t base = lo; base < end && running < n_needed; base += kPtThreads * each) {
        const uint64_t p = base + threadIdx.x * each;
        const uint32_t m = pt_test(qual, origin, shift, p, end, s_set);
        uint32_t sum;
        uint32_t rank = pt_rank<Q::kPages>(m, s_wave, sum);
#pragma unroll
        for (int k = 0; k < Q::kPages; ++k)
            if ((m >> k) & 1u)
                s_out[rank++] = (uint32_t)(p + k);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < sum; i += kPtThreads)
            if (running + i < n_needed)
                pt[running + i] = s_out[i];
        running += sum;
        __syncthreads();
    }
}

static HashArgs hash_args(const sgdrc_hash *h)
{
    HashArgs a;
    std::memset(&a, 0, sizeof a);
    for (uint32_t k = 0; k < h->n_masks; ++k) {
        a.lo[k] = (uint32_t)h->masks[k];
        a.hi[k] = (uint32_t)(h->masks[k] >> 32);
    }
    return a;
}

// Whether a table is gathered slice by slice: larger than an XCD's L2 by half
// (5 MiB, plain / by slices: 3 x 2^21 addresses 42.3 / 44.8 us; 6 MiB 48.3 / 46.7), few
// enough slices (each costs the wavefronts an instruction per index; measured
// up to 32), and enough addresses that a line fetched by an XCD is used
// several times (n / 8 addresses per XCD against entries / 128 lines) and all
// wavefronts have a tile.  Plain / by slices on MI355X: 2^22 addresses, 8 MiB
// 43 / 28 us, 16 MiB 60 / 35; 2^21 addresses, 8 MiB 25 / 31 us.
static bool gather_by_slices(const TableArgs &t, uint64_t n)
{
    return t.entries >= (3ull << kSliceShift) && t.entries <= (32ull << kSliceShift) &&
           n >= t.entries / 4u && n >= (1ull << 22);
}

typedef void (*ClassifyKernel)(const uint64_t *, uint64_t, uint8_t *, HashArgs, TableArgs,
                               uint64_t *, uint64_t *, uint32_t, Gate);

template <int K, bool TAB>
static int launch_classify(Ctx *c, const HashArgs &h, const TableArgs &tab,
                           const uint64_t *d_addrs, uint64_t n, uint8_t *d_colours,
                           uint64_t *d_hist, void *stream)
{
    const bool slices = TAB && gather_by_slices(tab, n);
    const uint32_t tile = cls_wave_tile(slices ? kPhasedLoads : kClsLoads);
    const uint64_t n_tiles = ((n & ~15ull) + tile - 1) / tile;
    // (the bound of 1024-address tiles, whatever the tile)
    const uint32_t small = cls_wave_tile(kClsLoads);
    if (((n & ~15ull) + small - 1) / small >= (1ull << 31))
        return set_error(SGDRC_EINVAL, "n too large");
    // grid sizing counts workgroups' worth of tiles
    const uint64_t wg_tiles = (n_tiles + kClsWaves - 1) / kClsWaves;
    Gate g;
    LaunchInfo li;
    int rc = make_gate(c, stream, n_tiles, kClsGroupCus, &g, &li, false, true);
    if (rc)
        return rc;
    uint64_t *acc = c->d_hist_acc + (size_t)(g.q - c->d_queues) * kHistAccCopies * kHistBins;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    ClassifyKernel k = d_hist ? k_classify<K, true, TAB> : k_classify<K, false, TAB>;
    int per_cu = d_hist ? kClsHistWgsPerCu : kClsWgsPerCu;
    if constexpr (TAB) {
        static const int occ[2][2] = {{occupancy(k_classify<K, false, true>, kClsThreads),
                                       occupancy(k_classify<K, true, true>, kClsThreads)},
                                      {occupancy(k_classify_slices<false>, kClsThreads),
                                       occupancy(k_classify_slices<true>, kClsThreads)}};
        if (slices)
            k = d_hist ? k_classify_slices<true> : k_classify_slices<false>;
        per_cu = std::min(occ[slices][d_hist != nullptr], slices ? kPhasedWgsPerCu : kClsTableWgsPerCu);
    } else {
        static const int occ[2] = {occupancy(k_classify<K, false, false>, kClsThreads),
                                   occupancy(k_classify<K, true, false>, kClsThreads)};
        per_cu = std::min(occ[d_hist != nullptr], per_cu);
    }
    const uint32_t grid = gated_grid(c, per_cu, wg_tiles, li);
    // the histogram's publication falls to the last workgroup (for 65536
    // addresses the call takes 7.2 us against 9.5 with a kernel that follows
    // the grid, for 2^26 the same)
    hipLaunchKernelGGL(k, dim3(grid), dim3(kClsThreads), 0, s, d_addrs, n, d_colours, h, tab, acc,
                       d_hist, (uint32_t)n_tiles, g);
    SGDRC_HIP(hipGetLastError());
    return finish_static_tlog(g, s);
}

template <int K>
static int launch_classify_xor(Ctx *c, const HashArgs &h, const uint64_t *d_addrs, uint64_t n,
                               uint8_t *d_colours, uint64_t *d_hist, void *stream)
{
    return launch_classify<K, false>(c, h, TableArgs{}, d_addrs, n, d_colours, d_hist, stream);
}

// The set of base-address colours whose pages lie wholly in ``set``.  A
// page holds every address base + o, o < 2^page_shift, and the hash is
// linear over GF(2), so its bytes have exactly the colours c ^ l, with c the
// colour of its base and l running over L, the colours of the in-page
// offsets: the span of colour(1 << b) for b < page_shift.  (Paper section 6
// colours whole sectors, whose bytes share their channels.)  The page
// qualifies when that coset lies in the set.  With no mask bit below
// page_shift, L = {0} and the set is unchanged.
static sgdrc_colour_set page_colour_set(const sgdrc_hash *h, uint32_t page_shift,
                                        const sgdrc_colour_set &set)
{
    const uint32_t n = 1u << h->n_masks;
    bool in_l[256] = {};
    in_l[0] = true;
    for (uint32_t b = 0; b < page_shift && b < 48u; ++b) {
        uint32_t v = 0;
        for (uint32_t k = 0; k < h->n_masks; ++k)
            v |= (uint32_t)((h->masks[k] >> b) & 1ull) << k;
        if (in_l[v])
            continue;
        bool grown[256];
        for (uint32_t c = 0; c < n; ++c)
            grown[c] = in_l[c] || in_l[c ^ v];
        for (uint32_t c = 0; c < n; ++c)
            in_l[c] = grown[c];
    }
    auto member = [&](uint32_t c) { return ((set.bits[c >> 6] >> (c & 63u)) & 1ull) != 0ull; };
    sgdrc_colour_set out{};
    for (uint32_t c = 0; c < n; ++c) {
        bool all = true;
        for (uint32_t l = 0; l < n && all; ++l)
            all = !in_l[l] || member(c ^ l);
        if (all)
            out.bits[c >> 6] |= 1ull << (c & 63u);
    }
    return out;
}

static std::mutex g_pt_mu;  // general builds share a context's scratch: serialised

static int check_pool_args(uint64_t addr_origin, uint32_t page_shift, uint64_t pool_pages,
                           const sgdrc_colour_set *set, uint64_t n_needed, uint32_t *d_pt,
                           uint64_t *n_found)
{
    int rc = check_shift(page_shift);
    if (rc)
        return rc;
    if (!set || !n_found)
        return set_error(SGDRC_EINVAL, "NULL colour set or n_found");
    if (addr_origin & ((1ull << page_shift) - 1ull))
        return set_error(SGDRC_EINVAL, "addr_origin not aligned to the page size");
    if (pool_pages == 0 || pool_pages > (1ull << 32))
        return set_error(SGDRC_EINVAL, "pool_pages must be in 1..2^32");
    if (addr_origin >= (1ull << 48) || pool_pages > (((1ull << 48) - addr_origin) >> page_shift))
        return set_error(SGDRC_EINVAL, "pool extends beyond the 48-bit address space");
    if (n_needed > pool_pages)
        return set_error(SGDRC_EINVAL, "n_needed exceeds pool_pages");
    if (n_needed > 0 && (!d_pt || (reinterpret_cast<uintptr_t>(d_pt) & 3u)))
        return set_error(SGDRC_EINVAL, "page table pointer NULL or not 4-byte aligned");
    return SGDRC_OK;
}

// Every colour of the set must be below ``colours``; the set must not be empty.
static int check_set(const sgdrc_colour_set *set, uint32_t colours)
{
    bool any = false;
    for (uint32_t cc = 0; cc < 256; ++cc) {
        if ((set->bits[cc >> 6] >> (cc & 63)) & 1ull) {
            if (cc >= colours)
                return set_error(SGDRC_EINVAL, "colour %u in set, hash has %u colours", cc, colours);
            any = true;
        }
    }
    if (!any)
        return set_error(SGDRC_EINVAL, "empty colour set");
    return SGDRC_OK;
}

static int check_table(const sgdrc_colour_table *t)
{
    if (!t)
        return set_error(SGDRC_EINVAL, "colour table is NULL");
    if (t->reserved != 0)
        return set_error(SGDRC_EINVAL, "colour table reserved field must be 0");
    if (t->shift < 8 || t->shift > SGDRC_MAX_PAGE_SHIFT)
        return set_error(SGDRC_EINVAL, "partition shift %u outside [8, %d]", t->shift,
                         SGDRC_MAX_PAGE_SHIFT);
    if (t->entries > 0 && !t->lut)
        return set_error(SGDRC_EINVAL, "colour table has entries but no device pointer");
    if (t->origin >= (1ull << 48) || t->entries > (((1ull << 48) - t->origin) >> t->shift))
        return set_error(SGDRC_EINVAL, "colour table extends beyond the 48-bit address space");
    return SGDRC_OK;
}

// Scratch of one build: a count per workgroup of the counting pass.
size_t pt_scratch_bytes() { return kPtMaxChunks * sizeof(uint32_t); }

// The no-allocation build's scratch: a fixed block of the library's own
// device memory (one per device, held until the process ends).  Host code
// never passes the array's name to a kernel (in host code it is only a
// stand-in): it uses the device address that noalloc_scratch_init looks up
// once per context, with the context's device current.
constexpr uint64_t kNoAllocMaxPages = 1ull << 26;
static __device__ __align__(256) uint32_t scratch[kPtMaxChunks];

int noalloc_scratch_init(Ctx *c)
{
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess)
        return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p)
        return set_error(SGDRC_EHIP, "no device address for the page-table scratch");
    c->d_static_scratch = p;
    return SGDRC_OK;
}

static SetArgs set_args(const sgdrc_colour_set &set)
{
    SetArgs sa;
    for (int i = 0; i < 4; ++i) {
        sa.w[2 * i] = (uint32_t)set.bits[i];
        sa.w[2 * i + 1] = (uint32_t)(set.bits[i] >> 32);
    }
    return sa;
}

// The one-launch build of an XOR hash: whether it applies, and its constants.
// counts[j][c] is the number of the 2^j page numbers r < 2^j with
// c ^ colour(r) in the set, colour(r) the XOR of v[b] over r's bits b (v[b] =
// the colour of address bit shift + b): counts[j + 1][c] = counts[j][c] +
// counts[j][c ^ v[j]].  An aligned run of 2^m pages whose first page has
// colour c holds counts[m][c] qualifying pages; the build applies when that
// is the same for every c.  It is whenever the masks have full rank on the
// m lowest page-number bits (all colours then occur equally often), as masks
// that interleave the colours over neighbouring pages do; a hash that only
// selects higher bits takes the general build.
struct PtRuns {
    uint32_t rounds = 0;      // rounds of 1024 pages per run
    uint32_t per_run = 0;     // qualifying pages per run
    uint32_t skip = 0;        // of the first run, before the pool's first page
    uint32_t v0 = 0, v1 = 0;  // the colours of page-number bits 0 and 1
    uint64_t total = 0;       // qualifying pages of the pool
};

static bool plan_runs(const sgdrc_hash *h, uint32_t page_shift, uint64_t q0, uint64_t pool_pages,
                      const sgdrc_colour_set &set, PtRuns *out)
{
    constexpr uint32_t kMaxLog = 12;  // runs of 2^10..2^12 pages: one to four rounds
    const uint32_t n = 1u << h->n_masks;
    uint16_t counts[kMaxLog + 1][256];
    uint32_t v[48] = {};
    for (uint32_t b = 0; page_shift + b < 48u; ++b)
        for (uint32_t k = 0; k < h->n_masks; ++k)
            v[b] |= (uint32_t)((h->masks[k] >> (page_shift + b)) & 1ull) << k;
    for (uint32_t c = 0; c < n; ++c)
        counts[0][c] = (uint16_t)((set.bits[c >> 6] >> (c & 63u)) & 1ull);
    uint32_t m = 0;
    bool same = false;
    while (m < kMaxLog && !(m >= 10u && same)) {
        same = true;
        for (uint32_t c = 0; c < n; ++c) {
            counts[m + 1][c] = (uint16_t)(counts[m][c] + counts[m][c ^ v[m]]);
            same = same && counts[m + 1][c] == counts[m + 1][0];
        }
        ++m;
    }
    if (!same)
        return false;
    const uint64_t run = 1ull << m;
    // qualifying pages of x's run before x
    auto within = [&](uint64_t x) {
        uint32_t c = 0, f = 0;
        for (uint32_t b = m; b < 48u - page_shift; ++b)
            c ^= (x >> b) & 1u ? v[b] : 0u;
        for (uint32_t b = m; b-- > 0;)
            if ((x >> b) & 1u) {
                f += counts[b][c];
                c ^= v[b];
            }
        return f;
    };
    const uint64_t q1 = q0 + pool_pages;
    out->rounds = 1u << (m - 10u);
    out->per_run = counts[m][0];
    out->skip = within(q0);
    out->v0 = v[0];
    out->v1 = v[1];
    out->total = (q1 / run - q0 / run) * out->per_run + within(q1) - out->skip;
    return true;
}

template <int K>
static int launch_runs(const HashArgs &h, const PtRuns &r, uint64_t q0, uint32_t shift,
                       uint64_t pool_pages, const SetArgs &set, uint64_t n_needed, uint32_t *d_pt,
                       uint64_t *d_total, hipStream_t s)
{
    // only the runs that hold the first n_needed qualifying pages
    const uint64_t run = 1024ull * r.rounds;
    const uint64_t runs = (q0 + pool_pages - 1) / run - q0 / run + 1;
    const uint64_t want = std::min(n_needed, r.total);
    const uint64_t grid = want ? std::min(runs, (want + r.skip + r.per_run - 1) / r.per_run) : d_total ? 1 : 0;
    if (!grid)
        return SGDRC_OK;
    hipLaunchKernelGGL((k_pt_runs<K>), dim3((uint32_t)grid), dim3(kPtThreads), 0, s, h, q0, shift,
                       pool_pages, set, r.rounds, r.per_run, r.skip, r.v0, r.v1, d_pt, want,
                       r.total, d_total);
    SGDRC_HIP(hipGetLastError());
    return SGDRC_OK;
}

// The general build: counting pass into ``d_counts``, emitting pass; the
// count of qualifying pages goes to *d_total (device or pinned host memory).
template <class Q>
static int launch_general(const Q &q, uint32_t pages, uint64_t origin, uint32_t shift,
                          uint64_t pool_pages, const SetArgs &set, uint64_t n_needed,
                          uint32_t *d_pt, uint32_t *d_counts, uint64_t *d_total, hipStream_t s)
{
    const uint64_t round = (uint64_t)kPtThreads * pages;  // ``pages``: q.pages()
    const uint64_t rounds = (pool_pages + round - 1) / round;
    const uint64_t chunk = (rounds + kPtMaxChunks - 1) / kPtMaxChunks * round;
    const uint32_t n_chunks = (uint32_t)((pool_pages + chunk - 1) / chunk);
    hipLaunchKernelGGL((k_pt_count<Q>), dim3(n_chunks), dim3(kPtThreads), 0, s, q, origin, shift,
                       pool_pages, chunk, set, d_counts);
    SGDRC_HIP(hipGetLastError());
    hipLaunchKernelGGL((k_pt_emit<Q>), dim3(n_needed ? n_chunks : 1), dim3(kPtThreads), 0, s, q,
                       origin, shift, pool_pages, chunk, set, (const uint32_t *)d_counts, n_chunks,
                       d_pt, n_needed, d_total);
    SGDRC_HIP(hipGetLastError());
    return SGDRC_OK;
}

template <int K>
static int launch_general_xor(const HashArgs &h, uint64_t origin, uint32_t shift,
                              uint64_t pool_pages, const SetArgs &set, uint64_t n_needed,
                              uint32_t *d_pt, uint32_t *d_counts, uint64_t *d_total, hipStream_t s)
{
    return launch_general(QXor<K>{h}, QXor<K>::kPages, origin, shift, pool_pages, set, n_needed, d_pt, d_counts,
                          d_total, s);
}

static int found_or_short(uint64_t found, uint64_t n_needed, uint64_t *n_found)
{
    *n_found = found;
    if (found < n_needed)
        return set_error(SGDRC_ENOMEM, "pool holds %llu pages of the set, %llu needed",
                         (unsigned long long)found, (unsigned long long)n_needed);
    return SGDRC_OK;
}

// The synchronous general build: the context's scratch, the count back
// through pinned host memory (written by the emitting pass).
template <class Launch>
static int build_general(Ctx *c, uint64_t n_needed, uint64_t *n_found, hipStream_t s, Launch launch)
{
    std::lock_guard<std::mutex> lock(g_pt_mu);
    int rc = launch(static_cast<uint32_t *>(c->d_scratch), c->h_pinned);
    if (rc)
        return rc;
    SGDRC_HIP(hipStreamSynchronize(s));
    return found_or_short(c->h_pinned[0], n_needed, n_found);
}

}  // namespace sgdrc

using namespace sgdrc;

#define SGDRC_DISPATCH_K(nm, fn, ...)                         \
    switch (nm) {                                             \
    case 1: rc = fn<1>(__VA_ARGS__); break;                   \
    case 2: rc = fn<2>(__VA_ARGS__); break;                   \
    case 3: rc = fn<3>(__VA_ARGS__); break;                   \
    case 4: rc = fn<4>(__VA_ARGS__); break;                   \
    case 5: rc = fn<5>(__VA_ARGS__); break;                   \
    case 6: rc = fn<6>(__VA_ARGS__); break;                   \
    case 7: rc = fn<7>(__VA_ARGS__); break;                   \
    default: rc = fn<8>(__VA_ARGS__); break;                  \
    }

extern "C" {

int colour_classify(sgdrc_ctx *ctx, const sgdrc_hash *hash, const uint64_t *d_addrs, uint64_t n,
                    uint8_t *d_colours, uint64_t *d_hist, void *stream)
{
    clear_error();
    int rc = check_hash(hash);
    if (rc)
        return rc;
    if (n > 0 && (!d_addrs || !d_colours))
        return set_error(SGDRC_EINVAL, "NULL address or colour buffer");
    if ((reinterpret_cast<uintptr_t>(d_addrs) & 15u) || (reinterpret_cast<uintptr_t>(d_colours) & 15u))
        return set_error(SGDRC_EINVAL, "address and colour buffers must be 16-byte aligned");
    if (reinterpret_cast<uintptr_t>(d_hist) & 7u)
        return set_error(SGDRC_EINVAL, "histogram not 8-byte aligned");
    Ctx *c = nullptr;
    rc = check_ctx(ctx, &c);
    if (rc)
        return rc;
    HashArgs h = hash_args(hash);
    SGDRC_DISPATCH_K(hash->n_masks, launch_classify_xor, c, h, d_addrs, n, d_colours, d_hist,
                     stream);
    return rc;
}

int colour_alloc_pagetable(sgdrc_ctx *ctx, const sgdrc_hash *hash, uint64_t addr_origin,
                           uint32_t page_shift, uint64_t pool_pages, const sgdrc_colour_set *set,
                           uint64_t n_needed, uint32_t *d_pt, uint64_t *n_found, void *stream)
{
    clear_error();
    int rc = check_hash(hash);
    if (rc)
        return rc;
    if ((rc = check_pool_args(addr_origin, page_shift, pool_pages, set, n_needed, d_pt, n_found)))
        return rc;
    if ((rc = check_set(set, 1u << hash->n_masks)))
        return rc;
    Ctx *c = nullptr;
    if ((rc = check_ctx(ctx, &c)))
        return rc;
    const HashArgs h = hash_args(hash);
    const sgdrc_colour_set whole = page_colour_set(hash, page_shift, *set);
    const SetArgs sa = set_args(whole);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    PtRuns r;
    if (plan_runs(hash, page_shift, addr_origin >> page_shift, pool_pages, whole, &r)) {
        SGDRC_DISPATCH_K(hash->n_masks, launch_runs, h, r, addr_origin >> page_shift, page_shift,
                         pool_pages, sa, n_needed, d_pt, (uint64_t *)nullptr, s);
        if (rc)
            return rc;
        SGDRC_HIP(hipStreamSynchronize(s));
        return found_or_short(r.total, n_needed, n_found);
    }
    return build_general(c, n_needed, n_found, s, [&](uint32_t *d_counts, uint64_t *d_total) {
        int rc = SGDRC_OK;
        SGDRC_DISPATCH_K(hash->n_masks, launch_general_xor, h, addr_origin, page_shift, pool_pages,
                         sa, n_needed, d_pt, d_counts, d_total, s);
        return rc;
    });
}

int colour_alloc_pagetable_noalloc(sgdrc_ctx *ctx, const sgdrc_hash *hash, uint64_t addr_origin,
                                   uint32_t page_shift, uint64_t pool_pages,
                                   const sgdrc_colour_set *set, uint64_t n_needed, uint32_t *d_pt,
                                   uint64_t *d_n_found, void *stream)
{
    clear_error();
    int rc = check_hash(hash);
    if (rc)
        return rc;
    if ((rc = check_pool_args(addr_origin, page_shift, pool_pages, set, n_needed, d_pt,
                              d_n_found)))
        return rc;
    if (reinterpret_cast<uintptr_t>(d_n_found) & 7u)
        return set_error(SGDRC_EINVAL, "d_n_found not 8-byte aligned");
    if (pool_pages > kNoAllocMaxPages)
        return set_error(SGDRC_EINVAL, "pool_pages %llu above the %llu pages this build serves",
                         (unsigned long long)pool_pages, (unsigned long long)kNoAllocMaxPages);
    if ((rc = check_set(set, 1u << hash->n_masks)))
        return rc;
    Ctx *c = nullptr;
    if ((rc = check_ctx(ctx, &c)))
        return rc;
    const HashArgs h = hash_args(hash);
    const sgdrc_colour_set whole = page_colour_set(hash, page_shift, *set);
    const SetArgs sa = set_args(whole);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    PtRuns r;
    if (plan_runs(hash, page_shift, addr_origin >> page_shift, pool_pages, whole, &r)) {
        SGDRC_DISPATCH_K(hash->n_masks, launch_runs, h, r, addr_origin >> page_shift, page_shift,
                         pool_pages, sa, n_needed, d_pt, d_n_found, s);
    } else {
        SGDRC_DISPATCH_K(hash->n_masks, launch_general_xor, h, addr_origin, page_shift, pool_pages,
                         sa, n_needed, d_pt, static_cast<uint32_t *>(c->d_static_scratch),
                         d_n_found, s);
    }
    return rc;
}

int colour_classify_table(sgdrc_ctx *ctx, const sgdrc_colour_table *table,
                          const uint64_t *d_addrs, uint64_t n, uint8_t *d_colours,
                          uint64_t *d_hist, void *stream)
{
    clear_error();
    int rc = check_table(table);
    if (rc)
        return rc;
    if (n > 0 && (!d_addrs || !d_colours))
        return set_error(SGDRC_EINVAL, "NULL address or colour buffer");
    if ((reinterpret_cast<uintptr_t>(d_addrs) & 15u) || (reinterpret_cast<uintptr_t>(d_colours) & 15u))
        return set_error(SGDRC_EINVAL, "address and colour buffers must be 16-byte aligned");
    if (reinterpret_cast<uintptr_t>(d_hist) & 7u)
        return set_error(SGDRC_EINVAL, "histogram not 8-byte aligned");
    Ctx *c = nullptr;
    if ((rc = check_ctx(ctx, &c)))
        return rc;
    // (an empty table: any readable byte, see table_colour)
    const uint8_t *lut = table->entries ? table->lut : reinterpret_cast<const uint8_t *>(c->d_lut);
    const TableArgs t{lut, table->origin, table->entries, table->shift};
    return launch_classify<8, true>(c, HashArgs{}, t, d_addrs, n, d_colours, d_hist, stream);
}

int colour_alloc_pagetable_table(sgdrc_ctx *ctx, const sgdrc_colour_table *table,
                                 uint64_t addr_origin, uint32_t page_shift, uint64_t pool_pages,
                                 const sgdrc_colour_set *set, uint64_t n_needed, uint32_t *d_pt,
                                 uint64_t *n_found, void *stream)
{
    clear_error();
    int rc = check_table(table);
    if (rc)
        return rc;
    if ((rc = check_pool_args(addr_origin, page_shift, pool_pages, set, n_needed, d_pt, n_found)))
        return rc;
    if ((rc = check_set(set, 255u)))
        return rc;
    Ctx *c = nullptr;
    if ((rc = check_ctx(ctx, &c)))
        return rc;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const TableArgs t{table->lut, table->origin, table->entries, table->shift};
    // a page is 1 to 16 whole partitions, counted from a partition's start
    const bool aligned = page_shift >= table->shift && page_shift <= table->shift + 4u &&
                         ((addr_origin - table->origin) & ((1ull << table->shift) - 1ull)) == 0u;
    return build_general(c, n_needed, n_found, s, [&](uint32_t *d_counts, uint64_t *d_total) {
        const SetArgs sa = set_args(*set);
        if (aligned) {
            const uint32_t lp = page_shift - table->shift;
            return launch_general(QTable<true>{t, lp}, 16u >> lp, addr_origin, page_shift,
                                  pool_pages, sa, n_needed, d_pt, d_counts, d_total, s);
        }
        return launch_general(QTable<false>{t, 0u}, 1u, addr_origin, page_shift, pool_pages, sa,
                              n_needed, d_pt, d_counts, d_total, s);
    });
}

}  // extern "C"
