// Top-k sparsification by magnitude on gfx950 (§2.2 "Structured
// Sparsification"; Alg. 1: TopK and the error update eps = acc - TopK(acc)).
//
// Exact radix select on the 31-bit magnitude key (IEEE bits, sign cleared),
// normally in one pass over the data.  A histogram of the top 11 key bits
// over a sample of the row (1024 segments of 256 elements) gives a gather
// bin safely below the k-th largest key; the gather pass collects, per
// 4096-element wave unit, every entry in that bin or above it as {element,
// value bits} in index order (a few per unit).  If the row then holds at
// least k gathered keys, the k-th largest key K* and how many entries equal
// to it are still needed follow from the gathered keys alone (11-, 10- and
// 10-bit histograms), which also give every unit its counts; a scan over
// the units gives output offsets, and the selection is written from the
// gathered entries (equal keys: lowest index first), zeroing the residual
// at the selected positions.  Otherwise the row takes the exact gather bin
// from a histogram of all its keys and gathers again; a row with a unit
// holding more than kSlots entries even then takes two more histogram
// passes, a count pass and a write pass over its data.
//
// Where a unit would gather too much (more than kSlots / 4 selections expected),
// a short row takes the histogram passes at once, and of a long one the
// selection is bracketed: a larger and finer sample gives a window
// of keys that holds K*, one pass counts each unit's keys above it and keeps
// those inside it (a few per unit), histograms of these give K*, and a second
// pass over the data writes the selection.  A row whose K* lies outside its
// window, or with a unit holding more than kWinSlots keys inside, takes the
// histogram passes over its data.  Every path is exact: the sample only
// decides how much data is read.
//
// One row of 23.5 M with k = 1% and a new residual: a call takes 449 us by the
// histogram passes from 64 workgroups, 126 us by the window.
#include "internal.h"

#include <algorithm>

namespace sparcml {
namespace {

constexpr uint32_t kUnit = 4096;  // elements per wave unit (64 iterations of 64 lanes)
constexpr uint32_t kSlots = 32;   // gathered entries per unit
constexpr int kHistBlocksPerRank = 64;
constexpr uint32_t kExactGatherBlocks = 64;  // workgroups per row of the exact path's gather (grid-stride)
constexpr uint64_t kSampleSegs = 1024;  // 256-element segments sampled per row
// Gathered keys are also listed per row in kSub sub-lists (unit u appends to
// sub-list u mod kSub, reserving its place with one atomic on that
// sub-list's counter, each counter on a cache line of its own, so that no
// counter takes more than a few hundred atomics); a full sub-list counts as
// an overflow.
constexpr uint32_t kSub = 64;
constexpr uint32_t kSubCap = 1024;                     // keys per sub-list
constexpr uint32_t kList = kSub * kSubCap;             // keys listed per row
constexpr uint32_t kCntStride = 32;                    // counter words apart (128 B)

__device__ __forceinline__ uint32_t mag_key(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

enum : uint32_t { kGathered = 0, kPasses = 1, kWindowed = 2 };  // RankState::full

struct RankState {
    uint32_t prefix;  // key bits fixed so far (gather: the lowest 11-bit bin gathered)
    uint32_t full;    // K* from the gathered keys; by passes over the data; from a window of keys
    uint64_t krem;    // entries still to take from keys matching the prefix
    uint32_t exact;   // 0: gather bin (or window) estimated from a sample; 1: from the full histogram
    uint32_t pad;
};

// The window's space in a row's key list (a windowed row lists no keys):
// sample histogram of the top 15 key bits, histogram of the window's keys in
// 2048 parts, histogram (or, of a wide one, list) of one part's keys, and the
// window.
constexpr uint32_t kFine = 32768;
constexpr uint32_t kWinHist = kFine, kWinPart = kFine + 2048, kWinState = kFine + 3072;
constexpr uint32_t kWinWords = kWinState + 4;  // lowest key, first key above, log2 of a part's width; keys listed
constexpr uint32_t kWinList = kList - kWinWords;
constexpr uint32_t kWinSlots = 2 * kSlots;     // keys a unit keeps, in the space of its kSlots entries
constexpr uint64_t kWinSegs = 2048;            // 256-element segments sampled per row
static_assert(kWinWords + 16384 <= kList, "the window fits the key list");

// Whether this is the last of a row's `blocks` workgroups to get here: what the others wrote
// before by device-scope atomics is then seen by device-scope loads (seen).  These bypass the XCDs' own L2s; a fence would write the whole L2
// back, once per workgroup (sparsification of 32 rows of 2^24: 923 against 474
// us).  Tickets: spare words of the row's list counters, one per kernel.
enum { kTickHist = 1, kTickSample = 4, kTickGather = 5, kTickPart = 6 };
__device__ __forceinline__ bool last_of_row(uint32_t* kcnt, uint32_t r, uint32_t tick, uint32_t blocks, uint32_t* s_last)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's atomics are done
    __syncthreads();
    if (threadIdx.x == 0)
        *s_last = atomicAdd(&kcnt[(uint64_t)r * kSub * kCntStride + tick], 1u) == blocks - 1u ? 1u : 0u;
    __syncthreads();
    return *s_last != 0u;
}
__device__ __forceinline__ uint32_t seen(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keys of row r from element lo to hi (lo a multiple of 4), in float4 loads
// where the row is 16-byte aligned; f(element, key) in any order.
template <typename F>
__device__ __forceinline__ void for_keys(const float* row, uint64_t lo, uint64_t hi, uint32_t t,
                                         uint32_t nt, F&& f)
{
    if ((reinterpret_cast<uintptr_t>(row) & 15u) == 0u) {
        // batches of four float4 loads per thread, all issued before use
        const uint64_t step = 16ull * nt, hb = lo + ((hi - lo) / step) * step;
        for (uint64_t e = lo + 4ull * t; e < hb; e += step) {
            float4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const float4*>(row + e + 4ull * nt * q);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t b = e + 4ull * nt * q;
                f(b, mag_key(v[q].x));
                f(b + 1, mag_key(v[q].y));
                f(b + 2, mag_key(v[q].z));
                f(b + 3, mag_key(v[q].w));
            }
        }
        const uint64_t hv = hb + ((hi - hb) & ~3ull);
        for (uint64_t e = hb + 4ull * t; e < hv; e += 4ull * nt) {
            const float4 v = *reinterpret_cast<const float4*>(row + e);
            f(e, mag_key(v.x));
            f(e + 1, mag_key(v.y));
            f(e + 2, mag_key(v.z));
            f(e + 3, mag_key(v.w));
        }
        for (uint64_t e = hv + t; e < hi; e += nt) f(e, mag_key(row[e]));
    } else {
        // eight single loads in flight (8 rows of 20,001, 43 selected of each: 85 -> 51 us)
        const uint64_t step = 8ull * nt, hb = lo + ((hi - lo) / step) * step;
        for (uint64_t e = lo + t; e < hb; e += step) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = row[e + (uint64_t)nt * q];
#pragma unroll
            for (int q = 0; q < 8; ++q) f(e + (uint64_t)nt * q, mag_key(v[q]));
        }
        for (uint64_t e = hb + t; e < hi; e += nt) f(e, mag_key(row[e]));
    }
}

// PASS 0: bins = key >> 20 (2048); PASS 1: (key >> 10) & 1023 among keys
// whose top 11 bits match; PASS 2: key & 1023 among keys whose top 21 bits
// match.  The row's last workgroup finds the bin holding the krem-th largest
// remaining key, refines the state and clears the histogram for the next pass.
template <int PASS>
__device__ void hist_pass(const float* x, uint64_t N, RankState* st, uint32_t* hist, uint32_t* kcnt)
{
    constexpr uint32_t NB = PASS == 0 ? 2048u : 1024u, PER = NB / 256;
    constexpr int BITS = PASS == 0 ? 11 : 10;
    constexpr int SHIFT = PASS == 0 ? 20 : (PASS == 1 ? 10 : 0);
    constexpr int PSHIFT = PASS == 1 ? 20 : 10;
    __shared__ uint32_t s_h[NB];
    __shared__ uint64_t s_w[4];
    __shared__ uint32_t s_last;
    const uint32_t r = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (PASS == 0 ? st[r].exact == 0u : st[r].full != kPasses) return;  // row not on this path
    for (uint32_t i = tid; i < NB; i += 256) s_h[i] = 0;
    __syncthreads();
    const uint32_t prefix = PASS == 0 ? 0u : st[r].prefix;
    const uint64_t krem = st[r].krem;
    const float* row = x + (uint64_t)r * N;
    const uint64_t per = ((N + gridDim.x - 1) / gridDim.x + 3) & ~3ull;
    const uint64_t lo_e = min((uint64_t)blockIdx.x * per, N), hi_e = min(lo_e + per, N);
    for_keys(row, lo_e, hi_e, tid, 256u, [&](uint64_t, uint32_t key) {
        if (PASS == 0 || (key >> PSHIFT) == prefix) atomicAdd(&s_h[(key >> SHIFT) & (NB - 1)], 1u);
    });
    __syncthreads();
    uint32_t* h = hist + (uint64_t)r * 2048;
    for (uint32_t i = tid; i < NB; i += 256)
        if (s_h[i]) atomicAdd(&h[i], s_h[i]);
    if (!last_of_row(kcnt, r, kTickHist + PASS, gridDim.x, &s_last)) return;
    // thread tid owns bins [lo, lo+PER); threads are ordered from the top
    const uint32_t lo = NB - (tid + 1) * PER;
    uint32_t cnt[PER];
    uint64_t mine = 0;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        cnt[i] = seen(&h[lo + i]);
        mine += cnt[i];
    }
    uint64_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(incl, o);
        if (lane >= (uint32_t)o) incl += y;
    }
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    uint64_t above = incl - mine;  // entries in bins above this thread's bins
    for (uint32_t w = 0; w < wv; ++w) above += s_w[w];
    uint64_t run = above;
    for (int i = (int)PER - 1; i >= 0; --i) {
        if (run < krem && run + cnt[i] >= krem) {
            st[r].prefix = (prefix << BITS) | (lo + (uint32_t)i);
            st[r].krem = krem - run;
        }
        run += cnt[i];
    }
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) h[lo + i] = 0;
}
template <int PASS>
__global__ void __launch_bounds__(256) k_hist(const float* x, uint64_t N, RankState* st, uint32_t* hist, uint32_t* kcnt)
{
    hist_pass<PASS>(x, N, st, hist, kcnt);
}

// win: the rows' windows are cleared too; passes: every row starts with the
// passes over its data.
__global__ void __launch_bounds__(256) k_init(RankState* st, uint32_t P, uint64_t k, uint32_t* hist, uint32_t* overflow,
                                              uint32_t* kcnt, uint32_t* klist, uint32_t win, uint32_t passes)
{
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x, nt = gridDim.x * 256u;
    for (uint32_t i = gid; i < P * kSub; i += nt) kcnt[(uint64_t)i * kCntStride] = 0;
    for (uint32_t i = gid; i < P * 6u; i += nt) kcnt[(uint64_t)(i / 6u) * kSub * kCntStride + 1u + i % 6u] = 0;
    for (uint32_t i = gid; i < P; i += nt) {
        st[i].prefix = 0;
        st[i].full = passes ? kPasses : kGathered;
        st[i].krem = k;
        st[i].exact = passes;
        st[i].pad = 0;
        overflow[i] = 0;
    }
    for (uint32_t i = gid; i < P * 2048u; i += nt) hist[i] = 0;
    if (win)
        for (uint32_t i = gid; i < P * kWinWords; i += nt) klist[(uint64_t)(i / kWinWords) * kList + i % kWinWords] = 0;
}

__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s_w, uint32_t* total)
{
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= (uint32_t)o) incl += y;
    }
    __syncthreads();
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    uint32_t ex = incl - v, t = 0;
    for (uint32_t w = 0; w < nw; ++w) {
        if (w < wv) ex += s_w[w];
        t += s_w[w];
    }
    *total = t;
    return ex;
}

// Sample histogram of the top 11 key bits: kSampleSegs segments of 256
// consecutive elements spread evenly over the row (all of a short row).
__global__ void __launch_bounds__(256) k_sample(const float* x, uint64_t N, uint32_t stride, uint32_t* hist)
{
    __shared__ uint32_t s_h[2048];
    const uint32_t r = blockIdx.y;
    for (uint32_t i = threadIdx.x; i < 2048; i += 256) s_h[i] = 0;
    __syncthreads();
    const float* row = x + (uint64_t)r * N;
    const uint64_t nseg = (N + 255) / 256, step = (uint64_t)gridDim.x * stride;
    for (uint64_t g = (uint64_t)blockIdx.x * stride; g < nseg; g += 4 * step) {
        float v[4];
        bool ok[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // four segments' loads in flight
            const uint64_t e = (g + q * step) * 256 + threadIdx.x;
            ok[q] = g + q * step < nseg && e < N;
            v[q] = ok[q] ? row[e] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (ok[q]) atomicAdd(&s_h[mag_key(v[q]) >> 20], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < 2048; i += 256)
        if (s_h[i]) atomicAdd(&hist[(uint64_t)r * 2048 + i], s_h[i]);
}

// The gather bin of a row from its sample: the 11-bit bin of the t-th
// largest sampled key, t = k f + 4 sqrt(k f) + 16 for sample fraction f --
// low enough that the row holds at least k keys at or above it, barring a
// sample off by more than four standard deviations (checked after the
// gather).  Clears the histogram.
__global__ void __launch_bounds__(256) k_estimate(RankState* st, uint32_t* hist, uint64_t k, double f)
{
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_bin;
    const uint32_t r = blockIdx.x, tid = threadIdx.x;
    uint32_t* h = hist + (uint64_t)r * 2048;
    const double kf = (double)k * f;
    const uint64_t t = (uint64_t)ceil(kf + 4.0 * sqrt(kf) + 16.0);
    // thread tid owns bins [lo, lo + 8), threads ordered from the top
    const uint32_t lo = 2048u - (tid + 1u) * 8u;
    uint32_t cnt[8], mine = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        cnt[i] = h[lo + i];
        mine += cnt[i];
    }
    if (tid == 0) s_bin = 0u;  // the whole row when the sample holds fewer than t keys
    uint32_t total;
    uint64_t run = block_excl_scan(mine, s_w, &total);
    for (int i = 7; i >= 0; --i) {
        if (run < t && run + cnt[i] >= t) s_bin = lo + (uint32_t)i;
        run += cnt[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) h[lo + i] = 0;
    if (tid == 0) st[r].prefix = s_bin;
}

// Per wave unit: every entry whose top 11 key bits are at or above the
// gather bin goes as {element, value bits} into the unit's kSlots slots in
// index order, and its key into the row's key list (a unit with more, or a
// full list, flags its row for the next path).  A separate residual
// receives a copy of the row here.
__global__ void __launch_bounds__(256) k_gather(const float* x, uint64_t N, uint32_t U, const RankState* st,
                                                uint2* cand, uint32_t* ccnt, uint32_t* overflow, float* residual,
                                                uint32_t exact, uint32_t* klist, uint32_t* kcnt)
{
    const uint32_t r = blockIdx.y, lane = threadIdx.x & 63;
    if (st[r].exact != exact) return;  // not this path
    // units one a wave, grid-stride: the fallback launch takes a grid
    // smaller than the row's units (most rows skip it at once)
    for (uint32_t u = blockIdx.x * 4 + (threadIdx.x >> 6); u < U; u += gridDim.x * 4) {
        if (overflow[r] != 0u) return;  // gathered too many
        const uint32_t bin = st[r].prefix;
        const float* row = x + (uint64_t)r * N;
        float* res = residual && residual != x ? residual + (uint64_t)r * N : nullptr;
        const uint64_t lo = (uint64_t)u * kUnit, hi = min(lo + kUnit, N);
        uint2* cu = cand + ((uint64_t)r * U + u) * kSlots;
        const uint32_t sub = u % kSub;
        uint32_t* kl = klist + ((uint64_t)r * kSub + sub) * kSubCap;
        uint32_t* kc = kcnt + ((uint64_t)r * kSub + sub) * kCntStride;
        // The unit's count first, then its entries: into the unit's slots in
        // index order and, at a place reserved with one atomic, into the row's
        // key list.  Returns whether the unit's entries are to be written.
        auto reserve = [&](uint32_t nc, uint32_t* base) {
            uint32_t b = kSubCap;
            if (lane == 0) {
                ccnt[(uint64_t)r * U + u] = nc;
                if (nc > kSlots) {
                    atomicOr(&overflow[r], 1u);
                } else if (nc) {
                    b = atomicAdd(kc, nc);
                    if (b + nc > kSubCap) atomicOr(&overflow[r], 1u);
                }
            }
            *base = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
            return nc != 0u && nc <= kSlots && *base + nc <= kSubCap;
        };
        auto put = [&](uint32_t at, uint32_t base, uint64_t e, float v) {
            cu[at] = make_uint2((uint32_t)e, __float_as_uint(v));
            kl[base + at] = mag_key(v);
        };
        const bool rvec = res == nullptr || (reinterpret_cast<uintptr_t>(res) & 15u) == 0u;
        if ((reinterpret_cast<uintptr_t>(row) & 15u) == 0u && rvec && hi - lo == kUnit) {
            // the unit's 16 float4 per lane, all requested before use (loads
            // marked nontemporal: the row is streamed once); lane i holds
            // elements 4i..4i+3 of every 256, so entries are placed in index
            // order by a wave scan per 256 elements that hold any
            float4 vs[kUnit / 256];
    #pragma unroll
            for (uint32_t q = 0; q < kUnit / 256; ++q)
                vs[q] = load_nt(row + lo + 256u * q + 4u * lane);
            // in-bin flags of the lane's elements, bit k of nibble q for element
            // 256q + 4 lane + k (two words of eight nibbles: a handful of
            // registers instead of 64 lane masks)
            auto in4 = [&](const float4& v) {
                return (uint32_t)((mag_key(v.x) >> 20) >= bin) | (uint32_t)((mag_key(v.y) >> 20) >= bin) << 1 |
                       (uint32_t)((mag_key(v.z) >> 20) >= bin) << 2 | (uint32_t)((mag_key(v.w) >> 20) >= bin) << 3;
            };
            uint32_t fl[2] = {0u, 0u};
    #pragma unroll
            for (uint32_t q = 0; q < kUnit / 256; ++q) {
                fl[q / 8] |= in4(vs[q]) << (4 * (q % 8));
                if (res) store_nt(res + lo + 256u * q + 4u * lane, vs[q]);
            }
            const uint32_t mine = (uint32_t)__popc(fl[0]) + (uint32_t)__popc(fl[1]);
            const uint32_t nc = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(mine), 63);
            uint32_t base;
            if (reserve(nc, &base)) {
                uint32_t run = 0;
    #pragma unroll
                for (uint32_t q = 0; q < kUnit / 256; ++q) {
                    const uint32_t f = (fl[q / 8] >> (4 * (q % 8))) & 15u;
                    const uint32_t n4 = (uint32_t)__popc(f);
                    if (__ballot(n4 != 0u) == 0ull) continue;  // no entry in these 256 elements
                    const uint64_t e = lo + 256u * q + 4u * lane;
                    const uint32_t incl = wave_scan(n4);
                    uint32_t at = run + incl - n4;
                    if (f & 1u) put(at++, base, e, vs[q].x);
                    if (f & 2u) put(at++, base, e + 1, vs[q].y);
                    if (f & 4u) put(at++, base, e + 2, vs[q].z);
                    if (f & 8u) put(at, base, e + 3, vs[q].w);
                    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                }
            }
        } else {
            // short or unaligned unit: count (and copy), then read again to place
            uint32_t nc = 0;
            for (uint64_t e0 = lo; e0 < hi; e0 += 64) {
                const uint64_t e = e0 + lane;
                const float v = e < hi ? row[e] : 0.0f;
                nc += (uint32_t)__popcll(__ballot(e < hi && (mag_key(v) >> 20) >= bin));
                if (res && e < hi) res[e] = v;
            }
            uint32_t base;
            if (reserve(nc, &base)) {
                uint32_t run = 0;
                for (uint64_t e0 = lo; e0 < hi; e0 += 64) {
                    const uint64_t e = e0 + lane;
                    const float v = e < hi ? row[e] : 0.0f;
                    const bool in = e < hi && (mag_key(v) >> 20) >= bin;
                    const uint64_t m = __ballot(in);
                    if (in) put(run + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)), base, e, v);
                    run += (uint32_t)__popcll(m);
                }
            }
        }
    }
}

// Bin (of NB, ordered from the top) holding the krem-th largest key of a
// histogram held one bin per thread (thread t: bin NB-1-t); returns the bin
// and, through *rem, krem less the keys in the bins above it.
__device__ uint32_t block_find(uint32_t cnt, uint64_t krem, uint32_t NB, uint64_t* rem, uint32_t* s_w,
                               uint32_t* s_res)
{
    uint32_t total;
    const uint32_t above = block_excl_scan(cnt, s_w, &total);
    if (above < krem && above + cnt >= krem) {
        s_res[0] = NB - 1u - threadIdx.x;
        s_res[1] = (uint32_t)(krem - above);
    }
    __syncthreads();
    *rem = s_res[1];
    return s_res[0];
}

// K* and the ties still needed, from the key list of row r (every key at or
// above its gather bin), for the rows on the path `exact` names.  After the
// sampled gather (exact = 0) a row that gathered fewer than k keys, or
// overflowed, is sent to the exact path instead; after the exact gather a row
// that overflowed is sent to the passes over its data.
__global__ void __launch_bounds__(1024) k_cand_select(uint64_t k, RankState* st, const uint32_t* klist,
                                                      uint32_t* kcnt, uint32_t* overflow, uint32_t exact)
{
    __shared__ uint32_t s_h[2048];
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_res[2];
    const uint32_t r = blockIdx.x, t = threadIdx.x;
    if (st[r].exact != exact || st[r].full != 0u) return;  // row not on this path (whole workgroup)
    // keys gathered for the row (the sub-list counters) and the overflow flag
    uint32_t total;
    block_excl_scan(t < kSub ? kcnt[((uint64_t)r * kSub + t) * kCntStride] : 0u, s_w, &total);
    const bool ov = overflow[r] != 0u;
    if (exact == 0u && (ov || total < k)) {
        // the sampled bin failed: the exact one from a histogram of the row,
        // then a second gather
        if (t == 0) {
            st[r].exact = 1u;
            st[r].prefix = 0u;
            st[r].krem = k;
            overflow[r] = 0u;
        }
        if (t < kSub) kcnt[((uint64_t)r * kSub + t) * kCntStride] = 0u;
        return;
    }
    if (ov) {  // too many to gather even from the exact bin: passes over the data
        if (t == 0) st[r].full = kPasses;
        return;
    }
    // every listed key: 16 threads per sub-list, four loads per thread in
    // flight: f(key)
    const uint32_t sub = t / 16u, j = t % 16u;
    const uint32_t* kl = klist + ((uint64_t)r * kSub + sub) * kSubCap;
    const uint32_t n = kcnt[((uint64_t)r * kSub + sub) * kCntStride];
    auto for_keys = [&](auto&& f) {
        for (uint32_t i0 = j; i0 < n; i0 += 64u) {
            uint32_t key[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) key[q] = i0 + 16u * q < n ? kl[i0 + 16u * q] : 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (i0 + 16u * q < n) f(key[q]);
        }
    };
    // The listed keys are every key at or above the gather bin, so the k-th
    // largest of them is the row's: its top 11 bits (2048 bins, two per
    // thread), then bits 19..10, then bits 9..0.
    uint64_t krem = k;
    s_h[t] = 0;
    s_h[t + 1024] = 0;
    __syncthreads();
    for_keys([&](uint32_t key) { atomicAdd(&s_h[key >> 20], 1u); });
    __syncthreads();
    uint32_t bin;
    {
        // thread t: bins 2047-2t and 2046-2t
        const uint32_t hb = s_h[2047u - 2u * t], lb = s_h[2046u - 2u * t];
        uint32_t total;
        const uint32_t above = block_excl_scan(hb + lb, s_w, &total);
        if (above < krem && above + hb >= krem) {
            s_res[0] = 2047u - 2u * t;
            s_res[1] = (uint32_t)(krem - above);
        } else if (above + hb < krem && above + hb + lb >= krem) {
            s_res[0] = 2046u - 2u * t;
            s_res[1] = (uint32_t)(krem - above - hb);
        }
        __syncthreads();
        bin = s_res[0];
        krem = s_res[1];
    }
    __syncthreads();
    s_h[t] = 0;
    __syncthreads();
    for_keys([&](uint32_t key) {
        if ((key >> 20) == bin) atomicAdd(&s_h[(key >> 10) & 1023u], 1u);
    });
    __syncthreads();
    const uint32_t b2 = block_find(s_h[1023u - t], krem, 1024u, &krem, s_w, s_res);
    const uint32_t p21 = bin << 10 | b2;
    __syncthreads();
    s_h[t] = 0;
    __syncthreads();
    for_keys([&](uint32_t key) {
        if ((key >> 10) == p21) atomicAdd(&s_h[key & 1023u], 1u);
    });
    __syncthreads();
    const uint32_t b3 = block_find(s_h[1023u - t], krem, 1024u, &krem, s_w, s_res);
    if (t == 0) {
        st[r].prefix = p21 << 10 | b3;
        st[r].krem = krem;
    }
}


// The row's window from a sample of the top 15 key bits (segments as in
// k_sample, read once): the bins of the t-th largest sampled keys, t = k f
// -+ (4 sqrt(k f) + 16) for sample fraction f; every key at or above the
// upper bin's end lies above the window.  One workgroup holds all bins in
// LDS; the row's last one finds the window.
__global__ void __launch_bounds__(1024) k_win_sample(const float* x, uint64_t N, uint32_t stride, uint64_t k, double f,
                                                     RankState* st, uint32_t* klist, uint32_t* kcnt)
{
    __shared__ __align__(16) uint32_t s_h[kFine];
    __shared__ uint32_t s_w[16], s_last, s_bin[2], s_cnt[2];  // the window's bins; samples from the lower on, above the upper
    const uint32_t r = blockIdx.y, tid = threadIdx.x;
    uint32_t* kw = klist + (uint64_t)r * kList;
    for (uint32_t i = tid * 4u; i < kFine; i += 4096u) *reinterpret_cast<uint4*>(&s_h[i]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const float* row = x + (uint64_t)r * N;
    const uint64_t nseg = (N + 255) / 256, step = (uint64_t)gridDim.x * 4u * stride;
    for (uint64_t g = ((uint64_t)blockIdx.x * 4u + (tid >> 8)) * stride; g < nseg; g += 4 * step) {
        float v[4];
        bool ok[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // four segments' loads in flight
            const uint64_t e = (g + q * step) * 256 + (tid & 255u);
            ok[q] = g + q * step < nseg && e < N;
            v[q] = ok[q] ? row[e] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (ok[q]) atomicAdd(&s_h[mag_key(v[q]) >> 16], 1u);
    }
    __syncthreads();
    for (uint32_t i = tid * 4u; i < kFine; i += 4096u) {
        const uint4 n = *reinterpret_cast<const uint4*>(&s_h[i]);
        if (n.x) atomicAdd(&kw[i], n.x);
        if (n.y) atomicAdd(&kw[i + 1u], n.y);
        if (n.z) atomicAdd(&kw[i + 2u], n.z);
        if (n.w) atomicAdd(&kw[i + 3u], n.w);
    }
    if (!last_of_row(kcnt, r, kTickSample, gridDim.x, &s_last)) return;
    const double kf = (double)k * f, d = 4.0 * sqrt(kf) + 16.0;
    const uint32_t t_lo = (uint32_t)ceil(kf + d), t_hi = kf > d ? (uint32_t)floor(kf - d) : 0u;
    if (tid < 2u) s_bin[tid] = tid ? kFine - 1u : 0u;  // (no such key: to the end of the range)
    // thread tid owns bins [lo, lo + 32), threads ordered from the top
    const uint32_t lo = kFine - (tid + 1u) * 32u;
    uint32_t mine = 0u;
    {
        uint32_t n[32];
#pragma unroll
        for (uint32_t i = 0; i < 32u; ++i) n[i] = seen(&kw[1024u * i + tid]);
#pragma unroll
        for (uint32_t i = 0; i < 32u; ++i) s_h[1024u * i + tid] = n[i];
    }
    __syncthreads();
    for (uint32_t i = 0; i < 32u; i += 4u) {
        const uint4 n = *reinterpret_cast<const uint4*>(&s_h[lo + i]);
        mine += n.x + n.y + n.z + n.w;
    }
    uint32_t total;
    uint32_t run = block_excl_scan(mine, s_w, &total);
    if (tid < 2u) s_cnt[tid] = tid ? 0u : total;
    __syncthreads();
    if (run < t_lo) {  // (few threads: those above the lower bound)
        for (int i = 31; i >= 0; --i) {
            const uint32_t n = s_h[lo + (uint32_t)i];
            if (run < t_lo && run + n >= t_lo) {
                s_bin[0] = lo + (uint32_t)i;
                s_cnt[0] = run + n;
            }
            if (run < t_hi && run + n >= t_hi) {
                s_bin[1] = lo + (uint32_t)i;
                s_cnt[1] = run;
            }
            run += n;
        }
    }
    __syncthreads();
    if (tid == 0) {
        // a window with more keys than units take (ties): the passes at once (64 rows
        // of 2^20 equal magnitudes, 1%: 1.18 -> 1.01 ms)
        if ((uint64_t)(s_cnt[0] - s_cnt[1]) * kUnit > (uint64_t)kWinSlots * total) {
            st[r].exact = 1u;
            st[r].full = kPasses;
        }
        const uint32_t klo = s_bin[0] << 16, khi = (s_bin[1] + 1u) << 16;
        uint32_t sh = 0u;
        while ((khi - 1u - klo) >> sh >= 2048u) ++sh;
        kw[kWinState] = klo;
        kw[kWinState + 1u] = khi;
        kw[kWinState + 2u] = sh;
    }
}

// Krem-th largest of NB bins (NB <= 2048, from the top) read through `get`,
// by 256 threads: the bin, and krem less the keys above it; false if the bins
// hold fewer.
template <uint32_t NB, typename F>
__device__ bool find_bin(F&& get, uint64_t krem, uint32_t* bin, uint32_t* rem, uint32_t* s_w, uint32_t* s_res)
{
    constexpr uint32_t PER = NB / 256u;
    const uint32_t lo = NB - (threadIdx.x + 1u) * PER;
    uint32_t cnt[PER], mine = 0u, total;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        cnt[i] = get(lo + i);
        mine += cnt[i];
    }
    uint32_t run = block_excl_scan(mine, s_w, &total);
    for (int i = (int)PER - 1; i >= 0; --i) {
        if (run < krem && run + cnt[i] >= krem) {
            s_res[0] = lo + (uint32_t)i;
            s_res[1] = (uint32_t)(krem - run);
        }
        run += cnt[i];
    }
    __syncthreads();
    *bin = s_res[0];
    *rem = s_res[1];
    return krem != 0u && total >= krem;
}

// Per wave unit: the number of keys above the window, and the keys inside it
// (in any order), also counted in 2048 parts of the window.  The row's last
// workgroup finds the part that holds K*, or sends the row to the passes over
// its data.
__global__ void __launch_bounds__(256) k_win_gather(const float* x, uint64_t N, uint64_t k, uint32_t U, RankState* st,
                                                    uint2* cand, uint32_t* ccnt, uint32_t* cgt, uint32_t* overflow,
                                                    uint32_t* klist, uint32_t* kcnt)
{
    __shared__ uint32_t s_h[2048];
    __shared__ uint32_t s_w[4], s_res[2], s_last, s_above;
    const uint32_t r = blockIdx.y, tid = threadIdx.x, lane = tid & 63u;
    if (st[r].exact != 0u) return;
    uint32_t* kw = klist + (uint64_t)r * kList;
    const uint32_t klo = kw[kWinState], khi = kw[kWinState + 1u], sh = kw[kWinState + 2u];
    for (uint32_t i = tid; i < 2048u; i += 256u) s_h[i] = 0u;
    if (tid == 0) s_above = 0u;
    __syncthreads();
    const float* row = x + (uint64_t)r * N;
    uint32_t above = 0u;
    for (uint32_t u = blockIdx.x * 4u + (tid >> 6); u < U; u += gridDim.x * 4u) {
        if (overflow[r] != 0u) break;
        const uint64_t lo = (uint64_t)u * kUnit, hi = min(lo + kUnit, N);
        uint32_t* cu = reinterpret_cast<uint32_t*>(cand + ((uint64_t)r * U + u) * kSlots);
        uint32_t nin = 0u, nup = 0u;  // of the unit
        auto put = [&](uint32_t key, uint32_t at) {
            cu[at] = key;
            atomicAdd(&s_h[(key - klo) >> sh], 1u);
        };
        if ((reinterpret_cast<uintptr_t>(row) & 15u) == 0u && hi - lo == kUnit) {
            constexpr uint32_t Q = 8u;  // float4 of a lane in flight (16: fewer waves fit, 35 against 33 us for 94 MB)
#pragma unroll 1
            for (uint32_t q0 = 0; q0 < kUnit / 256; q0 += Q) {
                float4 vs[Q];
#pragma unroll
                for (uint32_t q = 0; q < Q; ++q)
                    vs[q] = *reinterpret_cast<const float4*>(row + lo + 256u * (q0 + q) + 4u * lane);
                uint32_t fl = 0u, up = 0u;  // inside the window: bit k of nibble q, element 256 (q0 + q) + 4 lane + k
#pragma unroll
                for (uint32_t q = 0; q < Q; ++q) {
                    const float v4[4] = {vs[q].x, vs[q].y, vs[q].z, vs[q].w};
#pragma unroll
                    for (uint32_t i = 0; i < 4u; ++i) {
                        const uint32_t key = mag_key(v4[i]);
                        up += key >= khi ? 1u : 0u;
                        fl |= key - klo < khi - klo ? 1u << (4u * q + i) : 0u;
                    }
                }
                const uint32_t mine = (uint32_t)__popc(fl), incl = wave_scan(mine | up << 16);  // (at most 2048 each)
                const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                uint32_t at = nin + (incl & 0xFFFFu) - mine;
                nin += all & 0xFFFFu;
                nup += all >> 16;
                if (nin > kWinSlots) continue;
#pragma unroll
                for (uint32_t q = 0; q < Q; ++q) {
                    const uint32_t f = fl >> (4u * q) & 15u;
                    if (__ballot(f != 0u) == 0ull) continue;  // no entry in these 256 elements
                    if (f & 1u) put(mag_key(vs[q].x), at++);
                    if (f & 2u) put(mag_key(vs[q].y), at++);
                    if (f & 4u) put(mag_key(vs[q].z), at++);
                    if (f & 8u) put(mag_key(vs[q].w), at++);
                }
            }
        } else {
            for (uint64_t e0 = lo; e0 < hi; e0 += 64) {
                const uint64_t e = e0 + lane;
                const uint32_t key = e < hi ? mag_key(row[e]) : 0u;
                const bool in = e < hi && key - klo < khi - klo;
                const uint64_t m = __ballot(in);
                const uint32_t at = nin + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                if (in && at < kWinSlots) put(key, at);
                nin += (uint32_t)__popcll(m);
                nup += (uint32_t)__popcll(__ballot(e < hi && key >= khi));
            }
        }
        if (lane == 0) {
            ccnt[(uint64_t)r * U + u] = nin;
            cgt[(uint64_t)r * U + u] = nup;
            if (nin > kWinSlots) atomicOr(&overflow[r], 1u);
        }
        above += nup;
    }
    if (lane == 0 && above) atomicAdd(&s_above, above);
    __syncthreads();
    for (uint32_t i = tid; i < 2048u; i += 256u)
        if (s_h[i]) atomicAdd(&kw[kWinHist + i], s_h[i]);
    // (the list counters take the count above: a row has many workgroups)
    if (tid == 0 && s_above) atomicAdd(&kcnt[((uint64_t)r * kSub + blockIdx.x % kSub) * kCntStride], s_above);
    if (!last_of_row(kcnt, r, kTickGather, gridDim.x, &s_last)) return;
    uint32_t total, bin, rem;
    block_excl_scan(tid < kSub ? seen(&kcnt[((uint64_t)r * kSub + tid) * kCntStride]) : 0u, s_w, &total);
    __syncthreads();
    const bool ok = find_bin<2048>([&](uint32_t b) { return seen(&kw[kWinHist + b]); }, total < k ? k - total : 0u,
                                   &bin, &rem, s_w, s_res) &&
                    seen(&overflow[r]) == 0u;
    if (tid == 0) {
        st[r].prefix = ok ? klo + (bin << sh) : 0u;
        st[r].krem = ok ? rem : k;
        if (!ok) {
            st[r].exact = 1u;
            st[r].full = kPasses;
        }
    }
}

// K* and the ties needed from the keys of the part that holds it; a row
// without one starts its passes instead.
__global__ void __launch_bounds__(256) k_win_part(const float* x, uint64_t N, uint32_t U, RankState* st, uint32_t* hist,
                                                  const uint2* cand, const uint32_t* ccnt, uint32_t* klist,
                                                  uint32_t* kcnt)
{
    __shared__ uint32_t s_h[1024];
    __shared__ uint32_t s_w[4], s_res[2], s_last;
    const uint32_t r = blockIdx.y, tid = threadIdx.x, lane = tid & 63u;
    if (st[r].exact != 0u) return hist_pass<0>(x, N, st, hist, kcnt);
    // (the grid is the histogram's; the few keys here take 16 units a workgroup)
    const uint32_t nb = min(gridDim.x, min((U + 15u) / 16u, 256u));
    if (blockIdx.x >= nb) return;
    uint32_t* kw = klist + (uint64_t)r * kList;
    const uint32_t base = st[r].prefix, sh = kw[kWinState + 2u], width = 1u << sh;
    const uint64_t krem = st[r].krem;
    for (uint32_t i = tid; i < 1024u; i += 256u) s_h[i] = 0u;
    __syncthreads();
    constexpr uint32_t B = 4u;  // units of a wave in flight
    for (uint32_t u0 = (blockIdx.x * 4u + (tid >> 6)) * B; u0 < U; u0 += nb * 4u * B) {
        uint32_t n[B], key[B];
#pragma unroll
        for (uint32_t j = 0; j < B; ++j) n[j] = u0 + j < U ? ccnt[(uint64_t)r * U + u0 + j] : 0u;
#pragma unroll
        for (uint32_t j = 0; j < B; ++j)
            key[j] = lane < n[j] ? reinterpret_cast<const uint32_t*>(cand + ((uint64_t)r * U + u0 + j) * kSlots)[lane] : base - 1u;
#pragma unroll
        for (uint32_t j = 0; j < B; ++j)
            if (lane < n[j] && key[j] - base < width) {
                const uint32_t d = key[j] - base;
                if (sh <= 10u) {
                    atomicAdd(&s_h[d], 1u);
                } else {  // wider than a histogram (values sparse around K*): listed
                    const uint32_t at = atomicAdd(&kw[kWinState + 3u], 1u);
                    if (at < kWinList)
                        __hip_atomic_store(&kw[kWinWords + at], d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
    }
    __syncthreads();
    for (uint32_t i = tid; i < 1024u; i += 256u)
        if (s_h[i]) atomicAdd(&kw[kWinPart + i], s_h[i]);
    if (!last_of_row(kcnt, r, kTickPart, nb, &s_last)) return;
    uint32_t bin, rem;
    if (sh <= 10u) {
        find_bin<1024>([&](uint32_t b) { return seen(&kw[kWinPart + b]); }, krem, &bin, &rem, s_w, s_res);
    } else {
        // the part's keys, from the list or, if it was full, from the units
        const uint32_t nl = seen(&kw[kWinState + 3u]);
        auto for_part = [&](auto&& f) {
            if (nl <= kWinList) {
                for (uint32_t i = tid; i < nl; i += 256u) f(seen(&kw[kWinWords + i]));
            } else {
                for (uint64_t i = tid; i < (uint64_t)U * kWinSlots; i += 256u) {
                    const uint64_t u = (uint64_t)r * U + i / kWinSlots;
                    if ((uint32_t)(i % kWinSlots) >= ccnt[u]) continue;
                    const uint32_t d = reinterpret_cast<const uint32_t*>(cand + u * kSlots)[i % kWinSlots] - base;
                    if (d < width) f(d);
                }
            }
        };
        uint32_t hb;
        for_part([&](uint32_t d) { atomicAdd(&s_h[d >> 10], 1u); });  // (clear: sh > 10)
        __syncthreads();
        find_bin<1024>([&](uint32_t b) { return s_h[b]; }, krem, &hb, &rem, s_w, s_res);
        __syncthreads();
        for (uint32_t i = tid; i < 1024u; i += 256u) s_h[i] = 0u;
        __syncthreads();
        for_part([&](uint32_t d) {
            if (d >> 10 == hb) atomicAdd(&s_h[d & 1023u], 1u);
        });
        __syncthreads();
        const uint64_t left = rem;
        find_bin<1024>([&](uint32_t b) { return s_h[b]; }, left, &bin, &rem, s_w, s_res);
        bin |= hb << 10;
    }
    if (tid == 0) {
        st[r].prefix = base + bin;
        st[r].krem = rem;
        st[r].full = kWindowed;
    }
}

constexpr uint32_t kUPW = 8;  // units per wave in the count and write kernels

// Unit offsets: equal keys are taken in index order until `need` of them.
__global__ void __launch_bounds__(1024) k_unit_scan(uint32_t U, const RankState* st, const uint32_t* cnt, uint32_t* beq,
                                                    uint32_t* bout)
{
    __shared__ uint32_t s_w[16];
    const uint32_t r = blockIdx.x;
    const uint64_t need = st[r].krem;
    const uint32_t per = (U + 1023) / 1024;
    const uint32_t lo = min(threadIdx.x * per, U), hi = min(lo + per, U);
    const uint32_t* c = cnt + (uint64_t)r * U;
    auto g_of = [](uint32_t v) { return v & 0xFFFFu; };
    auto q_of = [](uint32_t v) { return v >> 16; };
    // the first kScanPer of a thread's units read at once (all of them at the
    // common sizes), the rest in turn
    constexpr uint32_t kScanPer = 8;
    const uint32_t h8 = min(hi, lo + kScanPer);
    uint32_t gv[kScanPer], qv[kScanPer];
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) {
        const uint32_t v = lo + j < h8 ? c[lo + j] : 0u;
        gv[j] = g_of(v);
        qv[j] = q_of(v);
    }
    uint32_t seq = 0;
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) seq += qv[j];
    for (uint32_t i = h8; i < hi; ++i) seq += q_of(c[i]);
    uint32_t tot;
    uint32_t run_eq = block_excl_scan(seq, s_w, &tot);
    // selections of a unit: its keys above K*, and its ties while needed
    auto take = [&](uint32_t re, uint32_t gi, uint32_t qi) {
        return gi + (re >= need ? 0u : (uint32_t)min<uint64_t>(need - re, qi));
    };
    uint32_t ssel = 0;
    {
        uint32_t re = run_eq;
#pragma unroll
        for (uint32_t j = 0; j < kScanPer; ++j) {
            ssel += take(re, gv[j], qv[j]);
            re += qv[j];
        }
        for (uint32_t i = h8; i < hi; ++i) {
            const uint32_t v = c[i];
            ssel += take(re, g_of(v), q_of(v));
            re += q_of(v);
        }
    }
    uint32_t run_out = block_excl_scan(ssel, s_w, &tot);
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; ++j) {
        if (lo + j < h8) {
            beq[(uint64_t)r * U + lo + j] = run_eq;
            bout[(uint64_t)r * U + lo + j] = run_out;
        }
        run_out += take(run_eq, gv[j], qv[j]);
        run_eq += qv[j];
    }
    for (uint32_t i = h8; i < hi; ++i) {
        beq[(uint64_t)r * U + i] = run_eq;
        bout[(uint64_t)r * U + i] = run_out;
        const uint32_t v = c[i];
        run_out += take(run_eq, g_of(v), q_of(v));
        run_eq += q_of(v);
    }
}

// Per unit: entries with key > K* (low half; at most 4096) and key == K*.  A
// wave takes kUPW consecutive units: from the gathered entries on a settled row
// (all loads in flight together), or the window's keys and the count above it,
// from the data on a row refined over it.
__global__ void __launch_bounds__(256) k_count(const float* x, uint64_t N, uint32_t U, const RankState* st,
                                                const uint2* cand, const uint32_t* ccnt, const uint32_t* cgt, uint32_t* cnt)
{
    const uint32_t r = blockIdx.y, lane = threadIdx.x & 63;
    const uint32_t u0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kUPW;
    const uint32_t K = st[r].prefix, full = st[r].full;
    if (full != kPasses) {
        const bool win = full == kWindowed;
        uint32_t n[kUPW], key[kUPW], up[kUPW], mine = 0u;
#pragma unroll
        for (uint32_t j = 0; j < kUPW; ++j) {
            n[j] = u0 + j < U ? ccnt[(uint64_t)r * U + u0 + j] : 0u;
            up[j] = win && u0 + j < U ? cgt[(uint64_t)r * U + u0 + j] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < kUPW; ++j) {
            const uint32_t* cu = reinterpret_cast<const uint32_t*>(cand + ((uint64_t)r * U + u0 + j) * kSlots);
            key[j] = lane < n[j] ? cu[win ? lane : 2u * lane + 1u] & 0x7FFFFFFFu : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < kUPW; ++j) {
            const uint32_t g = (uint32_t)__popcll(__ballot(lane < n[j] && key[j] > K));
            const uint32_t q = (uint32_t)__popcll(__ballot(lane < n[j] && key[j] == K));
            mine = lane == j ? g + up[j] | q << 16 : mine;
        }
        if (lane < kUPW && u0 + lane < U) cnt[(uint64_t)r * U + u0 + lane] = mine;
    } else {
        const float* row = x + (uint64_t)r * N;
        const bool vec = (reinterpret_cast<uintptr_t>(row) & 15u) == 0u;
        for (uint32_t u = u0; u < min(u0 + kUPW, U); ++u) {
            const uint64_t lo = (uint64_t)u * kUnit, hi = min(lo + kUnit, N);
            uint32_t ge = 0;  // above K*, and equal to it in the high half
            auto one = [&](float v) {
                const uint32_t key = mag_key(v);
                ge += (key > K ? 1u : 0u) + (key == K ? 0x10000u : 0u);
            };
            if (vec && hi - lo == kUnit) {
                for (uint32_t q0 = 0; q0 < kUnit / 256; q0 += 4u) {
                    float4 vs[4];
#pragma unroll
                    for (uint32_t q = 0; q < 4u; ++q)
                        vs[q] = *reinterpret_cast<const float4*>(row + lo + 256u * (q0 + q) + 4u * lane);
#pragma unroll
                    for (uint32_t q = 0; q < 4u; ++q) {
                        one(vs[q].x);
                        one(vs[q].y);
                        one(vs[q].z);
                        one(vs[q].w);
                    }
                }
            } else {
#pragma unroll 8
                for (uint64_t e = lo + lane; e < hi; e += 64) one(row[e]);
            }
            const uint32_t all = wave_scan(ge);  // (at most 4096 each)
            if (lane == 63) cnt[(uint64_t)r * U + u] = all;
        }
    }
}

// One unit of a row refined over its data: the selection compacted in index
// order from the data itself.  Q float4 of a lane are in flight together.
template <uint32_t Q>
__device__ void write_unit(const float* x, uint64_t N, uint64_t k, uint32_t U, uint32_t r, uint32_t u,
                           const RankState* st, const uint32_t* beq, const uint32_t* bout, uint32_t* out_idx,
                           float* out_val, float* residual)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t K = st[r].prefix;
    const uint64_t need = st[r].krem;
    const float* row = x + (uint64_t)r * N;
    float* res = residual ? residual + (uint64_t)r * N : nullptr;
    const bool inplace = res == row;
    uint32_t* oi = out_idx + (uint64_t)r * k;
    float* ov = out_val + (uint64_t)r * k;
    uint64_t eq_run = beq[(uint64_t)r * U + u];
    uint32_t out_run = bout[(uint64_t)r * U + u];
    const uint64_t lo = (uint64_t)u * kUnit, hi = min(lo + kUnit, N);
    const uint64_t lt = (1ull << lane) - 1ull;
    const bool res_vec = res == nullptr || inplace || (reinterpret_cast<uintptr_t>(res) & 15u) == 0u;
    if ((reinterpret_cast<uintptr_t>(row) & 15u) == 0u && res_vec && hi - lo == kUnit) {
        // Per 256 elements (lane i: elements 4i..4i+3) selections are placed in
        // index order by wave scans of the per-lane counts, two of them a scan
        // (its halves); ties are ranked only where there are any.
        static_assert(Q % 2u == 0u && Q <= 16u && 16u % Q == 0u, "pairs, in a 64-bit word of flags");
#pragma unroll 1
        for (uint32_t q0 = 0; q0 < kUnit / 256; q0 += Q) {
            const uint64_t e0 = lo + 256u * q0 + 4u * lane;
            float4 vs[Q];
#pragma unroll
            for (uint32_t q = 0; q < Q; ++q) vs[q] = *reinterpret_cast<const float4*>(row + e0 + 256u * q);
            uint64_t sel = 0u, tie = 0u;  // bit k of nibble q: element e0 + 256q + k
#pragma unroll
            for (uint32_t q = 0; q < Q; ++q) {
                const float v4[4] = {vs[q].x, vs[q].y, vs[q].z, vs[q].w};
                uint32_t s4 = 0u, t4 = 0u;
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) {
                    const uint32_t key = mag_key(v4[i]);
                    s4 |= key > K ? 1u << i : 0u;
                    t4 |= key == K ? 1u << i : 0u;
                }
                sel |= (uint64_t)s4 << (4u * q);
                tie |= (uint64_t)t4 << (4u * q);
            }
            if (__ballot(tie != 0u)) {
#pragma unroll 1
                for (uint32_t q = 0; q < Q; ++q) {
                    const uint32_t t4 = (uint32_t)(tie >> (4u * q)) & 15u;
                    const uint32_t n = (uint32_t)__popc(t4), incl = wave_scan(n);
                    uint64_t eb = eq_run + (incl - n);  // ties before this lane's first
                    uint32_t s4 = 0u;
                    for (uint32_t m = t4; m && eb < need; m &= m - 1u, ++eb) s4 |= m & (0u - m);
                    sel |= (uint64_t)s4 << (4u * q);
                    eq_run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < Q; q += 2u) {
                const uint32_t f2 = (uint32_t)(sel >> (4u * q)) & 0xFFu;
                const uint32_t n = (uint32_t)__popc(f2 & 15u) | (uint32_t)__popc(f2 >> 4) << 16;
                const uint32_t incl = wave_scan(n), all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63), ex = incl - n;
                uint32_t at[2] = {out_run + (ex & 0xFFFFu), out_run + (all & 0xFFFFu) + (ex >> 16)};
                out_run += (all & 0xFFFFu) + (all >> 16);
#pragma unroll
                for (uint32_t h = 0; h < 2u; ++h) {
                    const uint64_t e = e0 + 256u * (q + h);
                    const uint32_t f4 = f2 >> (4u * h) & 15u;
                    const float v4[4] = {vs[q + h].x, vs[q + h].y, vs[q + h].z, vs[q + h].w};
#pragma unroll
                    for (uint32_t i = 0; i < 4u; ++i) {
                        if (f4 >> i & 1u) {
                            oi[at[h]] = (uint32_t)(e + i);
                            ov[at[h]++] = v4[i];
                            if (inplace) res[e + i] = 0.0f;
                        }
                    }
                    if (res && !inplace)
                        *reinterpret_cast<float4*>(res + e) =
                            make_float4(f4 & 1u ? 0.0f : v4[0], f4 & 2u ? 0.0f : v4[1], f4 & 4u ? 0.0f : v4[2],
                                        f4 & 8u ? 0.0f : v4[3]);
                }
            }
        }
        return;
    }
    for (uint64_t e8 = lo; e8 < hi; e8 += 512) {  // (eight loads in flight)
        float v8[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v8[q] = e8 + 64u * q + lane < hi ? row[e8 + 64u * q + lane] : 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint64_t e = e8 + 64u * q + lane;
            const bool valid = e < hi;
            const float v = v8[q];
            const uint32_t key = mag_key(v);
            const bool eq = valid && key == K;
            const uint64_t beq_w = __ballot(eq);
            const bool take_eq = eq && (eq_run + (uint64_t)__popcll(beq_w & lt)) < need;
            const bool sel = (valid && key > K) || take_eq;
            const uint64_t bsel = __ballot(sel);
            if (sel) {
                const uint32_t o = out_run + (uint32_t)__popcll(bsel & lt);
                oi[o] = (uint32_t)e;
                ov[o] = v;
            }
            if (res && valid) {
                if (inplace) {
                    if (sel) res[e] = 0.0f;
                } else {
                    res[e] = sel ? 0.0f : v;
                }
            }
            eq_run += (uint64_t)__popcll(beq_w);
            out_run += (uint32_t)__popcll(bsel);
        }
    }
}

// Per UPW units of a wave: a row settled by its gathered entries writes
// its selection from them (a unit's entries in index order, one per lane):
// key > K*, or key == K* while ties are still needed, at the unit's offset,
// zeroing the residual there; a row refined over its data compacts it.
template <uint32_t UPW>
__global__ void __launch_bounds__(256) k_write(const float* x, uint64_t N, uint64_t k, uint32_t U,
                                               const RankState* st, const uint2* cand, const uint32_t* ccnt,
                                               const uint32_t* beq, const uint32_t* bout, uint32_t* out_idx,
                                               float* out_val, float* residual)
{
    const uint32_t r = blockIdx.y, lane = threadIdx.x & 63;
    const uint32_t u0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * UPW;
    if (u0 >= U) return;
    if (st[r].full != kGathered) {
        for (uint32_t u = u0; u < min(u0 + UPW, U); ++u)
            write_unit<UPW == 1u ? 16u : 4u>(x, N, k, U, r, u, st, beq, bout, out_idx, out_val, residual);
        return;
    }
    const uint32_t K = st[r].prefix;
    const uint64_t need = st[r].krem;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint32_t n[UPW], eqb[UPW], ob[UPW];
    uint2 c[UPW];
#pragma unroll
    for (uint32_t j = 0; j < UPW; ++j) {
        const bool in = u0 + j < U;
        n[j] = in ? ccnt[(uint64_t)r * U + u0 + j] : 0u;  // <= kSlots on a settled row
        eqb[j] = in ? beq[(uint64_t)r * U + u0 + j] : 0u;
        ob[j] = in ? bout[(uint64_t)r * U + u0 + j] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < UPW; ++j)
        c[j] = lane < n[j] ? cand[((uint64_t)r * U + u0 + j) * kSlots + lane] : make_uint2(0u, 0u);
#pragma unroll
    for (uint32_t j = 0; j < UPW; ++j) {
        const uint32_t key = c[j].y & 0x7FFFFFFFu;
        const bool eq = lane < n[j] && key == K;
        const uint64_t beq_w = __ballot(eq);
        const bool sel = (lane < n[j] && key > K) || (eq && (uint64_t)eqb[j] + (uint64_t)__popcll(beq_w & lt) < need);
        const uint64_t bsel = __ballot(sel);
        if (sel) {
            const uint64_t o = (uint64_t)r * k + ob[j] + (uint32_t)__popcll(bsel & lt);
            out_idx[o] = c[j].x;
            out_val[o] = __uint_as_float(c[j].y);
            if (residual) residual[(uint64_t)r * N + c[j].x] = 0.0f;
        }
    }
}

struct TLayout {
    RankState* st;
    uint32_t *hist, *cgt, *cnt, *beq, *bout, *ccnt, *overflow, *klist, *kcnt;
    uint2* cand;
    uint32_t U;
    size_t bytes;
};

TLayout tlayout(int P, uint64_t N, void* ws)
{
    Carve c(ws);
    TLayout l{};
    l.U = (uint32_t)((N + kUnit - 1) / kUnit);
    l.st = c.take<RankState>(P);
    l.overflow = c.take<uint32_t>(P);
    l.kcnt = c.take<uint32_t>((size_t)P * kSub * kCntStride);
    l.klist = c.take<uint32_t>((size_t)P * kList);
    l.ccnt = c.take<uint32_t>((size_t)P * l.U);
    l.cand = c.take<uint2>((size_t)P * l.U * kSlots);
    l.hist = c.take<uint32_t>((size_t)P * 2048);
    l.cgt = c.take<uint32_t>((size_t)P * l.U);
    l.cnt = c.take<uint32_t>((size_t)P * l.U);
    l.beq = c.take<uint32_t>((size_t)P * l.U);
    l.bout = c.take<uint32_t>((size_t)P * l.U);
    l.bytes = align_up(c.used, 256);
    return l;
}

}  // namespace

size_t topk_workspace(int P, uint64_t N, uint64_t /*k*/) { return tlayout(P, N, nullptr).bytes; }

hipError_t topk_run(int P, const float* x, uint64_t N, uint64_t k, uint32_t* out_idx,
                    float* out_val, float* residual, void* ws, hipStream_t s)
{
    if (k == 0) {
        if (residual && residual != x)
            return hipMemcpyAsync(residual, x, (size_t)P * N * sizeof(float), hipMemcpyDeviceToDevice, s);
        return hipSuccess;
    }
    const TLayout l = tlayout(P, N, ws);
    // The expected selections per unit decide where a row starts: up to a
    // quarter of what a unit gathers (of long rows a little more: 64 rows of 2^20,
    // 9 a unit: 156 us, through the window 274), with a gather (its entries, a few
    // times the selections, are then the only ones read again); up to a quarter of
    // the elements, long rows with a window; above, where a window of the sample's
    // accuracy could fill a unit's slots, and short rows with the passes over the
    // data: a window costs each row 140 KB of histograms, the passes three more
    // reads of it (41 a unit, us, window and passes: one row of 2^16 55, 43; of 2^20
    // 61, 51; of 2^22 65, 89; 8 rows of 2^20 82, 62; 64 rows of 2^12 58, 35; of 2^18
    // 128, 98; of 2^20 276, 309; 512 rows of 2^16 440, 169; 4096 of 2^12 648, 156).
    const double per_unit = (double)k * kUnit / (double)N;
    const bool gather = per_unit <= (N >= 1u << 18 ? 9.25 : 8.0);
    const bool wide = N >= 1u << 21 || (N >= 1u << 20 && (uint64_t)P * N >= 1u << 26);
    const bool win = !gather && wide && per_unit <= kUnit / 4, passes = !gather && !win;
    static_assert(kSlots == 32 && kUnit == 4096, "the lines above");
    const uint64_t ninit = (uint64_t)P * (win ? kWinWords : 2048u);
    hipLaunchKernelGGL(k_init, dim3((uint32_t)std::min<uint64_t>((ninit + 255) / 256, 1024)), dim3(256), 0, s, l.st,
                       (uint32_t)P, k, l.hist, l.overflow, l.kcnt, l.klist, win ? 1u : 0u, passes ? 1u : 0u);
    // Workgroups of a row: few rows share the chip (one row's histogram from
    // 64 workgroups took 75 us for 94 MB).
    auto blocks = [&](uint64_t work, uint32_t least, uint32_t chip) {
        return (uint32_t)std::min<uint64_t>(work, std::max<uint32_t>(least, chip / (uint32_t)P));
    };
    const dim3 hgrid(blocks((N + 4095) / 4096, kHistBlocksPerRank, 1024), P), ugrid((l.U + 3) / 4, P);
    // sample: every stride-th 256-element segment, about kSampleSegs or kWinSegs of them
    const uint64_t nseg = (N + 255) / 256;
    const uint64_t stride = std::max<uint64_t>(1, nseg / (win ? kWinSegs : kSampleSegs)), nsam = (nseg + stride - 1) / stride;
    // (only the row's last segment may be short)
    const uint64_t sampled = nsam * 256 - ((nsam - 1) * stride == nseg - 1 ? nseg * 256 - N : 0);
    const double frac = (double)sampled / (double)N;
    timer_begin(kTTopkSelect, s);
    if (win) {
        hipLaunchKernelGGL(k_win_sample, dim3(blocks((nsam + 15) / 16, 8, 64), P), dim3(1024), 0, s, x, N,
                           (uint32_t)stride, k, frac, l.st, l.klist, l.kcnt);
        hipLaunchKernelGGL(k_win_gather, dim3(blocks((l.U + 3) / 4, 64, 2048), P), dim3(256), 0, s, x, N, k, l.U, l.st,
                           l.cand, l.ccnt, l.cgt, l.overflow, l.klist, l.kcnt);
        hipLaunchKernelGGL(k_win_part, hgrid, dim3(256), 0, s, x, N, l.U, l.st, l.hist, l.cand, l.ccnt, l.klist,
                           l.kcnt);
    } else if (!passes) {
        hipLaunchKernelGGL(k_sample, dim3((uint32_t)std::min<uint64_t>(64, nsam), P), dim3(256), 0, s, x, N,
                           (uint32_t)stride, l.hist);
        hipLaunchKernelGGL(k_estimate, dim3(P), dim3(256), 0, s, l.st, l.hist, k, frac);
        hipLaunchKernelGGL(k_gather, ugrid, dim3(256), 0, s, x, N, l.U, l.st, l.cand, l.ccnt, l.overflow,
                           residual, 0u, l.klist, l.kcnt);
        // settles the rows whose sampled bin held; the others go exact
        hipLaunchKernelGGL(k_cand_select, dim3(P), dim3(1024), 0, s, k, l.st, l.klist, l.kcnt, l.overflow, 0u);
    }
    // rows on the exact path: the exact boundary bin, and a gather from it
    // where one was tried
    if (!win) hipLaunchKernelGGL(k_hist<0>, hgrid, dim3(256), 0, s, x, N, l.st, l.hist, l.kcnt);
    if (!win && !passes) {
        const dim3 xgrid(std::min<uint32_t>((l.U + 3) / 4, kExactGatherBlocks), P);
        hipLaunchKernelGGL(k_gather, xgrid, dim3(256), 0, s, x, N, l.U, l.st, l.cand, l.ccnt, l.overflow,
                           residual, 1u, l.klist, l.kcnt);
        hipLaunchKernelGGL(k_cand_select, dim3(P), dim3(1024), 0, s, k, l.st, l.klist, l.kcnt, l.overflow, 1u);
    }
    // rows refined over their data (the others return at once)
    hipLaunchKernelGGL(k_hist<1>, hgrid, dim3(256), 0, s, x, N, l.st, l.hist, l.kcnt);
    hipLaunchKernelGGL(k_hist<2>, hgrid, dim3(256), 0, s, x, N, l.st, l.hist, l.kcnt);
    timer_end(kTTopkSelect, s);
    timer_begin(kTTopkWrite, s);
    const dim3 wgrid((l.U + 4 * kUPW - 1) / (4 * kUPW), P);
    hipLaunchKernelGGL(k_count, wgrid, dim3(256), 0, s, x, N, l.U, l.st, l.cand, l.ccnt, l.cgt, l.cnt);
    hipLaunchKernelGGL(k_unit_scan, dim3(P), dim3(1024), 0, s, l.U, l.st, l.cnt, l.beq, l.bout);
    if (win || passes)
        hipLaunchKernelGGL(k_write<1>, ugrid, dim3(256), 0, s, x, N, k, l.U, l.st, l.cand, l.ccnt, l.beq, l.bout, out_idx,
                           out_val, residual);
    else
        hipLaunchKernelGGL(k_write<kUPW>, wgrid, dim3(256), 0, s, x, N, k, l.U, l.st, l.cand, l.ccnt,
                           l.beq, l.bout, out_idx, out_val, residual);
    timer_end(kTTopkWrite, s);
    return hipGetLastError();
}

}  // namespace sparcml
