// Sparse allreduce of P sparse streams on one gfx950 GPU: the local
// reduction work of SparCML's recursive-doubling sparse allreduce (§5.3.1,
// Fig. 2) with the sparse->dense switch of §5.1.
//
// Design (why it differs from a level-by-level merge): every rank's stream
// lives in HBM, so instead of materialising the P-1 intermediate streams of
// the tree (which moves log2(P) times the data), the coordinate space is cut
// into tiles and each tile evaluates the whole tree at once in LDS (accum.h):
// the streams are read once and the root is written once.
//
//  * two ranks need one addition, the same in either order; the tree over all
//    P slots with -0.0 where a rank holds nothing rounds as recursive doubling
//    over the ranks present;
//  * a dense node's value at an index equals the tree sum (+0.0 where no rank
//    contributes), so a dense root is written tile by tile, once;
//  * the switch rule needs the exact union size of every node only where the
//    root's own union U leaves it open: U > thr makes the root dense (its two
//    children hold at least U together), 2 U <= thr keeps every node sparse
//    (no two children hold more than 2 U).
//
// Passes, none of which waits for the host: partition (per-chunk stream
// offsets; where a stream lies unevenly over the chunks, the workgroups of the
// passes below take ranges of equal weight instead) -> dense pass, when the
// streams hold more than thr entries together (with the node sizes if the
// caller wants them and the streams meet often), else a counting pass -> a pass
// for the node sizes, from the indices alone or in tiles: where the caller
// wants them, or, after a dense pass, returning at once unless thr/2 < U <= thr
// -> sparse output, which applies the rule, reports the header and the nodes,
// and returns at once if the root is dense.  All-sparse inputs of up to 64
// slots and 2^21 entries go to the merge tree (merge.hip).
#include "internal.h"

#include "accum.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstddef>
#include <cstring>

namespace sparcml {
namespace {

__device__ __forceinline__ uint32_t lower_bound(const uint32_t* a, uint32_t lo, uint32_t hi,
                                                uint64_t x)
{
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if ((uint64_t)a[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// ------------------------------------------------------------------------
// Stream r's descriptor from the launch's arguments (fmt != kDescNone).
static_assert(sizeof(StreamDesc) == 48 && offsetof(StreamDesc, idx) == 0 && offsetof(StreamDesc, val) == 8 &&
                  offsetof(StreamDesc, qval) == 16 && offsetof(StreamDesc, qscale) == 24 &&
                  offsetof(StreamDesc, nnz) == 32,
              "descriptor words");
__device__ __forceinline__ StreamDesc arg_desc(const DescArgs& tb, uint32_t r)
{
    auto word2 = [&](uint32_t i) -> uint64_t { return (uint64_t)tb.words[i] | (uint64_t)tb.words[i + 1] << 32; };
    StreamDesc d{};
    if (tb.fmt == kDescFull) {
        const uint32_t b = r * (uint32_t)(sizeof(StreamDesc) / 4);
        d.idx = reinterpret_cast<const uint32_t*>(word2(b));
        d.val = reinterpret_cast<const float*>(word2(b + 2u));
        d.qval = reinterpret_cast<const uint8_t*>(word2(b + 4u));
        d.qscale = reinterpret_cast<const float*>(word2(b + 6u));
        d.nnz = word2(b + 8u);
    } else {
        const uint32_t b = r * 5u;
        d.idx = reinterpret_cast<const uint32_t*>(word2(b));
        if (tb.fmt == kDescCodes) {
            d.qval = reinterpret_cast<const uint8_t*>(word2(b + 2u));
            d.qscale = tb.scale0 + r;
        } else {
            d.val = reinterpret_cast<const float*>(word2(b + 2u));
        }
        d.nnz = tb.words[b + 4u];
    }
    return d;
}

// Per-chunk start offsets of every stream and zeroing of the counters the
// passes accumulate into; workgroup r takes stream r.  A sample of the
// stream (every stride-th index, at most kPartSamples, read at once) narrows
// each chunk start's search to one stride of positions, so a search waits on
// about half the dependent loads of a binary search over the whole stream.
// When the descriptors travel in the arguments this launch also stores them
// to `tab` for the later passes, and reads its own from the arguments.
constexpr uint32_t kPartSamples = 1024;
constexpr uint32_t kPartThreads = 256;
__global__ void __launch_bounds__(kPartThreads) k_partition(StreamDesc* tab, DescArgs tb, uint32_t* off, uint32_t nchunks,
                                                   uint64_t chunk_coords, uint64_t lo, uint64_t N, uint32_t* zero,
                                                   uint32_t nzero, ReduceResult* hdr, ReduceResult* res,
                                                   uint32_t qbits, uint32_t* pad, uint32_t* none, uint32_t* odd)
{
    __shared__ uint32_t s_smp[kPartSamples], s_off[kSegMax + 1];
    const uint32_t r = blockIdx.x, tid = threadIdx.x;
    if (r == 0) {
        for (uint32_t i = tid; i < nzero; i += blockDim.x) zero[i] = 0u;
        for (uint32_t i = tid; i < kVoid; i += blockDim.x) none[i] = 0xFFFFFFFFu;
        if (tid == 0) {  // error bits of the root's headers
            hdr->pad = 0u;
            if (res) res->pad = 0u;
        }
    }
    StreamDesc d = tb.fmt != kDescNone ? arg_desc(tb, r) : tab[r];
    // The tile pass loads codes as words inside the stream's array: one
    // shorter than a word moves to `pad`.
    const uint32_t per = qbits ? 8u / qbits : 1u, bytes = (uint32_t)((d.nnz + per - 1u) / per);
    const bool tiny = qbits && d.nnz && bytes < 4u;
    if (tid == 0 && (tb.fmt != kDescNone || tiny)) {
        if (tiny) {
            uint32_t w = 0u;
            for (uint32_t i = 0; i < bytes; ++i) w |= (uint32_t)d.qval[i] << (8u * i);
            pad[r] = w;
            d.qval = reinterpret_cast<const uint8_t*>(pad + r);
        }
        tab[r] = d;
    }
    const uint32_t* const idx = d.idx;
    const uint32_t nnz = (uint32_t)d.nnz;
    // samples j < ns: the index at position j * stride
    const uint32_t stride = nnz > kPartSamples ? (uint32_t)(((uint64_t)nnz + kPartSamples - 1u) / kPartSamples) : 1u;
    const uint32_t ns = (uint32_t)(((uint64_t)nnz + stride - 1u) / stride);
    for (uint32_t j = tid; j < ns; j += blockDim.x) s_smp[j] = idx[(uint64_t)j * stride];
    __syncthreads();
    uint32_t* const o = off + (uint64_t)r * (nchunks + 1u);
    for (uint32_t c = tid; c <= nchunks; c += blockDim.x) {
        uint32_t res = nnz;
        if (c < nchunks) {
            const uint64_t x = lo + min((uint64_t)c * chunk_coords, N);
            // js samples lie below x: the first position at or past x is
            // above sample js - 1's and at most sample js's
            uint32_t a = 0u, b = ns;
            while (a < b) {
                const uint32_t m = a + ((b - a) >> 1);
                if ((uint64_t)s_smp[m] < x) a = m + 1u;
                else b = m;
            }
            const uint32_t pa = a ? (a - 1u) * stride + 1u : 0u;
            const uint32_t pb = (uint32_t)min((uint64_t)a * stride, (uint64_t)nnz);
            res = lower_bound(idx, min(pa, pb), pb, x);
        }
        o[c] = res;
        s_off[c] = res;
    }
    __syncthreads();
    static_assert(kPartThreads == 256u, "four waves, four bytes");
    // Whether a chunk holds far more of the stream than the others (never, of
    // an evenly drawn one: half of the mean and 64 are six deviations or more)
    const uint32_t most = nnz / nchunks + nnz / nchunks / 2u + 64u;
    bool far = false;
    for (uint32_t c = tid; c < nchunks; c += blockDim.x) far |= s_off[c + 1u] > s_off[c] && s_off[c + 1u] - s_off[c] > most;
    // (a byte of the stream's word a wave: no further barrier)
    const bool any = __ballot(far) != 0u;
    if ((tid & 63u) == 0u) reinterpret_cast<uint8_t*>(odd + r)[tid >> 6] = any ? 1 : 0;
}

// Per-segment start offsets of every stream by one pass over its entries,
// for the merge path (whose inputs are few: a pass reads less than the
// searches wait for), and zeroing of that path's counters; the descriptor
// table as in k_partition.  Segment s of the range starts at index
// lo + s segw; for an ascending stream, off[s] = the first position whose
// index is at least that start, so entry e is the offset of every segment
// s with k(idx[e - 1]) <= s < k(idx[e]), where k(x) counts the segment
// starts (of the first nseg) at or below x (k = 0 before the first entry,
// nseg + 1 past the last).  Grid: x over positions 0..nnz of a stream,
// y over streams.  A stream that does not ascend leaves some offsets
// unwritten: the merge path clamps every offset to its stream.
__global__ void k_partition_pass(StreamDesc* tab, DescArgs tb, uint32_t* off, uint32_t nseg, uint64_t segw,
                                 uint64_t lo, uint32_t* zero, uint32_t nzero)
{
    const uint32_t r = blockIdx.y, e = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0) {
        if (e < nzero) zero[e] = 0u;
        if (tb.fmt != kDescNone && e < gridDim.y) tab[e] = arg_desc(tb, e);
    }
    const uint32_t* idx;
    uint32_t nnz;
    if (tb.fmt != kDescNone) {
        const StreamDesc d = arg_desc(tb, r);
        idx = d.idx;
        nnz = (uint32_t)d.nnz;
    } else {
        idx = tab[r].idx;
        nnz = (uint32_t)tab[r].nnz;
    }
    if (e > nnz) return;
    auto k = [&](uint32_t x) -> uint32_t {
        if ((uint64_t)x < lo) return 0u;
        const uint64_t d = (uint64_t)x - lo;  // < 2^32
        const uint64_t q = segw - 1ull >= 0xFFFFFFFFull ? 0ull : (uint64_t)((uint32_t)d / (uint32_t)segw);
        return (uint32_t)min(q + 1ull, (uint64_t)nseg);
    };
    const uint32_t ka = e == 0u ? 0u : k(idx[e - 1u]);
    const uint32_t kb = e == nnz ? nseg + 1u : k(idx[e]);
    uint32_t* o = off + (size_t)r * (nseg + 1u);
    for (uint32_t s = ka; s < kb; ++s) o[s] = e;
}

__global__ void k_set_result(ReduceResult* r, uint64_t nnz, uint32_t dense)
{
    if (threadIdx.x == 0) *r = ReduceResult{nnz, dense, 0u};
}

// Compute units of the current device (256 without one): the tile pass runs
// one workgroup on each, so that its grid is a single wave of equal chunks.
uint32_t compute_units()
{
    // per device; 0 = not queried yet (a race between threads only stores the
    // same value twice)
    constexpr int kCacheDevs = 64;
    static std::atomic<uint32_t> cache[kCacheDevs];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 256u;
    }
    std::atomic<uint32_t>* slot = dev >= 0 && dev < kCacheDevs ? &cache[dev] : nullptr;
    if (slot) {
        const uint32_t v = slot->load(std::memory_order_relaxed);
        if (v) return v;
    }
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
        (void)hipGetLastError();
        return 256u;
    }
    const uint32_t n = std::min<uint32_t>((uint32_t)cus, kSegMax);  // the offsets' space holds kSegMax chunks
    if (slot) slot->store(n, std::memory_order_relaxed);
    return n;
}

struct Layout {
    StreamDesc* tab;
    uint32_t *off, *zero, *node_cnt, *odd, *chunk_ne, *pad, *none;
    ReduceResult* hdr;
    size_t bytes;
};

Layout layout(const ReducePlan& p, void* ws)
{
    Carve c(ws);
    Layout l;
    l.tab = c.take<StreamDesc>(p.P);
    // stream offsets at the tile pass's chunks, or at the merge path's
    // segments; counters zeroed by the partition launch (either path's)
    l.off = c.take<uint32_t>((size_t)p.P * (kSegMax + 1));
    l.zero = c.take<uint32_t>(std::max<size_t>((size_t)p.P + 1, kSegStateWords + 2 * (size_t)kSegMax));
    l.node_cnt = l.zero;
    // behind the node counters (at most 255) a word a stream, and the union
    // sizes of the chunks
    l.odd = l.zero ? l.zero + 256 : nullptr;
    l.chunk_ne = l.zero ? l.zero + 512 : nullptr;
    // and a word per stream for codes of less than one
    l.pad = l.zero ? l.zero + 512 + kSegMax : nullptr;
    // and what empty slots read
    l.none = l.pad ? l.pad + 256 : nullptr;
    static_assert(512 + kSegMax + 256 + kVoid <= kSegStateWords + 2 * kSegMax, "they fit the counters' space");
    // (Three words per 2048 or 4096 indices are reserved and not used: the
    // size a caller is asked for, and with it what the allocation-free entry
    // point takes and refuses, is part of the interface.)
    const uint64_t T = p.P <= 32 ? 2048 : 4096, ntiles = (p.N + T - 1) / T;
    for (int i = 0; i < 3; ++i) c.take<uint32_t>(ntiles);
    l.hdr = c.take<ReduceResult>(1);
    l.bytes = align_up(c.used, 256);
    return l;
}

}  // namespace

int reduce_plan(int P, uint64_t N, uint64_t max_nnz, uint64_t sum_nnz, double delta, int qbits,
                ReducePlan* plan, uint64_t lo)
{
    ReducePlan p{};
    p.lo = lo;
    p.P = (uint32_t)P;
    p.L = 0;
    while ((1u << p.L) < p.P) ++p.L;
    p.N = N;
    // One chunk per compute unit, a multiple of 64 indices and at least 256
    // (a tile's fixed cost is a few microseconds, whatever its width).
    const uint64_t ncu = compute_units();
    p.chunk = std::max<uint64_t>(((N + ncu - 1) / ncu + 63) & ~63ull, 256);
    p.nchunks = (uint32_t)((N + p.chunk - 1) / p.chunk);
    const double t = std::floor(delta * (double)N);
    p.thr = t >= 18446744073709551615.0 ? UINT64_MAX : (uint64_t)t;
    p.sum_nnz = sum_nnz;
    p.max_nnz = max_nnz;
    p.qbits = (uint32_t)qbits;
    p.speculate_dense = sum_nnz > p.thr ? 1 : 0;
    p.small = merge_small_fits(p.P, sum_nnz, p.thr) ? 1 : 0;
    p.seg = !p.small && merge_seg_fits(p.P, sum_nnz, p.thr) ? 1 : 0;
    p.nseg = 0;
    p.segw = 0;
    if (p.seg) merge_seg_shape(N, sum_nnz, &p.nseg, &p.segw);
    *plan = p;
    return 0;
}

size_t reduce_workspace(const ReducePlan& p) { return layout(p, nullptr).bytes; }

hipError_t set_result_run(ReduceResult* r, uint64_t nnz, uint32_t dense, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_result, dim3(1), dim3(64), 0, s, r, nnz, dense);
    return hipGetLastError();
}

hipError_t reduce_run(const ReducePlan& p, const StreamDesc* host_tab, uint32_t* out_idx,
                      float* out_val, uint64_t* node_nnz, uint8_t* node_dense, void* ws,
                      hipStream_t s, ReduceResult* res, uint32_t nfold, ReduceResult* dev_result,
                      uint64_t out_cap)
{
    const Layout l = layout(p, ws);
    hipError_t e;
    if (p.small) {
        // few slots, every node sparse, few entries: one workgroup, one launch
        e = merge_small_run(p.P, p.L, p.qbits, nfold, host_tab, out_idx, out_val, node_nnz, node_dense, l.hdr,
                            dev_result, s);
        if (e != hipSuccess || dev_result) return e;
        if ((e = hipMemcpyAsync(res, l.hdr, sizeof(ReduceResult), hipMemcpyDeviceToHost, s)) != hipSuccess)
            return e;
        return hipStreamSynchronize(s);
    }
    // the descriptor table: in the partition launch's arguments when it fits
    // there (whole, or 5 words a stream when every stream's level unit
    // follows the previous one's), else uploaded first
    const size_t tab_bytes = sizeof(StreamDesc) * p.P;
    DescArgs tb;
    tb.nwords = 0;
    tb.fmt = kDescNone;
    tb.scale0 = nullptr;
    bool scales_follow = true;
    for (uint32_t r = 1; r < p.P && scales_follow; ++r) scales_follow = host_tab[r].qscale == host_tab[0].qscale + r;
    if (tab_bytes <= sizeof(tb.words)) {
        tb.fmt = kDescFull;
        tb.nwords = (uint32_t)(tab_bytes / 4);
        memcpy(tb.words, host_tab, tab_bytes);
    } else if (5u * p.P <= (uint32_t)kBlobWords && (!p.qbits || scales_follow)) {
        tb.fmt = p.qbits ? kDescCodes : kDescValues;
        tb.nwords = 5u * p.P;
        tb.scale0 = host_tab[0].qscale;
        for (uint32_t r = 0; r < p.P; ++r) {
            const uint64_t a = reinterpret_cast<uint64_t>(host_tab[r].idx);
            const uint64_t b = reinterpret_cast<uint64_t>(p.qbits ? static_cast<const void*>(host_tab[r].qval)
                                                                  : static_cast<const void*>(host_tab[r].val));
            uint32_t* w = tb.words + 5u * r;
            w[0] = (uint32_t)a;
            w[1] = (uint32_t)(a >> 32);
            w[2] = (uint32_t)b;
            w[3] = (uint32_t)(b >> 32);
            w[4] = (uint32_t)host_tab[r].nnz;
        }
    } else if ((e = upload(l.tab, host_tab, tab_bytes, s)) != hipSuccess) {
        return e;
    }
    // offsets of every stream at the tile pass's chunks (searches) or the
    // merge path's segments (one pass over the entries), and that path's
    // counters cleared
    if (p.seg) {
        const uint32_t nzero = kSegStateWords + 2u * p.nseg;
        const uint64_t nthreads = std::max<uint64_t>(p.max_nnz + 1u, std::max<uint32_t>(nzero, p.P));
        hipLaunchKernelGGL(k_partition_pass, dim3((uint32_t)((nthreads + 255) / 256), p.P), dim3(256), 0, s, l.tab,
                           tb, l.off, p.nseg, p.segw, p.lo, l.zero, nzero);
    } else {
        const uint32_t nzero = p.P;
        hipLaunchKernelGGL(k_partition, dim3(p.P), dim3(kPartThreads), 0, s, l.tab, tb, l.off, p.nchunks, p.chunk, p.lo,
                           p.N, l.zero, nzero, l.hdr, dev_result, p.qbits, l.pad, l.none, l.odd);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;

    if (p.seg) {
        // every node sparse: the merge tree, one workgroup per segment
        SegState st;
        st.node_cnt = l.zero;
        st.ticket = l.zero + 64;
        st.done = l.zero + 65;
        st.err = l.zero + 66;
        st.flags = reinterpret_cast<unsigned long long*>(l.zero + kSegStateWords);
        e = merge_seg_run(p.P, p.L, p.qbits, nfold, l.tab, l.off, st, p.nseg, p.lo, p.segw, p.N, out_idx,
                          out_val, node_nnz, node_dense, l.hdr, dev_result, merge_seg_short(p.sum_nnz, p.nseg), s);
        if (e != hipSuccess || dev_result) return e;
        if ((e = hipMemcpyAsync(res, l.hdr, sizeof(ReduceResult), hipMemcpyDeviceToHost, s)) != hipSuccess)
            return e;
        return hipStreamSynchronize(s);  // res->pad nonzero: a look-back gave up (the caller reports it)
    }

    AccArgs a{};
    a.tab = l.tab;
    a.off = l.off;
    a.chunk_ne = l.chunk_ne;
    a.node_cnt = l.node_cnt;
    a.none = l.none;
    a.odd = l.odd;
    for (uint64_t w = 2u * p.sum_nnz + p.N; w >> a.wshift >= 1ull << 31;) ++a.wshift;
    a.out_idx = out_idx;
    a.out_val = out_val;
    a.hdr = l.hdr;
    a.res = dev_result;
    a.node_nnz = node_nnz;
    a.node_dense = node_dense;
    a.N = p.N;
    a.thr = p.thr;
    a.chunk = p.chunk;
    a.P = p.P;
    a.L = p.L;
    a.nchunks = p.nchunks;
    a.qbits = p.qbits;
    a.lo = (uint32_t)p.lo;
    a.out_cap = (uint32_t)std::min<uint64_t>(out_cap, 0xFFFFFFFFull);
    a.nfold = nfold;
    a.out_vec = (reinterpret_cast<uintptr_t>(out_val) & 15u) == 0 ? 1u : 0u;
    const bool info = node_nnz || node_dense;
    const uint32_t pmax = std::max<uint32_t>(p.P, 16u), nb = acc_blocks(p.sum_nnz, p.N, p.P);
    // Tiles of equal width in every chunk, at most tmax wide and narrow enough
    // that a stream's entries usually fit one window of 64: a mean of 44 leaves
    // room for three standard deviations of a uniform stream; of streams of
    // many lengths the longest may have 52 (one window in 20 is continued; 48
    // ragged ranks of 2e7 with node sizes: 145 -> 137 us by the wider tiles).
    // Up to 16 slots a wave has one stream, and 15 waves of 16 may have none: there
    // a tile takes eight windows of it, the others read on together (2 and 8
    // ranks, 10% of 2^25, 4-bit codes: 540 -> 156 and 353 -> 175 us; two streams a
    // wave gain and lose alike, 32 ranks, 10% of 2^22: 91 -> 86, 2^20: 35 -> 40).
    const uint64_t live = std::max<uint64_t>(p.P / 2u + nfold, 1u), mean = (p.sum_nnz + live - 1u) / live;
    const uint64_t wide = p.P <= 16u ? 8u : 1u;
    auto shape = [&](uint32_t tmax) {
        const uint64_t fit = p.max_nnz ? std::min(44u * wide * p.N / mean, 52u * wide * p.N / p.max_nnz) : tmax;
        const uint64_t most = std::min<uint64_t>(tmax, std::max<uint64_t>(fit & ~63ull, 256));
        const uint64_t n = (p.chunk + most - 1) / most;
        a.T = (uint32_t)((((p.chunk + n - 1) / n) + 63) & ~63ull);
        // (a thread takes four indices of every 4096: tiles past that are whole
        // multiples, or the last few would cost as much)
        if (a.T > 4096u) a.T = std::min<uint32_t>((a.T + 4095u) & ~4095u, (uint32_t)most & ~4095u);
    };
    // Node sizes from the indices alone (a launch more, where a dense pass goes
    // before it), or in the tile pass: by the mean entries an index.  Dense root,
    // 2^25, us without and with: 2 ranks 0.25 294, 194; 16 ranks 0.5 340, 285 and
    // 2 688, 513; 32 ranks 0.1 77, 64 and 0.25 99, 152; 64 ranks 0.25 138, 115 and
    // 0.5 167, 191; 128 ranks 0.25 246, 129, 0.5 292, 250 and 1 335, 414; 256
    // ranks 0.1 1168, 232 and 1 2332, 967.  Below 2^22 indices (2^20 above 128
    // ranks) the launch shows (2^20, 64 ranks, 0.25: 22, 30; 2^18, 256 ranks, 0.25:
    // 46, 62).
    const uint64_t most = pmax <= 16u ? 16u : (pmax <= 32u ? 1u : (pmax <= 64u ? 2u : (pmax <= 128u ? 4u : 16u)));  // eighths
    const bool pairs = p.N >= (pmax > 128u ? 1u << 20 : 1u << 22) && 8u * p.sum_nnz <= most * p.N;
    a.when = info ? kWhenNodes : (p.speculate_dense ? kWhenUnion : kWhenSparse);
    if (p.speculate_dense) {
        const bool with = info && !pairs;
        shape(acc_tmax(nb, with, pmax));
        if ((e = acc_dense_launch(a, nb, with, s)) != hipSuccess) return e;
    }
    if (a.when != kWhenSparse && pairs) {
        if ((e = acc_pairs_launch(a, p.sum_nnz, s)) != hipSuccess) return e;
    } else if (!p.speculate_dense || !info) {
        const bool nodes = a.when != kWhenSparse;
        shape(acc_tmax(nodes ? nb : 2u, nodes, pmax));
        if ((e = acc_count_launch(a, nodes, s)) != hipSuccess) return e;
    }
    shape(acc_tmax(nb, false, pmax));
    if ((e = acc_write_launch(a, nb, s)) != hipSuccess) return e;
    if (dev_result) return hipSuccess;  // no host round trip
    if ((e = hipMemcpyAsync(res, l.hdr, sizeof(ReduceResult), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    return hipStreamSynchronize(s);
}

}  // namespace sparcml
